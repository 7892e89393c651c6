"""The quantised copies that go with a one-byte grouped GEMM call cover exactly the rows the GEMM covers: none where it
refuses the offsets (they leave the tensor, fall, or, with the 32x1 copy, lie off the 128-row grid), and offsets[0] ..
offsets[E] - 1 of a call on a part of the tensor."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

R, E, N, K = 640, 4, 512, 256     # fc1: [R, K] -> [R, N], activation [R, N / 2]; fc2 data gradient: [R, N] -> dZ [R, 2 K]
REFUSED = {"beyond": [0, 128, 256, 512, R + 128], "falling": [0, 256, 128, 384, 512], "before": [-128, 128, 256, 384, 512],
           "off_grid": [0, 120, 256, 384, 512]}


@pytest.fixture(scope="module")
def B():
    from paper_2603_07685_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(T=256, k=2, E=8, h=512, f_max=512)
    yield c
    c.close()


def _call(B, ctx, recipe, fwd, offsets):
    """Runs one call into buffers of a known filling; returns the stored bf16 tensor, its copies and their fillings."""
    g = torch.Generator("cuda").manual_seed(len(recipe) + fwd)
    b8 = lambda *s: torch.randint(0, 120, s, dtype=torch.uint8, device="cuda", generator=g)
    mx = recipe != "fp8"
    sc = (lambda *s: torch.randint(124, 130, s, dtype=torch.uint8, device="cuda", generator=g)) if mx else \
        (lambda *s: torch.rand(s, device="cuda", generator=g) + 0.5)
    C, cols = (K, N // 2) if fwd else (N, 2 * K)
    A, W = b8(R, C), b8(E, N, K)
    sa = sc(R, C // 32) if mx else sc(R, C // 128)
    if not mx:
        sw = sc(E, N // 128, K // 128)
    else:
        sw = sc(E, N, K // 32) if fwd else sc(E * N // 128, K, 4)
    o = torch.tensor(offsets, dtype=torch.int32, device="cuda")
    full = lambda *s, t=torch.uint8: torch.full(s, 0xA5 if t == torch.uint8 else -3, dtype=t, device="cuda")
    stored = torch.full((R, cols), -7, dtype=torch.bfloat16, device="cuda")
    Z = torch.randn((R, 2 * K), device="cuda", generator=g).bfloat16()
    if not mx:
        q, s = full(R, cols), full(R, cols // 128, t=torch.float32)
        copies = [q, s]
        if fwd:
            B.moe_grouped_gemm_fwd_quant(ctx, A, W, o, E, N, K, R, B.FP8_E4M3, B.EPI_SWIGLU, sa, sw, None, None, stored, q, s)
        else:
            B.moe_grouped_gemm_dgrad_quant(ctx, A, W, o, E, N, K, R, B.FP8_E4M3, Z, sa, sw, None, stored, None, q, s)
    else:
        col = recipe == "mx_col"
        copies = [full(R, cols), full(R, cols // 32)] + ([full(R, cols), full(R // 128, cols, 4)] if col else [])
        args = copies + ([] if col else [None, None])
        if fwd:
            B.moe_grouped_gemm_fwd_quant_mx(ctx, A, W, o, E, N, K, R, sa, sw, None, None, stored, *args)
        else:
            B.moe_grouped_gemm_dgrad_quant_mx(ctx, A, W, o, E, N, K, R, Z, sa, sw, None, stored, None, *args)
    return stored, copies


@pytest.mark.parametrize("fwd", [True, False])
@pytest.mark.parametrize("recipe,kind", [(r, k) for r in ("fp8", "mx", "mx_col") for k in REFUSED if k != "off_grid" or r == "mx_col"])
def test_refused_offsets_leave_the_copies_alone(B, ctx, recipe, kind, fwd):
    ctx.poll_error()
    stored, copies = _call(B, ctx, recipe, fwd, REFUSED[kind])
    assert ctx.poll_error() == 1 and (stored == -7).all()
    for c in copies:
        assert (c == (0xA5 if c.dtype == torch.uint8 else -3)).all()


@pytest.mark.parametrize("fwd", [True, False])
@pytest.mark.parametrize("recipe", ["fp8", "mx", "mx_col"])
def test_a_part_of_the_tensor(B, ctx, recipe, fwd):
    part = [128, 256, 256, 384, 512] if recipe == "mx_col" else [57, 200, 200, 311, 450]
    lo, hi = part[0], part[-1]
    stored, copies = _call(B, ctx, recipe, fwd, part)
    want = [torch.empty_like(c) for c in copies]
    if recipe == "fp8":
        B.moe_fp8_quantize(ctx, stored, B.Q_1x128, 1, R, stored.shape[1], None, *want)
    elif recipe == "mx":
        B.moe_mx_quantize(ctx, stored, B.MX_1x32, 1, R, stored.shape[1], None, *want)
    else:
        B.moe_mx_quantize_rowcol(ctx, stored, R, stored.shape[1], None, *want)
    assert ctx.poll_error() == 0
    for c, w in zip(copies, want):
        a, b = (lo // 128, hi // 128) if c.shape[0] == R // 128 else (lo, hi)
        fill = 0xA5 if c.dtype == torch.uint8 else -3
        assert torch.equal(c[a:b], w[a:b]) and (c[:a] == fill).all() and (c[b:] == fill).all()
