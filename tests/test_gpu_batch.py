"""Calls of a batch (moe_batch_create) against the same calls on their context, bit for bit: every kernel that serves several
calls in one launch, with uneven numbers of them, and what a batch promises beside the results."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


class _Alone:
    """In the batch's place: every call on the context itself."""

    def __init__(self, ctx):
        self.ctx = ctx

    def __enter__(self):
        return self.ctx

    def __exit__(self, *exc):
        pass


# sizes: tiles of 64 rows with two and three stage buffers, weight gradients on one and two, a routed and a shared expert of unlike
# sizes, calls that are launched at once beside ones that are kept, ragged columns
SIZES = [
    dict(T=96, h=128, f=64, E=4, k=2, sf=64),
    dict(T=1000, h=448, f=320, E=6, k=2, sf=192),
    dict(T=64, h=576, f=384, E=48, k=4, sf=1024),       # (one stage buffer for the routed weight gradients)
    dict(T=2048, h=1024, f=512, E=8, k=2, sf=512),
    dict(T=700, h=2048, f=1536, E=5, k=4, sf=192),      # (routed calls beyond the small tiles)
]


def _layers(size, shared, **kw):
    from paper_2603_07685_amd import layer as L
    from paper_2603_07685_amd import workloads as wl
    recipe = kw.pop("recipe", "bf16")
    cfg = wl.MoEConfig("batch", T=size["T"], h=size["h"], f=size["f"], E=size["E"], k=size["k"], E_router=size["E"],
                       score=wl.SOFTMAX, norm_topk=False, load="router", shared_f=size["sf"] if shared else 0,
                       fp8=recipe == "fp8", mx=recipe == "mxfp8", align=1 if recipe in ("bf16", "fp32") else 128, seed=5)
    hin = L.host_inputs(cfg) if recipe == "fp32" else None
    pair = [L.LayerState(cfg, hin, f32=recipe == "fp32", **kw) for _ in range(2)]
    pair[1].batch = _Alone(pair[1].ctx)
    return pair


OUT = ("Y", "A", "Z", "O", "dX", "dZ", "dW1", "dW2", "dprob")
QUANT = ("qXp", "sXp", "qXpc", "sXpc", "qA", "sA", "qAc", "sAc", "qdO", "sdO", "qdOc", "sdOc", "qdZ", "sdZ", "qdZc", "sdZc", "qW1", "sW1",
         "qW2d", "sW2d", "qWs1", "sWs1", "qWs2d", "sWs2d", "qX", "sX", "qXc", "qAs", "qAsc", "sAsc", "qdY", "sdYc", "qdZs", "qdZsc", "sdZsc")
SHARED = ("S", "As", "Zs", "dZs", "dXs", "dWs1", "dWs2")


def _compare(pair, shared):
    for st in pair:
        for n in OUT + (SHARED if shared else ()):
            getattr(st, n).zero_()
        st.step()
    torch.cuda.synchronize()
    a, b = pair
    assert a.ctx.poll_error() == 0 and b.ctx.poll_error() == 0
    for n in OUT + (SHARED if shared else ()):
        assert torch.equal(getattr(a, n), getattr(b, n)), n


@pytest.mark.parametrize("size", range(len(SIZES)))
@pytest.mark.parametrize("kw", [{}, dict(wgrad_f32=True), dict(gather=True), dict(eq2=True), dict(eq2=True, gather=True, wgrad_f32=True)],
                         ids=lambda kw: "+".join(kw) or "plain")
@pytest.mark.parametrize("shared", [False, True])
def test_layer_is_that_of_single_calls(size, kw, shared):
    _compare(_layers(SIZES[size], shared, **kw), shared)


@pytest.mark.parametrize("size", [0, 1, 2, 3])
@pytest.mark.parametrize("shared", [False, True])
def test_fp32_layer_is_that_of_single_calls(size, shared):
    _compare(_layers(SIZES[size], shared, recipe="fp32"), shared)


@pytest.mark.parametrize("size", range(len(SIZES)))
@pytest.mark.parametrize("kw", [{}, dict(wgrad_f32=True), dict(eq2=True), dict(epilogue_quant=True), dict(fp8_wgrad=False)],
                         ids=lambda kw: "+".join(kw) or "plain")
@pytest.mark.parametrize("recipe", ["fp8", "mxfp8"])
def test_one_byte_layer_is_that_of_single_calls(recipe, size, kw):
    if recipe == "mxfp8" and ("epilogue_quant" in kw or "fp8_wgrad" in kw):
        kw = dict(epilogue_quant=False)
    up = lambda n: (n + 127) // 128 * 128
    s = {n: v if n in ("E", "k") else up(v) for n, v in SIZES[size].items()}
    pair = _layers(s, True, recipe=recipe, **kw)
    for st in pair:
        for n in OUT + SHARED + QUANT:
            t = getattr(st, n)
            if t is not None:
                t.zero_()
        st.step()
    torch.cuda.synchronize()
    a, b = pair
    assert a.ctx.poll_error() == 0 and b.ctx.poll_error() == 0
    for n in OUT + SHARED + QUANT:
        t = getattr(a, n)
        assert t is None or torch.equal(t, getattr(b, n)), n


def test_what_is_kept_and_what_is_not():
    """Kept calls are launched at the end and not before, more of them than a batch holds are launched on the way, dropped ones never."""
    from paper_2603_07685_amd import binding as B
    T, K, N, n = 256, 128, 256, 21
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    A = torch.randn((T, K), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((n, N, K), generator=g, device="cuda").to(torch.bfloat16)
    off = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    ctx = B.Context(T, 1, 1, K, N)
    batch = B.Batch(ctx)
    want, got = (torch.full((n, T, N), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))

    def calls(c, out):
        for i in range(n):
            B.moe_grouped_gemm_fwd(c, A, W[i], off, 1, N, K, T, B.BF16, B.EPI_NONE, None, None, out[i], None)

    calls(ctx, want)
    with batch as b:
        calls(b, got)
        torch.cuda.synchronize()
        assert (got[-1] == 7).all()
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    got.fill_(7.0)
    with pytest.raises(B.MoeError):
        with batch as b:
            B.moe_grouped_gemm_fwd(b, A, W[0], off, 1, N, K, T, B.BF16, B.EPI_NONE, None, None, got[0], None)
            B.moe_grouped_gemm_fwd(b, A, W[1], off, 1, N, 7, T, B.BF16, B.EPI_NONE, None, None, got[1], None)
    with batch as b:
        B.moe_grouped_gemm_fwd(b, A, W[2], off, 1, N, K, T, B.BF16, B.EPI_NONE, None, None, got[2], None)
    torch.cuda.synchronize()
    assert (got[0] == 7).all() and (got[1] == 7).all() and torch.equal(got[2], want[2])


@pytest.mark.parametrize("at", [0, 1, 2])
def test_offsets_of_any_call_are_checked(at):
    """Offsets that fall: the error word is set and that call writes nothing, wherever it stands in the launch; the others are served."""
    from paper_2603_07685_amd import binding as B
    T, K, N = 192, 128, 256
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    A = torch.randn((T, K), generator=g, device="cuda").to(torch.bfloat16)
    dC = torch.randn((T, N), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((2, N, K), generator=g, device="cuda").to(torch.bfloat16)
    good = torch.tensor([0, 64, T], dtype=torch.int32, device="cuda")
    bad = torch.tensor([0, 128, 64], dtype=torch.int32, device="cuda")
    ctx = B.Context(T, 1, 2, K, N)
    dA = torch.full((2, T, K), 7.0, dtype=torch.bfloat16, device="cuda")
    dW = torch.full((2, N, K), 7.0, dtype=torch.bfloat16, device="cuda")
    with B.Batch(ctx) as b:
        for i in range(2):
            B.moe_grouped_gemm_dgrad(b, dC, W, bad if at == i else good, 2, N, K, T, B.BF16, None, None, None, dA[i])
        B.moe_grouped_gemm_wgrad(b, A, dC, bad if at == 2 else good, 2, N, K, T, B.BF16, None, None, 0, B.BF16, dW)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 1
    for i, t in enumerate((dA[0], dA[1], dW)):
        assert bool((t == 7).all()) == (i == at), i


def _gradient_in_pieces(N, K, R, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    A, dC = (torch.randn((R, n), generator=g, device="cuda").to(torch.bfloat16) for n in (K, N))
    return A, dC, torch.tensor([0, R], dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("width", [512, 2048], ids=["room for one", "room for all"])
def test_weight_gradients_in_pieces_side_by_side(width, f32):
    """Three weight gradients whose contraction is cut into pieces and a data gradient: their partial results lie side by side, or, where
    the workspace has no room for the next, what is kept goes first."""
    from paper_2603_07685_amd import binding as B
    N, K = 1024, 512
    dt = B.F32 if f32 else B.BF16
    new = lambda: torch.full((N, K), float("nan"), dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
    ops = [_gradient_in_pieces(N, K, R, 7 + R) for R in (2048, 3000, 2500)]
    ctx, bare = B.Context(T=64, k=1, E=1, h=width, f_max=512), B.Context(T=64, k=1, E=1, h=0, f_max=0)
    W = torch.randn((N, K), device="cuda").to(torch.bfloat16)

    def weight(c, o, out):
        A, dC, off = o
        B.moe_grouped_gemm_wgrad(c, A, dC, off, 1, N, K, A.shape[0], B.BF16, None, None, 0, dt, out)

    def data(c, out):
        B.moe_grouped_gemm_dgrad(c, ops[0][1], W, ops[0][2], 1, N, K, 2048, B.BF16, None, None, None, out)

    want, whole, got = ([new() for _ in ops] for _ in range(3))
    dwant, dgot = (torch.zeros((2048, K), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    for o, w, v in zip(ops, want, whole):
        weight(ctx, o, w)
        weight(bare, o, v)
    data(ctx, dwant)
    if f32:
        assert not any(torch.equal(w, v) for w, v in zip(want, whole))   # (cut: other sums)
    batch = B.Batch(ctx)
    for _ in range(3):                     # (the room is used again)
        for t in got:
            t.fill_(float("nan"))
        dgot.zero_()
        with batch as b:
            for o, t in zip(ops, got):
                weight(b, o, t)
            data(b, dgot)
            torch.cuda.synchronize()
            assert [bool(t.isnan().all()) for t in got] == [width == 2048, width == 2048, True]
        assert torch.equal(dgot, dwant)
        for t, w in zip(got, want):
            assert torch.equal(t, w)
    assert ctx.poll_error() == 0 and batch.kept() == (12, 0)


@pytest.mark.parametrize("recipe", ["bf16", "fp32", "fp8", "mxfp8"])
@pytest.mark.parametrize("size", [1, 2, 3])
def test_hot_and_empty_experts(recipe, size):
    """95 % of the pairs on one expert, some experts without rows, the first and the last among them."""
    up = (lambda n: (n + 127) // 128 * 128) if recipe in ("fp8", "mxfp8") else (lambda n: n)
    s = {n: v if n in ("E", "k") else up(v) for n, v in SIZES[size].items()}
    pair = _layers(s, True, recipe=recipe)
    g = torch.Generator()
    g.manual_seed(size)
    idx = torch.randint(1, s["E"] - 1, (s["T"], s["k"]), generator=g)
    idx[idx == 2] = 1
    idx[torch.rand(idx.shape, generator=g) < 0.95] = s["E"] - 2
    for st in pair:
        st.forced_idx = idx.to(torch.int32).cuda()
    _compare(pair, True)
    assert pair[0].counts.tolist() == torch.bincount(idx.flatten(), minlength=s["E"]).tolist()


@pytest.mark.parametrize("recipe", ["bf16", "fp32", "fp8", "mxfp8"])
def test_captured_step_with_a_shared_expert(recipe):
    """A step captured in a graph, batches and all: every replay gives the eager step's bits, on other loads too."""
    pair = _layers(dict(T=512, h=256, f=128, E=6, k=2, sf=128), True, recipe=recipe)
    st, eager = pair[0], pair[1]
    names = OUT + SHARED
    loads = [torch.randint(0, e, (512, 2), dtype=torch.int32, device="cuda") for e in (6, 2, 4)]
    st.forced_idx = loads[0].clone()
    st.step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        st.step()
    for i in (1, 0, 2, 2):
        st.forced_idx.copy_(loads[i])
        eager.forced_idx = loads[i]
        eager.step()
        for n in names:
            getattr(st, n).zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        live = int(eager.offsets[-1])      # (rows behind the last expert hold what an earlier load has left there)
        for n in names:
            a, b = getattr(st, n), getattr(eager, n)
            assert torch.equal(a[:live], b[:live]) if n in ("A", "Z", "O", "dZ") else torch.equal(a, b), (i, n)
    assert st.ctx.poll_error() == 0 and eager.ctx.poll_error() == 0
