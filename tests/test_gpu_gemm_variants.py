"""Every kernel behind the grouped-GEMM calls on the same rows.  Which one serves a call follows from its sizes, the row capacity
among them, so a call whose rows lie in a larger tensor runs on another kernel: all of them have to give the same bits (they add
a result's products in the same order; the fp32 kernel that splits its operands into bf16 parts does not, and is held to the 64-bit sums
alone), leave what lies behind the rows alone, and lie within the rounding of the output type of 64-bit sums.  The library is asked which kernel a capacity selects; where its rules change so that one is no longer reached, the
tests fail instead of testing less."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

gpu = pytest.mark.gpu
BF, F32, U8, F8 = torch.bfloat16, torch.float32, torch.uint8, torch.float8_e4m3fn
FWD, DGRAD, WGRAD = 0, 1, 2
STORE, SWIGLU, SWIGLU_BWD = 0, 1, 2

# (type, mode, epilogue, N, K): rows, and the kernels that serve it over the capacities
FEW = [65, 0, 1, 64, 129, 0, 17, 300] + [7] * 16                # 24 experts, up to 48 rows each on average: three buffers
SIX = [130, 0, 257, 1, 128, 100]
ROWS = {
    ("bf16", FWD, STORE, 336, 192): (FEW, {0, 1, 2, 3}),
    ("bf16", FWD, SWIGLU, 336, 192): (FEW, {0, 1, 2, 3}),
    ("bf16", DGRAD, STORE, 192, 264): (FEW, {0, 1, 2, 3}),
    ("bf16", DGRAD, SWIGLU_BWD, 2944, 264): (FEW, {0, 1, 2, 3}),
    ("bf16", WGRAD, STORE, 1528, 1512): ([70, 0, 150, 1, 64, 90, 129, 40, 100, 100, 63, 150, 60, 80, 110, 33], {0, 2, 4}),   # (none above
    # twice the mean: those the 256 x 256 kernel would cut)
    ("fp8", FWD, STORE, 768, 256): (SIX, {0, 1, 2}),
    ("fp8", FWD, SWIGLU, 768, 768): (SIX, {0, 1, 2}),
    ("fp8", DGRAD, STORE, 640, 640): (SIX, {0, 1, 2}),
    ("fp8", DGRAD, SWIGLU_BWD, 3840, 1280): (SIX, {0, 1, 2}),
    ("fp8", WGRAD, STORE, 1152, 1152): ([256, 0, 128, 0, 128, 256, 128, 0, 128, 128], {0, 2}),
    ("mx", FWD, STORE, 768, 256): (SIX, {1, 2, 3}),
    ("mx", FWD, SWIGLU, 768, 768): (SIX, {1, 2, 3}),
    ("mx", DGRAD, STORE, 640, 640): (SIX, {1, 2, 3}),
    ("mx", DGRAD, SWIGLU_BWD, 3840, 1280): (SIX, {1, 2, 3}),
    ("mx", WGRAD, STORE, 1408, 640): ([128, 0, 256, 128, 0, 128, 128, 256, 128, 0, 128, 128], {2, 3}),
    ("f32", FWD, STORE, 260, 100): (SIX, {64, 128}),
    ("f32", FWD, STORE, 259, 99): (SIX, {64, 128}),
    ("f32", FWD, SWIGLU, 520, 100): (SIX, {64, 128}),
    ("f32", FWD, SWIGLU, 518, 99): (SIX, {64, 128}),
    ("f32", DGRAD, STORE, 100, 260): (SIX, {64, 128}),
    ("f32", DGRAD, STORE, 99, 259): (SIX, {64, 128}),
    ("f32", DGRAD, SWIGLU_BWD, 100, 260): (SIX, {64, 128}),
    ("f32", DGRAD, SWIGLU_BWD, 99, 259): (SIX, {64, 128}),
    ("f32", WGRAD, STORE, 300, 260): (SIX, {64}),
    ("f32", WGRAD, STORE, 299, 259): (SIX, {64}),
    ("f32", WGRAD, STORE, 1916, 1660): (SIX + [3] * 6, {3, 128}),
    ("f32", WGRAD, STORE, 1915, 1659): (SIX + [3] * 6, {128}),
}
CASES = sorted(ROWS)
DT = {"bf16": 0, "fp8": 1, "f32": 2, "mx": 3}
PARTS = 3   # fp32: the kernel on bf16 parts


def _lib():
    from paper_2603_07685_amd import build
    import os
    if not os.path.exists(build.LIB):
        build.build_library()
    f = ctypes.CDLL(build.LIB).gg_kernel_choice
    f.argtypes = [ctypes.c_int] * 8 + [ctypes.c_longlong]
    return f


def _capacities(case, quant, cu=256):
    """The smallest capacity (a multiple of 128 rows) of a growing series that each kernel serves."""
    dt, mode, epi, N, K = case
    counts, _ = ROWS[case]
    f, seen, r = _lib(), {}, (sum(counts) + 127) // 128 * 128
    while r <= 1 << 17:
        seen.setdefault(f(cu, mode, epi, DT[dt], quant, len(counts), N, K, r), r)
        r = int(r * 1.15) // 128 * 128 + 128
    return seen


@pytest.mark.parametrize("case", CASES, ids=str)
def test_every_kernel_is_reached(case):
    assert set(_capacities(case, 0)) == ROWS[case][1]
    if case[0] in ("fp8", "mx") and case[2] != STORE:
        assert set(_capacities(case, 1)) == ROWS[case][1]


def test_swiglu_backward_tiles():
    """More 128 x 128 tiles than the chip holds at a time: 64 x 128 ones if the contraction is short beside the output phase."""
    f = _lib()
    for E, N, K, R, tile in ((12, 512, 1536, 6000, 1), (8, 512, 512, 16384, 1), (17, 1536, 2048, 4008, 1), (51, 3264, 640, 10230, 2),
                             (32, 4096, 1024, 6144, 2), (16, 2048, 768, 10240, 2)):
        assert f(256, DGRAD, SWIGLU_BWD, DT["bf16"], 0, E, N, K, R) == tile, (E, N, K, R)


def test_other_tests_sizes_reach_their_kernels():
    """The tests of single kernels take sizes that those kernels serve."""
    import test_gpu_f32_split
    import test_gpu_gate_tiles
    import test_gpu_wgrad_single
    f = _lib()
    for counts, N, K in test_gpu_f32_split.CASES:
        for mode, epi in ((FWD, STORE), (FWD, SWIGLU), (DGRAD, STORE), (DGRAD, SWIGLU_BWD), (WGRAD, STORE)):
            assert f(256, mode, epi, DT["f32"], 0, len(counts), N, K, sum(counts) + 3) == PARTS, (counts, N, K, mode, epi)
    for counts, N, K in test_gpu_wgrad_single.CASES:
        assert f(256, WGRAD, STORE, DT["bf16"], 0, len(counts), N, K, sum(counts) + 9) == 4, (counts, N, K)
    from paper_2603_07685_amd import build
    lib = ctypes.CDLL(build.LIB)
    lib.gg_gate_choice.argtypes = [ctypes.c_int] * 4 + [ctypes.c_size_t]
    lib.moe_workspace_bytes.restype = ctypes.c_size_t
    for tile, sizes in test_gpu_gate_tiles.SIZES.items():
        for T, E, h in sizes:
            assert lib.gg_gate_choice(256, T, E, h, lib.moe_workspace_bytes(T, 1, E, h, max(E, 8))) == tile, (T, E, h)


@pytest.fixture(scope="module")
def B():
    from paper_2603_07685_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(T=16384, k=8, E=64, h=4096, f_max=2048)
    yield c
    c.close()


def _codes(g, *s):
    """E4M3 codes of both signs, NaN's excluded."""
    return torch.randint(0, 127, s, dtype=U8, device="cuda", generator=g) | (torch.randint(0, 2, s, dtype=U8, device="cuda", generator=g) << 7)


class _Data:
    """Operands of a case: rows [R, .] without slack, weights, and their values in float64."""

    def __init__(self, case, seed=5):
        dt, mode, epi, N, K = case
        self.case, self.counts = case, ROWS[case][0]
        self.E, self.R = len(self.counts), sum(self.counts)
        self.off = torch.tensor(np.concatenate([[0], np.cumsum(self.counts)]), dtype=torch.int32, device="cuda")
        g = torch.Generator("cuda").manual_seed(seed)
        n = lambda *s: torch.randn(s, device="cuda", generator=g)
        R, E = self.R, self.E
        widths = {FWD: (K,), DGRAD: (N,), WGRAD: (N, K)}[mode]           # the operands with rows: dC before A
        self.rows, self.row_scales, self.row_vals = [], [], []
        for w in widths:
            if dt in ("bf16", "f32"):
                x = n(R, w).to(BF if dt == "bf16" else F32)
                v, s = x.double(), None
            else:
                x = _codes(g, R, w)
                v = x.view(F8).double()
                if dt == "mx":
                    if mode == WGRAD:
                        s = torch.randint(124, 130, (R // 128, w, 4), dtype=U8, device="cuda", generator=g)
                        v = v * torch.exp2(s.double() - 127).permute(0, 2, 1).reshape(R // 32, w).repeat_interleave(32, 0)
                    else:
                        s = torch.randint(124, 130, (R, w // 32), dtype=U8, device="cuda", generator=g)
                        v = v * torch.exp2(s.double() - 127).repeat_interleave(32, 1)
                elif mode == WGRAD:
                    s = torch.rand((R // 128, w), device="cuda", generator=g) + 0.5
                    v = v * s.double().repeat_interleave(128, 0)
                else:
                    s = torch.rand((R, w // 128), device="cuda", generator=g) + 0.5
                    v = v * s.double().repeat_interleave(128, 1)
            self.rows.append(x)
            self.row_scales.append(s)
            self.row_vals.append(v)
        self.W = self.sW = None
        if mode != WGRAD:
            if dt in ("bf16", "f32"):
                self.W = n(E, N, K).to(BF if dt == "bf16" else F32)
                self.Wv = self.W.double()
            else:
                self.W = _codes(g, E, N, K)
                self.Wv = self.W.view(F8).double()
                if dt == "fp8":
                    self.sW = torch.rand((E, N // 128, K // 128), device="cuda", generator=g) + 0.5
                    self.Wv = self.Wv * self.sW.double().repeat_interleave(128, 1).repeat_interleave(128, 2)
                elif mode == FWD:
                    self.sW = torch.randint(120, 126, (E, N, K // 32), dtype=U8, device="cuda", generator=g)
                    self.Wv = self.Wv * torch.exp2(self.sW.double() - 127).repeat_interleave(32, 2)
                else:
                    self.sW = torch.randint(120, 126, (E * N // 128, K, 4), dtype=U8, device="cuda", generator=g)
                    self.Wv = self.Wv * torch.exp2(self.sW.double() - 127).permute(0, 2, 1).reshape(E, N // 32, K).repeat_interleave(32, 1)
        self.Z = n(R, 2 * K).to(F32 if dt == "f32" else BF) if epi == SWIGLU_BWD else None
        self.p = torch.rand(R, device="cuda", generator=g)
        # a row map of three slots per token for the gathered calls; some rows without a source
        self.k, self.T = 3, R // 3 + 7
        self.src = torch.randperm(self.T * self.k, device="cuda", generator=g)[:R].to(torch.int32)
        self.src[::37] = -1

    def each(self):
        for e in range(self.E):
            a, b = int(self.off[e]), int(self.off[e + 1])
            yield e, slice(a, b)


def _slack(t, rows, fill=None):
    """t with rows appended (of whatever the allocator holds, or `fill`) up to `rows`."""
    if t is None:
        return None
    out = torch.empty((rows, *t.shape[1:]), dtype=t.dtype, device="cuda") if fill is None else \
        torch.full((rows, *t.shape[1:]), fill, dtype=t.dtype, device="cuda")
    out[:t.shape[0]] = t
    return out


def _run(B, ctx, d, cap, gather=None, out_f32=False):
    """One call at a capacity; its outputs' live rows (weight gradients: all of them)."""
    dt, mode, epi, N, K = d.case
    E, R, off = d.E, d.R, d.off
    D = getattr(B, {"bf16": "BF16", "f32": "F32", "fp8": "FP8_E4M3", "mx": "MXFP8_E4M3"}[dt])
    ot = F32 if dt == "f32" else BF
    new = lambda *s, t=ot: torch.full(s, 0xA5 if t == U8 else -3.0, dtype=t, device="cuda")
    rows = [x if gather and i == (0 if mode != WGRAD or gather == "dC" else 1) else _slack(x, cap) for i, x in enumerate(d.rows)]
    src = _slack(d.src, cap, -1)
    scales = [_slack(s, cap if mode != WGRAD else cap // 128) for s in d.row_scales]
    if gather:   # the operand in token order: row t of it for slot 0, 1, 2
        i = 0 if mode != WGRAD or gather == "dC" else 1
        tok = torch.randn((d.T, d.rows[i].shape[1]), device="cuda", generator=torch.Generator("cuda").manual_seed(9)).to(BF)
        rows[i] = tok
    if mode == WGRAD:
        out = torch.full((E, N, K), -3.0, dtype=F32 if out_f32 or dt == "f32" else BF, device="cuda")
        odt = B.F32 if out.dtype == F32 else B.BF16
        if gather:
            B.moe_grouped_gemm_wgrad_gather(ctx, rows[1], rows[0], B.GATHER_A if gather == "A" else B.GATHER_DC, d.T, src, d.k, off, E, N,
                                            K, cap, False, odt, out)
        else:
            B.moe_grouped_gemm_wgrad(ctx, rows[1], rows[0], off, E, N, K, cap, D, scales[1], scales[0], False, odt, out)
        return [out]
    p, quant = _slack(d.p, cap), dt in ("fp8", "mx") and epi != STORE
    if mode == FWD:
        outs = [new(cap, N)] + ([new(cap, N // 2)] if epi == SWIGLU else [])
        C, act = outs[0], outs[1] if epi == SWIGLU else None
        cols, arg = N // 2, B.EPI_SWIGLU if epi == SWIGLU else B.EPI_NONE
    else:
        parts = new(cap, 2 * ((K + 255) // 256), t=F32) if epi == SWIGLU_BWD and dt != "f32" else None
        outs = [new(cap, 2 * K if epi == SWIGLU_BWD else K)] + ([parts] if parts is not None else [])
        cols = 2 * K
    Z = _slack(d.Z, cap)
    pr = p if epi != STORE else None
    if gather and mode == FWD:
        B.moe_grouped_gemm_fwd_gather(ctx, rows[0], d.T, src, d.k, d.W, off, E, N, K, cap, arg, pr, C, act)
    elif gather:
        B.moe_grouped_gemm_dgrad_gather(ctx, rows[0], d.T, src, d.k, d.W, off, E, N, K, cap, Z, pr, outs[0], parts)
    elif not quant and mode == FWD:
        B.moe_grouped_gemm_fwd_weighted(ctx, rows[0], d.W, off, E, N, K, cap, D, arg, scales[0], d.sW, pr, C, act)
    elif not quant:
        B.moe_grouped_gemm_dgrad_weighted(ctx, rows[0], d.W, off, E, N, K, cap, D, Z, scales[0], d.sW, pr, outs[0], parts)
    elif dt == "fp8":
        q = [new(cap, cols, t=U8), new(cap, cols // 128, t=F32)]
        if mode == FWD:
            B.moe_grouped_gemm_fwd_quant(ctx, rows[0], d.W, off, E, N, K, cap, D, arg, scales[0], d.sW, pr, C, act, *q)
        else:
            B.moe_grouped_gemm_dgrad_quant(ctx, rows[0], d.W, off, E, N, K, cap, D, Z, scales[0], d.sW, pr, outs[0], parts, *q)
        outs += q
    else:
        q = [new(cap, cols, t=U8), new(cap, cols // 32, t=U8)]
        if mode == FWD:
            B.moe_grouped_gemm_fwd_quant_mx(ctx, rows[0], d.W, off, E, N, K, cap, scales[0], d.sW, pr, C, act, *q, None, None)
        else:
            B.moe_grouped_gemm_dgrad_quant_mx(ctx, rows[0], d.W, off, E, N, K, cap, Z, scales[0], d.sW, pr, outs[0], parts, *q, None, None)
        outs += q
    for t in outs:
        assert (t[R:] == (0xA5 if t.dtype == U8 else -3.0)).all()
    return [t[:R].clone() for t in outs]


def _reference(d, gather):
    """The first output (and the activation, if there is one) in float64."""
    dt, mode, epi, N, K = d.case
    vals = list(d.row_vals)
    if gather:
        i = 0 if mode != WGRAD or gather == "dC" else 1
        tok = torch.randn((d.T, d.rows[i].shape[1]), device="cuda", generator=torch.Generator("cuda").manual_seed(9)).to(BF)
        x = tok[(d.src.clamp(min=0) // d.k).long()].double()
        x[d.src < 0] = 0
        vals[i] = x
    if mode == WGRAD:
        return [torch.stack([vals[0][s].t().contiguous() @ vals[1][s] for _, s in d.each()])]
    outs = [torch.cat([vals[0][s] @ (d.Wv[e].t().contiguous() if mode == FWD else d.Wv[e]) for e, s in d.each()])]
    p = d.p.double()[:, None]
    if epi == SWIGLU:
        g, u = outs[0].chunk(2, 1)
        outs.append(p * g * torch.sigmoid(g) * u)
    elif epi == SWIGLU_BWD:
        g, u = d.Z.double().chunk(2, 1)
        s, da = torch.sigmoid(g), outs[0]
        outs = [torch.cat([p * da * u * s * (1 + g * (1 - s)), p * da * g * s], 1)]
        if dt != "f32":
            outs.append((da * g * s * u).sum(1))
    return outs


# relative 2-norm of the error: bf16 results are rounded once (2^-9 at most, about 0.4 of that on average); one-byte operands
# lose what the matrix unit drops of a group of eight products besides (2^-11 of the largest at most); fp32: sums of up to 300
# roundings of 2^-24 and the same of two factors
BOUND = {"bf16": 2.0 ** -9, "fp8": 2.0 ** -8, "mx": 2.0 ** -8, "f32": 4e-6}


@gpu
@pytest.mark.parametrize("case,gather", [(c, g) for c in CASES for g in
                                         ([None] if c[0] != "bf16" else [None, "rows"] if c[1] != WGRAD else [None, "A", "dC"])], ids=str)
def test_all_kernels_agree(B, ctx, case, gather):
    dt, mode, epi, N, K = case
    d = _Data(case)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    caps = _capacities(case, int(dt in ("fp8", "mx") and epi != STORE), cu)
    if cu == 256:
        assert set(caps) == ROWS[case][1]
    for out_f32 in ([False, True] if mode == WGRAD and dt != "f32" else [False]):
        res = {t: _run(B, ctx, d, r, gather, out_f32) for t, r in caps.items()}
        torch.cuda.synchronize()
        assert ctx.poll_error() == 0
        first = res[min(t for t in res if dt != "f32" or t != PARTS)]
        bound = 2e-6 * np.sqrt(max(d.counts)) if out_f32 and dt == "bf16" else BOUND[dt]
        refs = _reference(d, gather)
        for outs in [first] + ([res[PARTS]] if dt == "f32" and PARTS in res else []):
            for got, ref in zip(outs, refs):
                g = got.double().sum(1) if ref.dim() == 1 else got.double()
                assert ((g - ref).norm() / ref.norm()).item() <= (4 * BOUND[dt] if ref.dim() == 1 else bound)
        for t, outs in res.items():
            if dt == "f32" and t == PARTS:
                continue
            for i, (a, b) in enumerate(zip(first, outs)):
                if a.dtype == F32 and mode == DGRAD and i == 1 and a.shape[1] == 2 * ((K + 255) // 256):
                    # partial <dA, act> of a row: other groups of columns, the same fp32 terms
                    assert torch.allclose(a.double().sum(1), b.double().sum(1), rtol=0, atol=1e-5 * float(a.abs().sum(1).max())), t
                else:
                    assert torch.equal(a.view(U8), b.view(U8)), (t, i)
