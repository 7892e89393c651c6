"""GPU parity of the bf16 grouped GEMMs on either side of the choice between the small-tile kernels and the 256 x 256 one:
few rows per expert (64 x 128 tiles, three stage buffers), few tiles (64 x 128; the weight gradients 128 x 128), many (256 x 256, with a
split contraction under a skewed load).  (Which kernel a size selects is asked, and every kernel reached, in test_gpu_gemm_variants.py;
ragged split contractions are in test_gpu_wgrad_split.py.)  Row counts around the tile edges, column counts off the tile grid, one-row and
empty experts, the row map, routing weights.  Every element against float64, within one bf16 rounding of the result plus
the error bound of an fp32 sum in any order, (n + 2) 2^-24 sum |a||b|."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BF, F32 = torch.bfloat16, torch.float32


@pytest.fixture(scope="module")
def B():
    from paper_2603_07685_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(T=16384, k=8, E=256, h=4096, f_max=4096)
    yield c
    c.close()


FEW = [3, 0, 1, 64, 65, 0, 17] + [2] * 9
EDGE = [63, 0, 64, 65, 1, 127, 128, 129]
WIDE = [257, 255, 1, 0, 700, 640]
BIG = [3000, 1, 0, 2300, 515]
CASES = [(FEW, 320, 192), (FEW, 144, 64), (EDGE, 144, 128), (EDGE, 336, 576), (WIDE, 2320, 1088), (BIG, 3088, 2112)]


class Group:
    def __init__(self, counts, N, K, seed):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        self.counts, self.E, self.N, self.K, self.R = counts, len(counts), N, K, int(sum(counts))
        self.Rcap = self.R + 9
        self.off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
        self.k, self.T = 3, self.R // 3 + 1
        src = torch.randperm(self.T * self.k, generator=g, device="cuda")[: self.Rcap].to(torch.int32)
        self.src = torch.full((self.Rcap,), -1, dtype=torch.int32, device="cuda")
        self.src[: self.R] = src[: self.R]
        self.src[self.R // 2] = -1                           # a padding row inside a group
        r = lambda *s: torch.randn(*s, generator=g, device="cuda").to(BF)
        self.X, self.G, self.W, self.Zsaved = r(self.T, K), r(self.T, N), r(self.E, N, K), r(self.Rcap, 2 * K)
        self.A, self.dC = self.rows(self.X), self.rows(self.G)
        self.p = torch.rand(self.Rcap, generator=g, device="cuda")

    def rows(self, X):
        y = X[torch.div(self.src.clamp(min=0).long(), self.k, rounding_mode="floor")].clone()
        y[self.src < 0] = 0
        return y

    def each(self):
        lo = 0
        for e, c in enumerate(self.counts):
            yield e, slice(lo, lo + c)
            lo += c


def _within(got, ref, mag, n, what, ulp=2.0 ** -8):
    assert torch.isfinite(got).all(), what
    over = (got.double() - ref).abs() - (ulp * ref.abs() + (n + 2) * 2.0 ** -24 * mag + 1e-30)
    assert got.numel() == 0 or float(over.max()) <= 0, (what, float(over.max()))


def _nan(*s, dt=BF):
    return torch.full(s, float("nan"), dtype=dt, device="cuda")


@pytest.mark.parametrize("counts,N,K", CASES)
@pytest.mark.parametrize("gather", [False, True])
def test_forward_and_swiglu(B, ctx, counts, N, K, gather):
    q = Group(counts, N, K, 1)
    f, R = N // 2, q.R
    C, Z, act = _nan(q.Rcap, N), _nan(q.Rcap, N), _nan(q.Rcap, f)
    if gather:
        B.moe_grouped_gemm_fwd_gather(ctx, q.X, q.T, q.src, q.k, q.W, q.off, q.E, N, K, q.Rcap, B.EPI_NONE, None, C, None)
        B.moe_grouped_gemm_fwd_gather(ctx, q.X, q.T, q.src, q.k, q.W, q.off, q.E, N, K, q.Rcap, B.EPI_SWIGLU, q.p, Z, act)
    else:
        B.moe_grouped_gemm_fwd(ctx, q.A, q.W, q.off, q.E, N, K, q.Rcap, B.BF16, B.EPI_NONE, None, None, C, None)
        B.moe_grouped_gemm_fwd_weighted(ctx, q.A, q.W, q.off, q.E, N, K, q.Rcap, B.BF16, B.EPI_SWIGLU, None, None, q.p, Z, act)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    for e, s in q.each():
        a, w = q.A[s].double(), q.W[e].double()
        z, mag = a @ w.T, a.abs() @ w.abs().T
        _within(C[s], z, mag, K, "C")
        _within(Z[s], z, mag, K, "Z")
        g, u, mg, mu = z[:, :f], z[:, f:], mag[:, :f], mag[:, f:]
        sg, p = torch.sigmoid(g), q.p[s, None].double()
        # |silu'| <= 1.1; the hardware sigmoid is good to a few ulps, grown by |g| through its argument
        err = p * (1.1 * u.abs() * mg + (g * sg).abs() * mu) + (16 + 4 * g.abs()) * (p * g * sg * u).abs() / (K + 2)
        _within(act[s], p * g * sg * u, err, K, "act")
    for t in (C, Z, act):
        assert t[R:].isnan().all()


@pytest.mark.parametrize("counts,N,K", CASES)
@pytest.mark.parametrize("gather", [False, True])
def test_data_gradient_and_swiglu_backward(B, ctx, counts, N, K, gather):
    N = (N + 63) // 64 * 64                                  # (the contraction of this call)
    q = Group(counts, N, K, 2)
    R, parts = q.R, 2 * ((K + 255) // 256)
    dA, dZ, part = _nan(q.Rcap, K), _nan(q.Rcap, 2 * K), _nan(q.Rcap, parts, dt=F32)
    if gather:
        B.moe_grouped_gemm_dgrad_gather(ctx, q.G, q.T, q.src, q.k, q.W, q.off, q.E, N, K, q.Rcap, None, None, dA, None)
        B.moe_grouped_gemm_dgrad_gather(ctx, q.G, q.T, q.src, q.k, q.W, q.off, q.E, N, K, q.Rcap, q.Zsaved, q.p, dZ, part)
    else:
        B.moe_grouped_gemm_dgrad(ctx, q.dC, q.W, q.off, q.E, N, K, q.Rcap, B.BF16, None, None, None, dA)
        B.moe_grouped_gemm_dgrad_weighted(ctx, q.dC, q.W, q.off, q.E, N, K, q.Rcap, B.BF16, q.Zsaved, None, None, q.p, dZ, part)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    for e, s in q.each():
        d, w = q.dC[s].double(), q.W[e].double()
        da, mag = d @ w, d.abs() @ w.abs()
        _within(dA[s], da, mag, N, "dA")
        g, u = q.Zsaved[s, :K].double(), q.Zsaved[s, K:].double()
        sg, p = torch.sigmoid(g), q.p[s, None].double()
        rel = (16 + 4 * g.abs()) / (N + 2)                   # rounding of the derivative, in the units of `mag`
        k0, c0, k1 = u * sg * (1 + g * (1 - sg)), u.abs() * sg * (1 + g.abs()), g * sg
        _within(dZ[s, :K], p * da * k0, p * (mag + rel * da.abs()) * c0, N, "dZ gate")
        _within(dZ[s, K:], p * da * k1, p * (mag + rel * da.abs()) * k1.abs(), N, "dZ up")
        dot = k1 * u
        _within(part[s].double().sum(1), (da * dot).sum(1), ((mag + (rel + K / (N + 2)) * da.abs()) * dot.abs()).sum(1), N, "dprob", 0.0)
    for t in (dA, dZ, part):
        assert t[R:].isnan().all()


@pytest.mark.parametrize("counts,N,K", CASES + [([2500, 40, 40, 0, 40, 40], 256, 264), ([9000, 5000] + [100] * 8, 2048, 2048)])
@pytest.mark.parametrize("which", [None, 0, 1])
@pytest.mark.parametrize("f32", [False, True])
def test_weight_gradient(B, ctx, counts, N, K, which, f32):
    q = Group(counts, N, K, 3)
    dt, odt = (F32, B.F32) if f32 else (BF, B.BF16)
    dW = _nan(q.E, N, K, dt=dt)

    def go(acc):
        if which is None:
            B.moe_grouped_gemm_wgrad(ctx, q.A, q.dC, q.off, q.E, N, K, q.Rcap, B.BF16, None, None, acc, odt, dW)
        else:
            A, dC = (q.X, q.dC) if which == B.GATHER_A else (q.A, q.G)
            B.moe_grouped_gemm_wgrad_gather(ctx, A, dC, which, q.T, q.src, q.k, q.off, q.E, N, K, q.Rcap, acc, odt, dW)
        torch.cuda.synchronize()
        assert ctx.poll_error() == 0

    ulp = 2.0 ** -24 if f32 else 2.0 ** -8
    go(0)
    first = dW.clone()
    for e, s in q.each():
        a, d = q.A[s].double(), q.dC[s].double()
        _within(dW[e], d.T @ a, d.abs().T @ a.abs(), counts[e], "dW", ulp)
    go(1)
    for e, s in q.each():
        a, d = q.A[s].double(), q.dC[s].double()
        _within(dW[e], first[e].double() + d.T @ a, d.abs().T @ a.abs() + 2 * first[e].double().abs(), counts[e], "dW accumulated", ulp)


def test_offsets_that_decrease_write_nothing(B, ctx):
    q = Group([40, 20, 30], 128, 64, 4)
    q.off[1] = 70
    C = _nan(q.Rcap, 128)
    B.moe_grouped_gemm_fwd(ctx, q.A, q.W, q.off, 3, 128, 64, q.Rcap, B.BF16, B.EPI_NONE, None, None, C, None)
    torch.cuda.synchronize()
    assert ctx.poll_error() != 0 and C.isnan().all()
