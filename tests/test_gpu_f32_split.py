"""GPU parity of the fp32 grouped GEMMs that split their operands into bf16 parts, at the edges of their tiles and stages: calls
large enough to take that kernel, one-row and empty experts, contractions and columns off the 32 / 64 / 128 grid, and operands
that three bf16 parts cannot hold (infinities, NaN, the top of the range, magnitudes below 2^-110), whose tiles are computed
on the fp32 instruction.  Every element against float64, within the bound of an fp32 dot product summed in any order:
|error| <= (n + 2) 2^-24 sum |a||b|."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from test_gpu_f32_gemm import EPS, _case, _rows, _within


@pytest.fixture(scope="module")
def B():
    from paper_2603_07685_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(T=4096, k=2, E=8, h=1024, f_max=1024)
    yield c
    c.close()


# counts per expert, N, K: both forwards, both data gradients and the weight gradient take the split kernel
CASES = [
    ([1100, 0, 31, 500], 1016, 772),        # a last column tile of 120 (SwiGLU 60), stages that end after 4 and 24 elements
    ([2048, 1, 63, 65, 1200], 640, 1024),   # whole stages; 200 weight-gradient tiles
    ([1537], 2048, 1664),
]


@pytest.mark.parametrize("counts,N,K", CASES)
def test_split_forward_and_data_gradient(B, ctx, counts, N, K):
    off, R, Rcap, A, W, dC = _case(counts, N, K, 7)
    E, nan = len(counts), float("nan")
    C = torch.full((Rcap, N), nan, device="cuda")
    dA = torch.full((Rcap, K), nan, device="cuda")
    Z = torch.full((Rcap, N), nan, device="cuda")
    act = torch.full((Rcap, N // 2), nan, device="cuda")
    dZ = torch.full((Rcap, 2 * K), nan, device="cuda")
    Zs = torch.randn(Rcap, 2 * K, device="cuda")
    B.moe_grouped_gemm_fwd(ctx, A, W, off, E, N, K, Rcap, B.F32, B.EPI_NONE, None, None, C, None)
    B.moe_grouped_gemm_fwd(ctx, A, W, off, E, N, K, Rcap, B.F32, B.EPI_SWIGLU, None, None, Z, act)
    B.moe_grouped_gemm_dgrad(ctx, dC, W, off, E, N, K, Rcap, B.F32, None, None, None, dA)
    B.moe_grouped_gemm_dgrad(ctx, dC, W, off, E, N, K, Rcap, B.F32, Zs, None, None, dZ)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    for e, s in _rows(counts):
        a, w, d = A[s].double(), W[e].double(), dC[s].double()
        bc = (K + 2) * EPS * (a.abs() @ w.abs().T)
        _within(C[s], a @ w.T, bc)
        _within(Z[s], a @ w.T, bc)
        g, u = Z[s, :N // 2].double(), Z[s, N // 2:].double()
        ref = g * torch.sigmoid(g) * u
        _within(act[s], ref, (16 + 4 * g.abs()) * EPS * ref.abs() + 1e-30)
        da, bd = d @ w, (N + 2) * EPS * (d.abs() @ w.abs())
        _within(dA[s], da, bd)
        g, u = Zs[s, :K].double(), Zs[s, K:].double()
        sg, rel = torch.sigmoid(g), (16 + 4 * g.abs()) * EPS
        cancel = u.abs() * sg * (1 + g.abs())
        _within(dZ[s, :K], da * u * sg * (1 + g * (1 - sg)), bd * cancel + rel * da.abs() * cancel + 1e-30)
        _within(dZ[s, K:], da * g * sg, bd * (g * sg).abs() + rel * (da * g * sg).abs() + 1e-30)
    for t in (C, Z, act, dA, dZ):
        assert t[R:].isnan().all()


@pytest.mark.parametrize("counts,N,K", CASES)
@pytest.mark.parametrize("accumulate", [0, 1])
def test_split_weight_gradient(B, ctx, counts, N, K, accumulate):
    off, R, Rcap, A, W, dC = _case(counts, N, K, 9)
    dB = W.clone() if accumulate else torch.full_like(W, float("nan"))
    B.moe_grouped_gemm_wgrad(ctx, A, dC, off, len(counts), N, K, Rcap, B.F32, None, None, accumulate, B.F32, dB)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    for e, s in _rows(counts):
        a, d = A[s].double(), dC[s].double()
        ref, bound = d.T @ a, (counts[e] + 2) * EPS * (d.abs().T @ a.abs())
        if accumulate:
            ref, bound = ref + W[e].double(), bound + 2 * EPS * (W[e].double().abs() + ref.abs())
        _within(dB[e], ref, bound)


@pytest.mark.parametrize("scale_a,scale_w", [(2.0 ** -118, 1.0), (2.0 ** -118, 2.0 ** 100), (2.0 ** 63, 2.0 ** 56), (2.0 ** -60, 2.0 ** -60)])
def test_split_magnitudes(B, ctx, scale_a, scale_w):
    """Whole rows of tiny and of huge values: tiles beside ordinary ones, each within the bound at its own scale."""
    counts, N, K = CASES[0]
    off, R, Rcap, A, W, _ = _case(counts, N, K, 11)
    A[100:140] *= scale_a
    W[:, 64:70] *= scale_w
    C = torch.full((Rcap, N), float("nan"), device="cuda")
    B.moe_grouped_gemm_fwd(ctx, A, W, off, len(counts), N, K, Rcap, B.F32, B.EPI_NONE, None, None, C, None)
    torch.cuda.synchronize()
    for e, s in _rows(counts):
        a, w = A[s].double(), W[e].double()
        # (2^-149 per addition: results below the normal range)
        _within(C[s], a @ w.T, (K + 2) * (EPS * (a.abs() @ w.abs().T) + 2.0 ** -149))


def test_split_infinities_and_nan(B, ctx):
    counts, N, K = CASES[0]
    off, R, Rcap, A, W, dC = _case(counts, N, K, 12)
    inf = float("inf")
    A[5, 7], A[300, 0], A[301, 1], W[0, 900, 3], W[2, 10, K - 1] = inf, -inf, float("nan"), inf, 3.4e38
    A[1100:1131, K - 1] = 2.0
    C = torch.zeros((Rcap, N), device="cuda")
    dB = torch.zeros_like(W)
    B.moe_grouped_gemm_fwd(ctx, A, W, off, len(counts), N, K, Rcap, B.F32, B.EPI_NONE, None, None, C, None)
    B.moe_grouped_gemm_wgrad(ctx, A, dC, off, len(counts), N, K, Rcap, B.F32, None, None, 0, B.F32, dB)
    torch.cuda.synchronize()
    for got, ref in [(C[s], (A[s].double() @ W[e].double().T).float()) for e, s in _rows(counts)] + \
                    [(dB[e], (dC[s].double().T @ A[s].double()).float()) for e, s in _rows(counts)]:
        assert torch.equal(got.isnan(), ref.isnan())
        assert torch.equal(got.isinf(), ref.isinf()) and torch.equal(got[got.isinf()], ref[ref.isinf()])
        ok = torch.isfinite(ref)
        assert (got[ok] - ref[ok]).abs().max() <= 1e-4 * ref[ok].abs().max() if ok.any() else True
