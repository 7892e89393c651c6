"""GPU parity of the fp32 grouped GEMMs that split their operands into bf16 parts, at the edges of their tiles and stages: calls
large enough to take that kernel, one-row and empty experts, contractions and columns off the 32 / 64 / 128 grid, and operands
that three bf16 parts cannot hold (infinities, NaN, the top of the range, magnitudes below 2^-110), whose tiles are computed
on the fp32 instruction.  Every element against float64, within the bound of an fp32 dot product summed in any order:
|error| <= (n + 2) 2^-24 sum |a||b|; and, where that bound is too wide to see a part of an operand missing: sums of one and two
terms, sums of one term with a factor of one (exact), and the 2-norm of the error."""
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


def _three(B, ctx, counts, N, K, off, Rcap, A, W, dC):
    """C = A W^T, dA = dC W and dB = dC^T A, with the contractions' lengths."""
    E = len(counts)
    C, dA, dB = (torch.full(s, float("nan"), device="cuda") for s in ((Rcap, N), (Rcap, K), (E, N, K)))
    B.moe_grouped_gemm_fwd(ctx, A, W, off, E, N, K, Rcap, B.F32, B.EPI_NONE, None, None, C, None)
    B.moe_grouped_gemm_dgrad(ctx, dC, W, off, E, N, K, Rcap, B.F32, None, None, None, dA)
    B.moe_grouped_gemm_wgrad(ctx, A, dC, off, E, N, K, Rcap, B.F32, None, None, 0, B.F32, dB)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    return C, dA, dB


@pytest.mark.parametrize("counts,N,K", CASES)
@pytest.mark.parametrize("terms", [1, 2])
def test_split_sums_of_few_terms(B, ctx, counts, N, K, terms):
    """Contractions of which all but one or two terms are zero.  One rounding of the whole, where the leading parts' products meet the
    others, 2^-7 of it, which seven additions per term round to theirs; two terms: the matrix unit adds the leading products, and
    drops up to a last place of their sum (2 x 2^-24) where their exponents differ.  The product left out is 2^-34."""
    off, R, Rcap, A, W, dC = _case(counts, N, K, 21)
    g = torch.Generator("cuda").manual_seed(22)
    ones = lambda rows, n: torch.zeros(rows, n, device="cuda").scatter_(1, torch.rand(rows, n, generator=g, device="cuda").topk(terms, 1)[1], 1.0)
    sA, sC = A * ones(Rcap, K), dC * ones(Rcap, N)
    tA = A.clone()                                                    # (the weight gradient's: terms rows per expert and column)
    for e, s in _rows(counts):
        if counts[e] > terms:
            tA[s] *= ones(K, counts[e]).t()
    bound = (1 + 2 * (terms - 1) + terms * 7 * 2.0 ** -7 + 2.0 ** -9) * EPS
    C, dA, _ = _three(B, ctx, counts, N, K, off, Rcap, sA, W, sC)
    _, _, dB = _three(B, ctx, counts, N, K, off, Rcap, tA, W, dC)
    for e, s in _rows(counts):
        a, w, c, t, d = sA[s].double(), W[e].double(), sC[s].double(), tA[s].double(), dC[s].double()
        _within(C[s], a @ w.T, bound * (a.abs() @ w.abs().T))
        _within(dA[s], c @ w, bound * (c.abs() @ w.abs()))
        _within(dB[e], d.T @ t, bound * (d.abs().T @ t.abs()))


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -106])
@pytest.mark.parametrize("counts,N,K", CASES)
def test_split_holds_every_bit(B, ctx, counts, N, K, scale):
    """One factor of 24 significant bits, the other a single one per sum: the result is that factor, bit for bit, with either operand
    as the former.  (At 2^-106 the third part is a subnormal number.)"""
    off, R, Rcap, *x = _case(counts, N, K, 23)
    g = torch.Generator("cuda").manual_seed(24)
    A, W, dC = (torch.sign(t) * (1.0 + torch.rand(t.shape, generator=g, device="cuda")) * scale for t in x)
    E = len(counts)
    pick = lambda n, m: torch.randint(0, m, (n,), generator=g, device="cuda")
    onehot = lambda at, m: torch.zeros(at.shape[0], m, device="cuda").scatter_(1, at[:, None], 1.0)
    ak, cn = pick(Rcap, K), pick(Rcap, N)
    C, dA, _ = _three(B, ctx, counts, N, K, off, Rcap, onehot(ak, K), W, onehot(cn, N))
    for e, s in _rows(counts):
        assert torch.equal(C[s], W[e][:, ak[s]].t()) and torch.equal(dA[s], W[e][cn[s]])
    wk, wn = pick(N, K), pick(K, N)
    C, _, _ = _three(B, ctx, counts, N, K, off, Rcap, A, onehot(wk, K).repeat(E, 1, 1), dC)
    _, dA, _ = _three(B, ctx, counts, N, K, off, Rcap, A, onehot(wn, N).t().contiguous().repeat(E, 1, 1), dC)
    assert torch.equal(C[:R], A[:R][:, wk]) and torch.equal(dA[:R], dC[:R][:, wn])
    oA, oC = torch.zeros_like(A), torch.zeros_like(dC)
    rk, rn = {}, {}
    for e, s in _rows(counts):
        if counts[e]:
            rk[e], rn[e] = pick(K, counts[e]), pick(N, counts[e])
            oA[s], oC[s] = onehot(rk[e], counts[e]).t(), onehot(rn[e], counts[e]).t()
    _, _, dB = _three(B, ctx, counts, N, K, off, Rcap, oA, W, dC)
    _, _, dB2 = _three(B, ctx, counts, N, K, off, Rcap, A, W, oC)
    for e, s in _rows(counts):
        if counts[e]:
            assert torch.equal(dB[e], dC[s][rk[e]].t()) and torch.equal(dB2[e], A[s][rn[e]])


@pytest.mark.parametrize("counts,N,K", CASES)
def test_split_error_norm(B, ctx, counts, N, K):
    """The 2-norm of the error over that of the result.  Each of the four roundings per 32 elements is off by 0.41 x 2^-24 of the sum so
    far in the root mean square, whose square grows linearly: 0.41 x 2^-24 sqrt(2 stages).  Twice that; one operand's third
    part left out would be ten times it."""
    off, R, Rcap, A, W, dC = _case(counts, N, K, 25)
    C, dA, dB = _three(B, ctx, counts, N, K, off, Rcap, A, W, dC)
    for e, s in _rows(counts):
        if counts[e] < 64:
            continue
        a, w, d = A[s].double(), W[e].double(), dC[s].double()
        for got, ref, n in ((C[s], a @ w.T, K), (dA[s], d @ w, N), (dB[e], d.T @ a, counts[e])):
            err = ((got.double() - ref).norm() / ref.norm()).item()
            assert err <= 2 * 0.41 * EPS * (2 * ((n + 31) // 32)) ** 0.5 + EPS, (e, n, err)


@pytest.mark.parametrize("counts,N,K", CASES)
def test_split_weighted(B, ctx, counts, N, K):
    """Routing weights, and a forward call that keeps no pre-activations."""
    off, R, Rcap, A, W, dC = _case(counts, N, K, 26)
    E = len(counts)
    p, Zs = torch.rand(Rcap, device="cuda"), torch.randn(Rcap, 2 * K, device="cuda")
    Z, act, weighted = (torch.full((Rcap, n), float("nan"), device="cuda") for n in (N, N // 2, N // 2))
    dZ, dA = (torch.full((Rcap, n), float("nan"), device="cuda") for n in (2 * K, K))
    B.moe_grouped_gemm_fwd(ctx, A, W, off, E, N, K, Rcap, B.F32, B.EPI_SWIGLU, None, None, Z, act)
    B.moe_grouped_gemm_fwd_weighted(ctx, A, W, off, E, N, K, Rcap, B.F32, B.EPI_SWIGLU, None, None, p, None, weighted)
    B.moe_grouped_gemm_dgrad(ctx, dC, W, off, E, N, K, Rcap, B.F32, None, None, None, dA)
    B.moe_grouped_gemm_dgrad_weighted(ctx, dC, W, off, E, N, K, Rcap, B.F32, Zs, None, None, p, dZ, None)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    assert torch.equal(weighted[:R], p[:R, None] * act[:R]) and weighted[R:].isnan().all()
    da = dA[:R].double() * p[:R, None].double()                        # (the same sums: only the derivative's roundings differ)
    g, u = Zs[:R, :K].double(), Zs[:R, K:].double()
    s, rel = torch.sigmoid(g), (16 + 4 * g.abs()) * EPS
    _within(dZ[:R, :K], da * u * s * (1 + g * (1 - s)), rel * (da * u * s).abs() * (1 + g.abs()) + 1e-30)
    _within(dZ[:R, K:], da * g * s, rel * (da * g * s).abs() + 1e-30)
    assert dZ[R:].isnan().all()


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
