"""GPU parity of the all-fp32 grouped GEMMs at the edges of their tiles: one-row and empty experts, contractions that end
inside a stage, rows and columns off the 64 / 128 grid, row lengths that allow 16-byte accesses and that do not, and sizes
on either side of the choice between the two tile sizes.  Every element against float64, within the error bound of an
fp32 dot product summed in any order: |error| <= (n + 2) 2^-24 sum |a||b|."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = 2.0 ** -24


@pytest.fixture(scope="module")
def B():
    from paper_2603_07685_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(T=1024, k=2, E=16, h=512, f_max=256)
    yield c
    c.close()


CASES = [
    # counts per expert, N, K
    ([1], 2, 1),
    ([0, 1, 63, 64, 65, 129, 0], 132, 20),
    ([5, 0, 130], 70, 33),                 # row lengths that are no multiple of 16 bytes
    ([64, 128], 64, 16),
    ([4500, 1, 0, 3700], 4096, 20),        # eight 128 x 128 tiles per compute unit: the larger tile (forward)
    ([4500, 1, 0, 3700], 4094, 19),
    ([700, 1], 8192, 2048),                # ... (weight gradient)
]


def _case(counts, N, K, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    R = int(sum(counts))
    Rcap = R + 3
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return off, R, Rcap, r(Rcap, K), r(len(counts), N, K), r(Rcap, N)


def _rows(counts):
    lo = 0
    for e, c in enumerate(counts):
        yield e, slice(lo, lo + c)
        lo += c


def _within(got, ref, bound):
    assert torch.isfinite(got).all()
    over = ((got.double() - ref).abs() - bound).max() if got.numel() else torch.zeros(())
    assert float(over) <= 0, f"error above the summation bound by {float(over):.3e}"


@pytest.mark.parametrize("counts,N,K", CASES)
def test_f32_forward_and_data_gradient(B, ctx, counts, N, K):
    off, R, Rcap, A, W, dC = _case(counts, N, K, 7)
    E, nan = len(counts), float("nan")
    C = torch.full((Rcap, N), nan, device="cuda")
    dA = torch.full((Rcap, K), nan, device="cuda")
    B.moe_grouped_gemm_fwd(ctx, A, W, off, E, N, K, Rcap, B.F32, B.EPI_NONE, None, None, C, None)
    B.moe_grouped_gemm_dgrad(ctx, dC, W, off, E, N, K, Rcap, B.F32, None, None, None, dA)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    for e, s in _rows(counts):
        a, w, d = A[s].double(), W[e].double(), dC[s].double()
        _within(C[s], a @ w.T, (K + 2) * EPS * (a.abs() @ w.abs().T))
        _within(dA[s], d @ w, (N + 2) * EPS * (d.abs() @ w.abs()))
    assert C[R:].isnan().all() and dA[R:].isnan().all()


@pytest.mark.parametrize("counts,N,K", CASES)
def test_f32_swiglu_and_its_backward(B, ctx, counts, N, K):
    off, R, Rcap, A, W, _ = _case(counts, N, K, 8)
    E, f, nan = len(counts), N // 2, float("nan")
    p = torch.rand(Rcap, device="cuda")
    Z = torch.full((Rcap, N), nan, device="cuda")
    act = torch.full((Rcap, f), nan, device="cuda")
    B.moe_grouped_gemm_fwd_weighted(ctx, A, W, off, E, N, K, Rcap, B.F32, B.EPI_SWIGLU, None, None, p, Z, act)
    # the data gradient of a [E, K, f] weight, whose output carries the derivative at Z
    W2 = torch.randn(E, K, f, device="cuda")
    dZ = torch.full((Rcap, N), nan, device="cuda")
    B.moe_grouped_gemm_dgrad_weighted(ctx, A, W2, off, E, K, f, Rcap, B.F32, Z, None, None, p, dZ, None)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    for e, s in _rows(counts):
        a, w = A[s].double(), W[e].double()
        bz = (K + 2) * EPS * (a.abs() @ w.abs().T)
        _within(Z[s], a @ w.T, bz)
        g, u = Z[s, :f].double(), Z[s, f:].double()        # the stored values: rounding of the activation alone
        sg, q = torch.sigmoid(g), p[s, None].double()
        # (the sigmoid's relative error: a few ulps of exp, grown by |g| through its argument)
        rel = (16 + 4 * g.abs()) * EPS
        ref = q * g * sg * u
        _within(act[s], ref, rel * ref.abs() + 1e-30)
        da = a @ W2[e].double()
        bd = (K + 2) * EPS * (a.abs() @ W2[e].double().abs())
        k0, k1 = u * sg * (1 + g * (1 - sg)), g * sg
        cancel = u.abs() * sg * (1 + g.abs())              # the terms of k0 before they cancel
        _within(dZ[s, :f], q * da * k0, q * (bd * cancel + rel * da.abs() * cancel) + 1e-30)
        _within(dZ[s, f:], q * da * k1, q * (bd * k1.abs() + rel * (da * k1).abs()) + 1e-30)
    for t in (Z, act, dZ):
        assert t[R:].isnan().all()


@pytest.mark.parametrize("counts,N,K", CASES)
@pytest.mark.parametrize("accumulate", [0, 1])
def test_f32_weight_gradient(B, ctx, counts, N, K, accumulate):
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


def test_f32_inconsistent_offsets_write_nothing(B, ctx):
    off, R, Rcap, A, W, dC = _case([40, 20], 64, 32, 10)
    off[1] = 70                                             # the second expert would end before it starts
    C = torch.full((Rcap, 64), float("nan"), device="cuda")
    B.moe_grouped_gemm_fwd(ctx, A, W, off, 2, 64, 32, Rcap, B.F32, B.EPI_NONE, None, None, C, None)
    torch.cuda.synchronize()
    assert ctx.poll_error() != 0 and C.isnan().all()
