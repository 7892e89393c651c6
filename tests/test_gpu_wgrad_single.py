"""GPU parity of the bf16 weight gradient on one stage buffer (many tiles, few rows per expert): experts of no, one, a whole stage's,
one more and many rows (past the 16 stages whose row map is looked up at a time), columns off the tile grid, the row map on either operand,
accumulation; and offsets that fall or leave the tensor, which write nothing.  Every element against float64, within one
rounding of the result plus the error bound of an fp32 sum in any order."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from test_gpu_gemm_variants import DT, STORE, WGRAD, _lib
from test_gpu_tile_dispatch import BF, F32, Group, _nan, _within

# (more than 512 tiles of 128 x 128, at most 160 rows in all per 256 of them)
CASES = [([0, 1, 63, 64, 65, 130, 0, 7] + [20] * 16, 904, 712), ([2100, 3, 0, 1] + [32] * 36, 1536, 1408), ([5] * 33, 512, 520)]


@pytest.fixture(scope="module")
def B():
    from paper_2603_07685_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(T=2048, k=4, E=64, h=1024, f_max=1024)
    yield c
    c.close()


@pytest.mark.parametrize("counts,N,K", CASES)
@pytest.mark.parametrize("which", [None, 0, 1])
@pytest.mark.parametrize("f32", [False, True])
def test_weight_gradient_one_buffer(B, ctx, counts, N, K, which, f32):
    q = Group(counts, N, K, 5)
    dt, odt = (F32, B.F32) if f32 else (BF, B.BF16)
    dW = _nan(q.E, N, K, dt=dt)
    ulp = 2.0 ** -24 if f32 else 2.0 ** -8
    for acc in (0, 1):
        old = dW.double() if acc else None
        if which is None:
            B.moe_grouped_gemm_wgrad(ctx, q.A, q.dC, q.off, q.E, N, K, q.Rcap, B.BF16, None, None, acc, odt, dW)
        else:
            A, dC = (q.X, q.dC) if which == B.GATHER_A else (q.A, q.G)
            B.moe_grouped_gemm_wgrad_gather(ctx, A, dC, which, q.T, q.src, q.k, q.off, q.E, N, K, q.Rcap, acc, odt, dW)
        torch.cuda.synchronize()
        assert ctx.poll_error() == 0
        for e, s in q.each():
            a, d = q.A[s].double(), q.dC[s].double()
            ref, mag = d.T @ a, d.abs().T @ a.abs()
            if acc:
                ref, mag = ref + old[e], mag + 2 * old[e].abs()
            _within(dW[e], ref, mag, counts[e], "dW", ulp)


def test_a_hot_experts_walk_is_bounded():
    """One expert may hold all rows: they are few beside the tiles of the call.  (Whatever the load, no call was slower there than on two
    buffers; from 192 rows per 256 tiles on, some with nearly all rows on one expert were.)"""
    f = _lib()
    for E in (4, 16, 24, 64):
        for N in (256, 512, 704, 1024, 2048):
            for K in (384, 512, 1024):
                for R in (64, 256, 512, 1024, 2048, 4096, 6144):
                    if f(256, WGRAD, STORE, DT["bf16"], 0, E, N, K, R) == 4:
                        assert R * 256 <= 160 * E * (-(-N // 128)) * (-(-K // 128)), (E, N, K, R)


@pytest.mark.parametrize("bad", ["falls", "behind the rows", "before them"])
def test_wrong_offsets_write_nothing(B, ctx, bad):
    counts, N, K = CASES[0]
    q = Group(counts, N, K, 6)
    if bad == "falls":
        q.off[3] = q.R
    elif bad == "behind the rows":
        q.off[-1] = q.Rcap + 1
    else:
        q.off[0] = -1
    dW = _nan(q.E, N, K)
    B.moe_grouped_gemm_wgrad(ctx, q.A, q.dC, q.off, q.E, N, K, q.Rcap, B.BF16, None, None, 0, B.BF16, dW)
    torch.cuda.synchronize()
    assert ctx.poll_error() != 0 and dW.isnan().all()
