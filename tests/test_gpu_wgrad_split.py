"""bf16 weight gradients whose contraction is split: every kernel that splits (256 x 256 tiles; 128 x 128 tiles from 24576 rows
on), output sizes off the tile grid, both output types, accumulation, gathered operands; against 64-bit sums, against the call
without room for partial results, and against itself."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# rows per expert, N, K.  256 x 256 tiles: two experts above twice the mean and a third of a workgroup's share, N and K ragged;
# 128 x 128 tiles: three experts above a fifth of the rows, an empty one, N and K ragged
LARGE = ([3001, 1900, 900, 0, 40, 20, 10, 17], 2952, 2888)
SMALL = ([9001, 17, 11000, 0, 6500, 1, 100, 300], 264, 136)


@pytest.fixture(scope="module")
def B():
    from paper_2603_07685_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def room(B):
    c = B.Context(T=64, k=1, E=8, h=2888, f_max=1476)
    yield c
    c.close()


@pytest.fixture(scope="module")
def no_room(B):
    c = B.Context(T=64, k=1, E=8, h=0, f_max=0)
    yield c
    c.close()


def _case(rows, N, K, gather, seed=3):
    R, E, k = sum(rows), len(rows), 3
    g = torch.Generator("cuda").manual_seed(seed)
    T = R if not gather else (R + k - 1) // k + 5
    x = {n: torch.randn((T if gather == n else R, w), device="cuda", generator=g).bfloat16() for n, w in (("A", K), ("dC", N))}
    src = torch.randperm(T * k, device="cuda", generator=g)[:R].to(torch.int32)
    src[torch.randperm(R, device="cuda", generator=g)[:R // 50]] = -1
    o = torch.tensor([0] + list(np.cumsum(rows)), dtype=torch.int32, device="cuda")
    full = dict(x)
    if gather:
        full[gather] = torch.where((src >= 0)[:, None], x[gather][(src.clamp(min=0) // k).long()], 0)
    ref = torch.stack([full["dC"][a:b].double().t() @ full["A"][a:b].double() for a, b in zip(o[:-1].tolist(), o[1:].tolist())])
    return x, src, T, k, o, E, R, ref


def _run(B, ctx, case, N, K, gather, acc, dt, out):
    x, src, T, k, o, E, R, _ = case
    if gather:
        B.moe_grouped_gemm_wgrad_gather(ctx, x["A"], x["dC"], B.GATHER_A if gather == "A" else B.GATHER_DC, T, src, k, o, E, N, K, R,
                                        acc, dt, out)
    else:
        B.moe_grouped_gemm_wgrad(ctx, x["A"], x["dC"], o, E, N, K, R, B.BF16, None, None, acc, dt, out)
    return out


@pytest.mark.parametrize("gather", [None, "A", "dC"])
@pytest.mark.parametrize("rows,N,K", [LARGE, SMALL], ids=["tiles256", "tiles128"])
def test_split_contraction(B, room, no_room, rows, N, K, gather):
    case = _case(rows, N, K, gather)
    E, ref = case[5], case[7]
    # fp32 sums of n products that are exact: a random walk of roundings of 2^-24, four times that
    tol = 4 * np.sqrt(max(rows)) * 2.0 ** -24
    rel = lambda t, r: ((t.double() - r).norm() / r.norm()).item()
    f32 = lambda fill=float("nan"): torch.full((E, N, K), fill, dtype=torch.float32, device="cuda")
    a = _run(B, room, case, N, K, gather, False, B.F32, f32())
    b = _run(B, room, case, N, K, gather, False, B.F32, f32())
    c = _run(B, no_room, case, N, K, gather, False, B.F32, f32())
    assert torch.equal(a, b)                      # the same bits whatever the timing
    for e, n in enumerate(rows):
        assert torch.isfinite(a[e]).all() and (n > 0 or (a[e] == 0).all())
        if n:
            assert rel(a[e], ref[e]) <= tol and rel(c[e], ref[e]) <= tol
    big = int(np.argmax(rows))
    assert not torch.equal(a[big], c[big])        # (other sums: it was split, and is not without room)
    assert torch.equal(a[rows.index(17)], c[rows.index(17)])
    base = torch.randn((E, N, K), device="cuda")
    acc = _run(B, room, case, N, K, gather, True, B.F32, base.clone())
    assert rel(acc, ref + base.double()) <= tol
    h = _run(B, room, case, N, K, gather, False, B.BF16, torch.full((E, N, K), float("nan"), dtype=torch.bfloat16, device="cuda"))
    assert torch.equal(h, a.bfloat16())           # one rounding of the same sums
    hb = base.bfloat16()
    h = _run(B, room, case, N, K, gather, True, B.BF16, hb.clone())
    assert torch.equal(h, (a + hb.float()).bfloat16())
    assert room.poll_error() == 0 and no_room.poll_error() == 0


@pytest.mark.parametrize("rows,N,K", [LARGE, SMALL], ids=["tiles256", "tiles128"])
def test_refused_offsets_write_nothing(B, room, rows, N, K):
    x, src, T, k, o, E, R, _ = _case(rows, N, K, None)
    for bad in (o + 1, o.flip(0)):
        out = torch.full((E, N, K), -7.0, dtype=torch.float32, device="cuda")
        B.moe_grouped_gemm_wgrad(room, x["A"], x["dC"], bad.contiguous(), E, N, K, R, B.BF16, None, None, False, B.F32, out)
        assert room.poll_error() == 1 and (out == -7).all()
