"""bf16 weight gradients of few tiles, whose contraction is split to fill the chip, and of skewed loads below that: as
test_gpu_wgrad_split.py, with sizes on both sides of the rule (the last of each pair of single experts is not split)."""
import numpy as np
import pytest

from test_gpu_wgrad_split import _case, _run

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# rows per expert, N, K, the expert that has to be split (None: none)
CASES = [
    ([1537], 136, 72, 0), ([640], 136, 72, None),              # one expert: pieces of 8 stages and what is left; too short
    ([16384], 192, 256, 0), ([1400], 3000, 512, None),          # as many pieces as slices; output too large beside the walk
    ([6000, 0, 129, 3000], 264, 136, 0),                        # several experts, some below a piece
    ([25000] + [40] * 24, 704, 256, 0), ([1000] * 25, 704, 256, None),  # one hot expert among many tiles; equal ones
    ([7000] + [40] * 24, 704, 256, None), ([24000] + [24] * 24, 704, 256, None),   # too few rows for it; all that are too few
    ([24000] + [25] * 23 + [2], 704, 256, 0),                               # one row more
]


@pytest.mark.parametrize("gather", [None, "A", "dC"])
@pytest.mark.parametrize("rows,N,K,big", CASES, ids=lambda v: "" if isinstance(v, list) else str(v))
def test_few_tiles(rows, N, K, big, gather):
    from paper_2603_07685_amd import binding as B
    room = B.Context(T=64, k=1, E=len(rows), h=4096, f_max=512)
    none = B.Context(T=64, k=1, E=len(rows), h=0, f_max=0)
    case = _case(rows, N, K, gather)
    E, ref = case[5], case[7]
    # fp32 sums of n products that are exact: a random walk of roundings of 2^-24, four times that
    tol = 4 * np.sqrt(max(rows)) * 2.0 ** -24
    rel = lambda t, r: ((t.double() - r).norm() / r.norm()).item()
    f32 = lambda: torch.full((E, N, K), float("nan"), dtype=torch.float32, device="cuda")
    a = _run(B, room, case, N, K, gather, False, B.F32, f32())
    assert torch.equal(a, _run(B, room, case, N, K, gather, False, B.F32, f32()))
    c = _run(B, none, case, N, K, gather, False, B.F32, f32())
    for e, n in enumerate(rows):
        assert n > 0 or ((a[e] == 0).all() and (c[e] == 0).all())
        if n:
            assert rel(a[e], ref[e]) <= tol and rel(c[e], ref[e]) <= tol
        assert torch.equal(a[e], c[e]) or n * 4 >= max(rows)
    assert big is None or not torch.equal(a[big], c[big])       # (other sums)
    assert big is not None or torch.equal(a, c)
    base = torch.randn((E, N, K), device="cuda").bfloat16()
    h = _run(B, room, case, N, K, gather, True, B.BF16, base.clone())
    assert torch.equal(h, (a + base.float()).bfloat16())
    assert room.poll_error() == 0 and none.poll_error() == 0
