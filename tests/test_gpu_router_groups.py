"""GPU parity of the group-limited router where the groups' best one or two are found in registers: groups of 16, 32 and 48 members, one
and two that count, more tokens than the smaller workgroup's launch takes, ties, infinities; and the sigmoid backward, whose unselected
experts are written without their scores (zeros, and NaN where the logit is)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,E,k,ng,tg", [(7, 16, 1, 1, 1), (33, 64, 4, 4, 4), (130, 96, 2, 2, 1), (4097, 256, 8, 8, 4), (61, 256, 16, 16, 8),
                                         (19, 144, 3, 3, 3)])
@pytest.mark.parametrize("fn", [0, 1])
def test_groups_in_registers(oracle, T, E, k, ng, tg, fn):
    from gpu_util import dev
    from paper_2603_07685_amd import binding as B
    g = np.random.default_rng(T + E + k)
    logits = (np.round(g.normal(size=(T, E)) * 4) / 4).astype(np.float32)
    logits[g.random((T, E)) < 0.02] = -np.inf
    if fn == 1:
        logits[g.random((T, E)) < 0.02] = np.inf
    bias = (np.round(g.normal(size=E) * 4) / 16).astype(np.float32)
    ctx = B.Context(T, k, E, 64, 64)
    for b in (bias, None):
        o_idx, o_prob, o_counts = oracle.route_topk_grouped(logits, k, ng, tg, b, fn, False, 2.5)
        idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
        prob = torch.full((T, k), float("nan"), device="cuda")
        counts = torch.full((E,), -7, dtype=torch.int32, device="cuda")
        B.moe_route_topk_grouped(ctx, dev(logits), None if b is None else dev(b), T, E, k, ng, tg, fn, False, 2.5, idx, prob, counts)
        torch.cuda.synchronize()
        assert np.array_equal(idx.cpu().numpy(), o_idx) and np.array_equal(counts.cpu().numpy(), o_counts)
        np.testing.assert_allclose(prob.cpu().numpy(), o_prob, rtol=2e-6, atol=1e-9)
    ctx.close()


def test_sigmoid_backward_of_nan_logits():
    from paper_2603_07685_amd import binding as B
    T, E, k = 37, 40, 4
    g = torch.Generator("cuda").manual_seed(3)
    logits = torch.randn(T, E, device="cuda", generator=g)
    logits[3, 5] = logits[4, 6] = float("nan")
    idx = torch.stack([torch.randperm(E, device="cuda", generator=g)[:k] for _ in range(T)]).to(torch.int32)
    idx[4] = torch.tensor([1, 6, 2, 3], dtype=torch.int32)            # a selected one
    idx[3] = torch.tensor([1, 2, 3, -1], dtype=torch.int32)           # an unselected one, and a slot that names no expert
    dw = torch.randn(T, k, device="cuda", generator=g)
    out = torch.full((T, E), float("nan"), device="cuda")
    ctx = B.Context(T, k, E, 64, 64)
    B.moe_route_topk_bwd(ctx, logits, idx, dw, T, E, k, 1, False, 1.5, out)
    torch.cuda.synchronize()
    ctx.close()
    s = torch.sigmoid(logits.double())
    ref = torch.zeros(T, E, dtype=torch.float64, device="cuda")
    ok = idx >= 0
    ref.scatter_add_(1, idx.clamp(min=0).long(), torch.where(ok, 1.5 * dw, 0).double())
    ref = ref * s * (1 - s)
    assert torch.equal(out.isnan(), logits.isnan()) and torch.equal(ref.isnan(), logits.isnan())
    ref, got = torch.nan_to_num(ref), torch.nan_to_num(out).double()
    assert (got - ref).abs().max() <= 4e-7 * ref.abs().max()           # (a few ulps of exp and of the products)
