"""GPU parity of the router at the edges of its lane layout: experts around multiples of 16 and 64, slots beyond 16, groups
beyond 16, token counts around a wavefront's and a workgroup's share, the histogram of one and of many workgroups, calls
in a row (the shared histogram is left at zero by each), no histogram, values that order specially."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    from paper_2603_07685_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(T=8192, k=8, E=64, h=64, f_max=64)
    yield c
    c.close()


def _out(T, E, k):
    e = lambda s, v, t: torch.full(s, v, dtype=t, device="cuda")
    return e((T, k), -7, torch.int32), e((T, k), float("nan"), torch.float32), e((E,), -7, torch.int32)


@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (3, 16, 16), (4, 17, 17), (5, 15, 3), (16, 33, 16), (17, 64, 17), (63, 65, 4),
                                   (257, 256, 16), (255, 257, 16), (4096, 129, 6), (4097, 128, 6), (4100, 512, 20)])
@pytest.mark.parametrize("fn,norm", [(0, False), (1, True)])
def test_top_k_and_backward(B, ctx, oracle, T, E, k, fn, norm):
    from gpu_util import dev
    g = np.random.default_rng(T + E + k)
    logits = (np.round(g.normal(size=(T, E)) * 8) / 4).astype(np.float32)     # ties, and zeros of both signs
    logits[g.random((T, E)) < 0.02] = -0.0
    if E > 2 * k:
        logits[::2, E // 2] = -np.inf
    o_idx, o_prob, o_counts = oracle.route_topk(logits, k, fn, norm, 1.5)
    d = dev(logits)
    for _ in range(3):
        idx, prob, counts = _out(T, E, k)
        B.moe_route_topk(ctx, d, T, E, k, fn, norm, 1.5, idx, prob, counts)
        torch.cuda.synchronize()
        assert np.array_equal(idx.cpu().numpy(), o_idx) and np.array_equal(counts.cpu().numpy(), o_counts)
        np.testing.assert_allclose(prob.cpu().numpy(), o_prob, rtol=2e-6, atol=1e-9)
    B.moe_route_topk(ctx, d, T, E, k, fn, norm, 1.5, idx, prob, None)
    assert np.array_equal(idx.cpu().numpy(), o_idx)
    logits = np.where(np.isinf(logits), -3, logits).astype(np.float32)
    o_idx, _, _ = oracle.route_topk(logits, k, fn, norm, 1.5)
    dw = g.normal(size=(T, k)).astype(np.float32)
    out = torch.full((T, E), float("nan"), dtype=torch.float32, device="cuda")
    B.moe_route_topk_bwd(ctx, dev(logits), dev(o_idx), dev(dw), T, E, k, fn, norm, 1.5, out)
    ref = oracle.route_topk_bwd(logits, o_idx, dw, fn, norm, 1.5)
    got = out.cpu().numpy().astype(np.float64)
    # (fp32 terms of size |dw|, which cancel where one weight is normalised by itself)
    assert np.abs(got - ref).max() <= 2e-5 * np.abs(ref).max() + 2e-6 * np.abs(dw).max()


@pytest.mark.parametrize("T,E,k,ng,tg", [(5, 48, 8, 16, 4), (33, 51, 4, 17, 2), (70, 128, 16, 8, 8), (9, 320, 8, 8, 4),
                                         (130, 64, 32, 64, 32), (66, 96, 6, 3, 2), (20, 256, 17, 1, 1), (1030, 256, 8, 8, 4)])
@pytest.mark.parametrize("fn", [0, 1])
def test_group_limited_top_k(B, ctx, oracle, T, E, k, ng, tg, fn):
    from gpu_util import dev
    g = np.random.default_rng(T + E + k)
    logits = (np.round(g.normal(size=(T, E)) * 4) / 4).astype(np.float32)
    bias = (np.round(g.normal(size=E) * 4) / 16).astype(np.float32)
    for b in (bias, None):
        o_idx, o_prob, o_counts = oracle.route_topk_grouped(logits, k, ng, tg, b, fn, True, 2.5)
        for _ in range(2):
            idx, prob, counts = _out(T, E, k)
            B.moe_route_topk_grouped(ctx, dev(logits), None if b is None else dev(b), T, E, k, ng, tg, fn, True, 2.5, idx, prob, counts)
            torch.cuda.synchronize()
            assert np.array_equal(idx.cpu().numpy(), o_idx) and np.array_equal(counts.cpu().numpy(), o_counts)
            np.testing.assert_allclose(prob.cpu().numpy(), o_prob, rtol=2e-6, atol=1e-9)


@pytest.mark.parametrize("T,E", [(31, 16), (32, 17), (33, 256), (65, 257), (2100, 1000)])
@pytest.mark.parametrize("fn", [0, 1])
def test_aux_loss(B, ctx, oracle, T, E, fn):
    from gpu_util import dev
    g = np.random.default_rng(T + E)
    logits = g.normal(size=(T, E)).astype(np.float32)
    counts = g.multinomial(2 * T, np.ones(E) / E).astype(np.int32)
    ref_loss, ref_grad = oracle.aux_loss(logits, counts, 2, fn, 0.01)
    base = (1e-4 * g.normal(size=(T, E))).astype(np.float32)
    seen = []
    for acc in (0, 1, 1):
        dl, loss = dev(base), torch.full((1,), float("nan"), dtype=torch.float32, device="cuda")
        B.moe_aux_loss(ctx, dev(logits), dev(counts), T, E, 2, fn, 0.01, 0.7, acc, loss, dl)
        torch.cuda.synchronize()
        want = 0.7 * ref_grad + (base if acc else 0)
        assert np.abs(dl.cpu().numpy() - want).max() <= 2e-5 * np.abs(want).max()
        assert abs(loss.item() - ref_loss) <= 2e-6 * abs(ref_loss)
        seen.append(loss.item())
    assert len(set(seen)) == 1


@pytest.mark.parametrize("T,E", [(37, 17), (70, 33), (301, 64), (130, 129), (515, 256)])
@pytest.mark.parametrize("fn", [0, 1])
def test_the_lane_layout_does_not_show_in_the_bits(B, ctx, T, E, fn):
    """16 lanes per token (16 slots) and a whole wavefront (17 slots, the last with a gradient of zero) add in the same order:
    weights, gradients, and the loss with 64 experts of no probability appended beyond 256 are the same bits."""
    from gpu_util import dev
    g = np.random.default_rng(T * E)
    logits = g.normal(size=(T, E)).astype(np.float32)
    d = dev(logits)
    dw = np.zeros((T, 17), np.float32)
    dw[:, :16] = g.normal(size=(T, 16))
    bits = lambda t: t.cpu().numpy().view(np.int32)
    seen = {}
    for k in (16, 17):
        idx, prob, counts = _out(T, E, k)
        out = torch.empty((T, E), dtype=torch.float32, device="cuda")
        B.moe_route_topk(ctx, d, T, E, k, fn, False, 1.5, idx, prob, counts)
        B.moe_route_topk_bwd(ctx, d, idx, dev(dw[:, :k]), T, E, k, fn, False, 1.5, out)
        gidx, gprob, gcounts = _out(T, E, k)
        B.moe_route_topk_grouped(ctx, d, None, T, E, k, 1, 1, fn, False, 1.5, gidx, gprob, gcounts)
        seen[k] = [bits(prob)[:, :16], bits(out), bits(gprob)[:, :16]]
    for a, b in zip(seen[16], seen[17]):
        assert np.array_equal(a, b)
    wide = np.full((T, 320), -np.inf, np.float32)
    wide[:, :E] = logits
    counts = np.zeros(320, np.int32)
    counts[:E] = g.multinomial(2 * T, np.ones(E) / E)
    res = []
    for e in (E, 320):
        dl, loss = torch.empty((T, e), dtype=torch.float32, device="cuda"), torch.empty(1, dtype=torch.float32, device="cuda")
        B.moe_aux_loss(ctx, dev(wide[:, :e]), dev(counts[:e]), T, e, 2, fn, (E if e == 320 else 320) / 256, 0.7, 0, loss, dl)
        res.append((bits(loss), bits(dl)[:, :E]))
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])


def test_calls_that_overlap_leave_nothing_behind(B, oracle):
    """The router keeps nothing in the context: calls of several token counts on two streams at once each count right, and so
    does a later call."""
    from gpu_util import dev
    ctx = B.Context(T=8192, k=8, E=64, h=64, f_max=64)
    E, k, cases = 96, 4, []
    for i, T in enumerate((8192, 6000, 8000, 4097)):
        logits = np.random.default_rng(i).normal(size=(T, E)).astype(np.float32)
        cases.append((T, dev(logits), oracle.route_topk(logits, k, 0, False, 1.0)[2], _out(T, E, k)))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for _ in range(5):
        torch.cuda.synchronize()
        torch.cuda._sleep(2_000_000)   # (both streams start on what has been queued by then together)
        queued = torch.cuda.Event()
        queued.record()
        for s in streams:
            s.wait_event(queued)
        for i, (T, d, _, out) in enumerate(cases):
            with torch.cuda.stream(streams[i & 1]):
                B.moe_route_topk(ctx, d, T, E, k, 0, False, 1.0, *out)
        torch.cuda.synchronize()
        for T, d, want, out in cases:
            assert np.array_equal(out[2].cpu().numpy(), want)
    T, d, want, out = cases[3]
    B.moe_route_topk(ctx, d, T, E, k, 0, False, 1.0, *out)
    assert np.array_equal(out[2].cpu().numpy(), want)
    ctx.close()
