"""Blockwise layer with one-byte weight gradients: both copies of the activation and of dZ come from one quantiser launch, at every size,
unless the caller asks for the row-wise ones from the GEMM calls.  Every copy and result has the same bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("eq2", [False, True])
def test_one_launch_for_both_copies_is_bit_identical(eq2):
    from paper_2603_07685_amd import layer as L
    from paper_2603_07685_amd import workloads as wl
    cfg = wl.CONFIGS["C5S"]
    hin = L.host_inputs(cfg)
    a = L.LayerState(cfg, hin, eq2=eq2, epilogue_quant=True)
    b = L.LayerState(cfg, hin, eq2=eq2)
    assert a.epilogue_quant and a.fp8_wgrad and not b.epilogue_quant
    for st in (a, b):
        for n in ("qA", "sA", "qdZ", "sdZ", "qAc", "sAc", "qdZc", "sdZc"):
            getattr(st, n).zero_()
        st.step()
    torch.cuda.synchronize()
    assert a.ctx.poll_error() == 0 and b.ctx.poll_error() == 0
    for n in ("qA", "sA", "qdZ", "sdZ", "qAc", "sAc", "qdZc", "sdZc", "qAs", "sAs", "qdZs", "sdZs", "qAsc", "sAsc", "qdZsc", "sdZsc",
              "Y", "dX", "dW1", "dW2", "dprob", "dWs1", "dWs2"):
        assert torch.equal(getattr(a, n), getattr(b, n)), n


@pytest.mark.parametrize("T,E", [(256, 8), (16384, 32), (16384, 33), (32768, 8)])
def test_the_choice_does_not_hang_on_the_capacity(monkeypatch, T, E):
    from paper_2603_07685_amd import binding as B
    from paper_2603_07685_amd import layer as L
    from paper_2603_07685_amd import workloads as wl
    asked = []
    for name, last in (("moe_grouped_gemm_fwd_quant", 2), ("moe_grouped_gemm_dgrad_quant", 2)):
        f = getattr(B, name)
        monkeypatch.setattr(B, name, lambda *a, f=f, n=last: (asked.append([x is not None for x in a[-n:]]), f(*a)))
    cfg = wl.MoEConfig("two_copies", T=T, h=128, f=128, E=E, k=8, E_router=E, score=wl.SOFTMAX, norm_topk=False, load="router",
                       shared_f=128, fp8=True, align=128, seed=3)
    for epilogue in (None, True):
        st = L.LayerState(cfg, epilogue_quant=epilogue)
        st.step()
        torch.cuda.synchronize()
        assert st.ctx.poll_error() == 0
        assert asked == [[bool(epilogue)] * 2] * 4, (epilogue, asked)   # (routed and shared expert, forward and backward)
        asked.clear()
