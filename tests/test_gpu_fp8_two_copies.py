"""Blockwise layer: with few rows both copies of the activation and of dZ come from one quantiser launch, with many the row-wise one from the
GEMM call.  Either side of the line, and with the routed and the shared expert on different sides, every copy and result has the same bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("eq2", [False, True])
@pytest.mark.parametrize("line", ["default", "shared_only", "at", "below"])
def test_one_launch_for_both_copies_is_bit_identical(line, eq2):
    from paper_2603_07685_amd import layer as L
    from paper_2603_07685_amd import workloads as wl
    cfg = wl.CONFIGS["C5S"]
    hin = L.host_inputs(cfg)
    a = L.LayerState(cfg, hin, eq2=eq2, epilogue_quant=True)
    b = L.LayerState(cfg, hin, eq2=eq2)
    assert a.epilogue_rows == 0 and a.fp8_wgrad and cfg.T < b.Rcap <= b.epilogue_rows
    b.epilogue_rows = {"default": b.epilogue_rows, "shared_only": cfg.T, "at": b.Rcap, "below": b.Rcap - 1}[line]
    for st in (a, b):
        for n in ("qA", "sA", "qdZ", "sdZ", "qAc", "sAc", "qdZc", "sdZc"):
            getattr(st, n).zero_()
        st.step()
    torch.cuda.synchronize()
    assert a.ctx.poll_error() == 0 and b.ctx.poll_error() == 0
    for n in ("qA", "sA", "qdZ", "sdZ", "qAc", "sAc", "qdZc", "sdZc", "qAs", "sAs", "qdZs", "sdZs", "qAsc", "sAsc", "qdZsc", "sdZsc",
              "Y", "dX", "dW1", "dW2", "dprob", "dWs1", "dWs2"):
        assert torch.equal(getattr(a, n), getattr(b, n)), n
