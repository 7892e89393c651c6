"""What bench.py books to a batch's end is what the batch has kept, as the library says, and not what looks short."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# every GEMM of the first is kept; of the second, beyond the small tiles, the routed ones are launched at once
@pytest.mark.parametrize("T,h,f,E,k,sf,every", [(96, 128, 64, 4, 2, 64, True), (700, 2048, 1536, 5, 4, 192, False)])
def test_kept_calls(T, h, f, E, k, sf, every):
    import bench
    from paper_2603_07685_amd import layer as L
    from paper_2603_07685_amd import workloads as wl
    st = L.LayerState(wl.MoEConfig("kept", T=T, h=h, f=f, E=E, k=k, E_router=E, score=wl.SOFTMAX, norm_topk=False, load="router",
                                   shared_f=sf, seed=5))
    st.step()
    at = st.batch.kept()
    kept = bench.kept_calls(st)
    recs, _ = bench.timed_step_with_events(st, torch)
    assert len(kept) == len(recs) and 2 * sum(kept) == st.batch.kept()[0] - at[0]     # (two steps since)
    gemms = [is_kept for is_kept, (_, fl, _) in zip(kept, recs) if fl]
    assert len(gemms) == 12 and all(gemms) == every and any(gemms)
    assert not any(is_kept for is_kept, (_, fl, _) in zip(kept, recs) if not fl)   # (bf16: nothing else can be)
    assert st.ctx.poll_error() == 0
