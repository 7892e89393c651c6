"""The native argument conversion of the binding: what it refuses and what it passes on."""
import pytest

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    import os
    from paper_2603_07685_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2603_07685_amd import build
        build.build_library()
    binding.lib()
    return binding


class _Ctx:                                                  # stands for a context where the call must not get that far
    _addr = None


def test_host_tensors_and_wrong_types_are_refused(B):
    t = torch.zeros(8, 64)
    with pytest.raises(AssertionError):
        B.moe_gate_gemm(_Ctx, t, None, 1, 8, 64, None)
    with pytest.raises(AssertionError):
        B.moe_gate_gemm(_Ctx, None, None, 1, 8, 64, torch.nn.Parameter(t))
    for bad in (1.0, "1", None):
        with pytest.raises(TypeError):
            B.moe_gate_gemm(_Ctx, None, None, bad, 8, 64, None)
    with pytest.raises(TypeError):
        B._native.moe_gate_gemm(None, None, None, 1, 8, 64)
    with pytest.raises(AttributeError):
        B.moe_gate_gemm(_Ctx, [1, 2], None, 1, 8, 64, None)


def test_the_c_library_suffices():
    """Without the native module (built against one torch) the library loads all the same, with a warning, and a call's
    arguments meet the same refusals."""
    import subprocess
    import sys
    code = """
import sys, warnings
sys.modules['paper_2603_07685_amd._pycall'] = None      # (an import of it fails)
import pytest, torch
from paper_2603_07685_amd import binding as B
with pytest.warns(RuntimeWarning, match='ctypes'):
    L = B.lib()
assert L.moe_workspace_bytes(256, 2, 8, 128, 256) > 0
B._stream = lambda: 0
class Ctx:
    _addr = None
    def check(st, what):
        raise B.MoeError(what, st)
t = torch.zeros(8, 64)
with pytest.raises(AssertionError):
    B.moe_gate_gemm(Ctx, t, None, 1, 8, 64, None)
with pytest.raises(TypeError):
    B.moe_gate_gemm(Ctx, None, None, 1.0, 8, 64, None)
with pytest.raises(TypeError):
    B._native.moe_gate_gemm(None, None, None, 1, 8, 64)
for name in B.EXPORTS:
    if hasattr(B, name) and name not in ('moe_workspace_bytes', 'moe_permute_static'):
        assert callable(getattr(B._native, name)), name
with pytest.raises(B.MoeError):
    B.moe_gate_gemm(Ctx, None, None, 1, 8, 64, None)
"""
    subprocess.run([sys.executable, "-c", code], check=True, timeout=300)


class _Sub(torch.Tensor):
    pass


@pytest.mark.gpu
def test_pointers_stream_and_status(B):
    T, E, h = 64, 8, 64
    ctx = B.Context(T, 1, E, h, h)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    X = torch.randint(-4, 5, (T, h), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randint(-4, 5, (E, h), generator=g, device="cuda").to(torch.bfloat16)
    ref = X.float() @ W.float().T                            # small integers: exact
    for wrap in (lambda t: t, torch.nn.Parameter, lambda t: t.as_subclass(_Sub)):
        out = torch.zeros(T, E, device="cuda")
        B.moe_gate_gemm(ctx, wrap(X), wrap(W), T, E, h, out)
        assert torch.equal(out, ref)
    for bad in (X[:, ::2], X.T):
        with pytest.raises(AssertionError):
            B.moe_gate_gemm(ctx, bad, W, T, E, h, out)
    with pytest.raises(B.MoeError, match="moe_gate_gemm"):
        B.moe_gate_gemm(ctx, X, W, T, 7, h, out)
    # the current stream: the launch is captured where the stream is
    out = torch.zeros(T, E, device="cuda")
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        B.moe_gate_gemm(ctx, X, W, T, E, h, out)
    torch.cuda.synchronize()
    assert not out.any()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    ctx.close()
    with pytest.raises(B.MoeError):
        B.moe_gate_gemm(ctx, X, W, T, E, h, out)


@pytest.mark.gpu
def test_through_ctypes(B, monkeypatch):
    """A layer's step with ctypes conversions gives the bits of the native module's."""
    from paper_2603_07685_amd import layer, workloads as wl
    cfg = wl.CONFIGS["C1"]
    hin = layer.host_inputs(cfg, shared_f=64)
    seen = []
    for native in (B._native, B._Ctypes(B.lib())):
        monkeypatch.setattr(B, "_native", native)
        st = layer.LayerState(cfg, hin, shared_f=64)
        st.step()
        torch.cuda.synchronize()
        assert st.ctx.poll_error() == 0
        seen.append([t.clone() for t in (st.Y, st.dX, st.dW1, st.dW2, st.dprob)])
    for a, b in zip(*seen):
        assert torch.equal(a, b)
