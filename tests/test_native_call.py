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
