"""GPU parity of the gate GEMM at the edges of its split contraction: one and several pieces, a last piece that is shorter,
ragged row tiles, more than one column tile, a workspace with no room for partial results.  Every element against float64,
within the error bound of an fp32 sum in any order (the products of bf16 values are exact)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    from paper_2603_07685_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("T,E,h", [(1, 8, 64), (255, 16, 960), (256, 256, 1024), (257, 264, 1088), (700, 8, 4160),
                                   (3000, 40, 2624), (20000, 512, 1152), (66000, 256, 1024),
                                   (300, 64, 5184), (300, 64, 5760), (520, 72, 6720)])   # (as many pieces as have stages)
@pytest.mark.parametrize("room", [True, False])
def test_gate_gemm(B, T, E, h, room):
    ctx = B.Context(T, 1, E, h, max(E, 8)) if room else B.Context(1, 1, 1, 0, 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(T + E + h)
    X = torch.randn(T, h, generator=g, device="cuda").to(torch.bfloat16)
    W = (0.02 * torch.randn(E, h, generator=g, device="cuda")).to(torch.bfloat16)
    out = torch.full((T, E), float("nan"), device="cuda")
    again = out.clone()
    B.moe_gate_gemm(ctx, X, W, T, E, h, out)
    B.moe_gate_gemm(ctx, X, W, T, E, h, again)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    x, w = X.double(), W.double()
    over = (out.double() - x @ w.T).abs() - (h + 8) * 2.0 ** -24 * (x.abs() @ w.abs().T)
    assert float(over.max()) <= 0
    assert torch.equal(out, again)
    ctx.close()
