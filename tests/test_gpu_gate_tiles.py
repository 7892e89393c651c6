"""GPU parity of the gate GEMM on each of its tiles (16 x 16 to 64 x 128 with the contraction split among a workgroup's waves) and on
the 256 x 256 kernel with a split contraction: ragged rows and columns, fewer chunks of the contraction than waves, chunk
counts that no number of waves divides.  Every element against float64, within the error bound of an fp32 sum in any order
(the products of bf16 values are exact); two runs give the same bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# T, E, h by the number of the tile that takes them (-1: the 256 x 256 kernel, in pieces)
SIZES = {0: [(17, 8, 64), (33, 24, 192), (300, 200, 4160)],                  # 16 x 16
         1: [(499, 248, 7168), (1000, 128, 2112)],                           # 32 x 16
         2: [(4000, 40, 2048), (3971, 40, 1984)],                            # 32 x 32
         3: [(16384, 32, 512), (16001, 24, 576)],                            # 64 x 32
         4: [(8000, 104, 512), (7999, 104, 448), (15991, 64, 4096)],         # 64 x 64
         5: [(16383, 128, 448), (16001, 248, 1088)],                         # 64 x 128
         -1: [(2048, 256, 7168), (4100, 248, 6720), (16384, 128, 7168), (8192, 64, 7168), (12283, 120, 4096)]}


@pytest.mark.parametrize("T,E,h", sum(SIZES.values(), []))
def test_gate_gemm_tiles(T, E, h):
    from paper_2603_07685_amd import binding as B
    ctx = B.Context(T, 1, E, h, max(E, 8))
    g = torch.Generator(device="cuda")
    g.manual_seed(T + E + h)
    X = torch.randn(T, h, generator=g, device="cuda").to(torch.bfloat16)
    W = (0.02 * torch.randn(E, h, generator=g, device="cuda")).to(torch.bfloat16)
    out = torch.full((T + 1, E), float("nan"), device="cuda")
    again = out.clone()
    B.moe_gate_gemm(ctx, X, W, T, E, h, out)
    B.moe_gate_gemm(ctx, X, W, T, E, h, again)
    torch.cuda.synchronize()
    assert ctx.poll_error() == 0
    x, w = X.double(), W.double()
    over = (out[:T].double() - x @ w.T).abs() - (h + 8) * 2.0 ** -24 * (x.abs() @ w.abs().T)
    assert float(over.max()) <= 0
    assert torch.equal(out[:T], again[:T]) and out[T].isnan().all()
    ctx.close()
