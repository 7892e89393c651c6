"""GPU parity of the row-ID map at the edges of its kernels: pair counts around a wavefront, a chunk and the size up to which
one workgroup does it all; expert counts around the same; skipped slots; padded experts; more rows than pairs; and the
combine's backward, whose launch also zeroes the rows no pair owns.  Everything bit for bit against a stable sort."""
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
    c = B.Context(T=40000, k=1, E=1024, h=64, f_max=64)
    yield c
    c.close()


def _maps(idx, E, align, Rcap):
    flat = idx.reshape(-1)
    ok = (flat >= 0) & (flat < E)
    counts = np.bincount(flat[ok], minlength=E).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum((counts + align - 1) // align * align)]).astype(np.int32)
    order = np.argsort(np.where(ok, flat, E), kind="stable")[: ok.sum()]
    first = np.concatenate([[0], np.cumsum(counts)])[:-1]
    rows = offsets[flat[order]] + np.arange(len(order)) - first[flat[order]]
    row_of = np.full(flat.shape, -1, np.int32)
    src_of = np.full(Rcap, -1, np.int32)
    row_of[order], src_of[rows] = rows, order
    return row_of.reshape(idx.shape), src_of, offsets, counts


@pytest.mark.parametrize("T,k,E,align,slack", [
    (0, 2, 5, 4, 3), (1, 1, 1, 1, 0), (21, 3, 7, 1, 0), (64, 1, 33, 16, 5), (65, 1, 64, 128, 0), (1023, 1, 3, 1, 1),
    (512, 2, 512, 2, 0), (205, 5, 513, 1, 0), (4096, 2, 32, 128, 0), (8193, 1, 300, 1, 0), (1000, 2, 8, 1, 70000),
    (6000, 4, 1024, 1, 0), (40000, 1, 1, 128, 9000), (5000, 8, 257, 8, 0)])
def test_row_map(B, ctx, T, k, E, align, slack):
    g = np.random.default_rng(T + k + E)
    idx = g.integers(-1, E + 1, size=(T, k)).astype(np.int32)          # some slots name no expert of this GPU
    idx[g.random((T, k)) < 0.4] = E // 2                                # ... and one expert is hot
    Rcap = T * k + E * (align - 1) + slack + (1 if T == 0 else 0)
    ref = _maps(idx, E, align, Rcap)
    for static in (False, True):
        src_of, offsets, counts = (torch.full(r.shape, -9, dtype=torch.int32, device="cuda") for r in ref[1:])
        room = max(T, 1)                                               # (an empty tensor has no address)
        row_of = torch.full((room, k), -9, dtype=torch.int32, device="cuda")
        d = torch.zeros((room, k), dtype=torch.int32, device="cuda")
        d[:T] = torch.from_numpy(idx)
        if static:
            B.moe_permute_static(None, B.BF16, d, T, k, 64, E, align, None, Rcap, row_of, src_of, offsets, counts)
        else:
            B.moe_permute(ctx, None, B.BF16, d, T, k, 64, E, align, None, Rcap, row_of, src_of, offsets, counts)
        torch.cuda.synchronize()
        for name, got, want in zip(("row_of", "src_of", "offsets", "counts"), (row_of[:T], src_of, offsets, counts), ref):
            assert np.array_equal(got.cpu().numpy(), want), (name, static)
    # dO: copies of dY in the mapped rows, zeros in all the others
    h = 72
    dY = torch.from_numpy(g.normal(size=(room, h)).astype(np.float32)).cuda()
    dO = torch.full((Rcap, h), float("nan"), device="cuda")
    B.moe_unpermute_combine_bwd(ctx, dY, None, B.F32, row_of, src_of, None, T, k, h, Rcap, dO, None)
    want = torch.zeros_like(dO)
    s = src_of.long()
    want[s >= 0] = dY[torch.div(s[s >= 0], k, rounding_mode="floor")]
    assert torch.equal(dO, want)
