"""ELL products at the edges of their chunks: the generic-width kernel (eight slots a
chunk) against the 28-wide one with zero weights behind, bit for bit (the sums are
taken in the same order), and the transposed product at column lengths around its
chunk of entries against an FP64 sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 63, 65, 4097])
@pytest.mark.parametrize("k", [1, 7, 8, 9, 16, 23, 24, 27])
def test_generic_width_equals_padded(gpu, rows, k):
    import torch
    import paper_2206_06495_amd as P
    g = torch.Generator().manual_seed(100 * k + rows)
    n = rows + 5
    idx = torch.randint(0, n, (28, rows), generator=g, dtype=torch.int32)
    for dt in (torch.float64, torch.float32):
        w = torch.rand(28, rows, generator=g, dtype=dt) - 0.5
        w[k:] = 0
        x = torch.rand(n, generator=g, dtype=dt).to(gpu)
        full = P.ell_apply(idx.to(gpu), w.to(gpu), x)
        part = P.ell_apply(idx[:k].contiguous().to(gpu), w[:k].contiguous().to(gpu), x)
        assert torch.equal(full, part)


@pytest.mark.parametrize("ncols", [1, 2, 64, 65, 130])
@pytest.mark.parametrize("rows", [3, 63, 64, 65, 127, 257, 1000])
def test_transposed_chunk_edges(gpu, rows, ncols):
    import torch
    import paper_2206_06495_amd as P
    r = np.random.default_rng(rows * 1000 + ncols)
    k = 5
    idx = r.integers(0, ncols, (k, rows)).astype(np.int32)
    if ncols > 2:
        idx[idx == 1] = 0  # one empty column
    w = r.random((k, rows)) - 0.5
    y = r.random(rows) - 0.5
    ref = np.zeros(ncols)
    mag = np.zeros(ncols)
    np.add.at(ref, idx, w * y)
    np.add.at(mag, idx, np.abs(w * y))
    if np.bincount(idx.ravel()).max() > 4096:  # refused: the documented column limit
        with pytest.raises(P.RbfError):
            P.ell_transpose(torch.from_numpy(idx).to(gpu), ncols)
        return
    tr = P.ell_transpose(torch.from_numpy(idx).to(gpu), ncols)
    z = tr.apply(tr.weights(torch.from_numpy(w).to(gpu)), torch.from_numpy(y).to(gpu))
    z = z.cpu().numpy()
    # a serial sum of m products is off by at most m eps times their magnitudes
    assert np.all(np.abs(z - ref) <= 2 * k * rows * np.finfo(float).eps * mag)
