"""ELL products at the sizes where their default launch shapes change: 32,768 rows (block
size and group of slots), 48 MiB (load kind) and, transposed, 131,072 columns (entries
in a chunk), with widths that leave every remainder of their groups, on columns
scattered around the row.  Forward bit for bit against the 28-wide kernel or a fused
sum in the same order, transposed against an FP64 sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _operator(rows, ncols, k, gen, dt):
    import torch
    at = torch.arange(rows, dtype=torch.int64)
    idx = ((at + torch.randint(-500, 501, (k, rows), generator=gen)) % ncols).int()
    return idx, torch.rand(k, rows, generator=gen, dtype=dt) - 0.5


@pytest.mark.parametrize("rows", [32767, 32768, 32769, 149796, 149797])
@pytest.mark.parametrize("k", [3, 4, 12, 21, 22, 23, 28])
def test_default_shapes(gpu, rows, k):
    import torch
    import paper_2206_06495_amd as P
    print(rows, k, flush=True)
    g = torch.Generator().manual_seed(rows + k)
    idx, w = _operator(rows, rows, 28, g, torch.float64)
    w[k:] = 0
    for dt in (torch.float64, torch.float32):
        x = torch.rand(rows, generator=g, dtype=dt).to(gpu)
        wd = w.to(dt).to(gpu)
        full = P.ell_apply(idx.to(gpu), wd, x)
        part = P.ell_apply(idx[:k].contiguous().to(gpu), wd[:k].contiguous(), x)
        assert torch.equal(full, part)
        ref = (w[:k].to(dt).double() * x.cpu().double()[idx[:k].long()]).sum(0)
        # a fused sum of k products below 1/2: at most k roundings of at most k / 2
        tol = k * k / 2 * torch.finfo(dt).eps
        assert float((part.cpu().double() - ref).abs().max()) <= tol


@pytest.mark.parametrize("ncols", [131071, 131072, 131073, 131500])
@pytest.mark.parametrize("k", [1, 5])
def test_transposed_chunks(gpu, ncols, k):
    import torch
    import paper_2206_06495_amd as P
    print(ncols, k, flush=True)
    g = torch.Generator().manual_seed(ncols + k)
    rows = ncols + 300
    idx, w = _operator(rows, ncols, k, g, torch.float64)
    idx[0, :600] = 7  # a column longer than a chunk
    y = torch.rand(rows, generator=g, dtype=torch.float64) - 0.5
    T = P.ell_transpose(idx.to(gpu), ncols)
    for dt in (torch.float64, torch.float32):
        wt = T.weights(w.to(dt).to(gpu))
        z = T.apply(wt, y.to(dt).to(gpu)).cpu().double().numpy()
        prod = (w.to(dt).double() * y.to(dt).double()).numpy().ravel()
        ref = np.bincount(idx.numpy().ravel(), prod, ncols)
        mag = np.bincount(idx.numpy().ravel(), np.abs(prod), ncols)
        count = np.bincount(idx.numpy().ravel(), minlength=ncols)
        # a serial sum of m rounded products is off by at most m + 1 eps of their magnitudes
        assert np.all(np.abs(z - ref) <= (count + 1) * float(torch.finfo(dt).eps) * mag)
