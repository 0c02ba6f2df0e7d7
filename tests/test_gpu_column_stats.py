"""Column statistics at the edges of the kernels' row ranges against a sort.

Both results are order statistics, so they must equal the sorted column's
exactly: the largest magnitude and the mean of the two middle ones, formed in
fp64 from two fp32 values (numpy's median of the fp64 column)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrows", [1, 2, 127, 128, 129, 4095, 4096, 4097, 8192, 8193, 12287, 12288,
                                   12289])
@pytest.mark.parametrize("ncols", [1, 13, 264])
def test_order_statistics_at_range_edges(nrows, ncols):
    import torch

    import paper_2609_38477_amd as sq
    rng = np.random.default_rng(nrows * 1000 + ncols)
    W = rng.normal(0, 0.02, (nrows, ncols)).astype(np.float32)
    kinds = ncols // 13
    if kinds:
        W[:, 0] = 0.0                                                   # all equal, all zero
        W[:, 1] = np.where(np.arange(nrows) % 2, np.float32(-3.5), np.float32(3.5))
        W[: (nrows + 1) // 2, 2] = 0.0                                  # the middle pair far apart
        W[:, 3] = np.float32(1) + np.float32(2**-23) * rng.integers(0, 4, nrows)
        W[:, 4] = np.ldexp(np.float32(1), rng.integers(-149, 127, nrows)).astype(np.float32)
        W[nrows - 1, 5] = np.inf
        W[0, 6] = np.finfo(np.float32).max
        W[:, 7] = np.float32(2**-149) * rng.integers(0, 3, nrows)       # denormals
        W[:, 8] = np.arange(nrows, dtype=np.float32)
    mx = torch.full((ncols,), -1.0, dtype=torch.float64, device="cuda")
    md = torch.full_like(mx, -1.0)
    sq.seedq_column_stats(torch.from_numpy(W).cuda(), nrows, ncols, mx, md)
    a = np.abs(W).astype(np.float64)
    assert np.array_equal(mx.cpu().numpy(), a.max(axis=0))
    assert np.array_equal(md.cpu().numpy(), np.median(a, axis=0))


def test_more_columns_than_the_register_kernels_grid_holds():
    # 2^25 columns in groups of 8 by 1024 threads would make 2^32 threads
    import torch

    import paper_2609_38477_amd as sq
    ncols = (1 << 25) + 13
    W = torch.randn(2, ncols, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    mx = torch.full((ncols,), -1.0, dtype=torch.float64, device="cuda")
    md = torch.full_like(mx, -1.0)
    sq.seedq_column_stats(W, 2, ncols, mx, md)
    a = W.abs()
    assert torch.equal(mx, a.max(0).values.double())
    assert torch.equal(md, (a[0].double() + a[1].double()) / 2)
