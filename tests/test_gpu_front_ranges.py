"""The front end's launch rules at their lines, and at sizes where a launch of sixteen threads an
element would hold more than 2^32 of them."""
import numpy as np
import pytest

from oracle import importance as oimp
from test_gpu_frontend import _t, sq  # noqa: F401

pytestmark = pytest.mark.gpu


def _silu(sq, var, nodes):
    import torch
    out = torch.full_like(var, -1.0)
    sq.seedq_expect_silu_sq(var, var.numel(), nodes, out)
    return out


def test_expectation_of_more_channels_than_sixteen_threads_each(sq):  # noqa: F811
    import torch
    n = (1 << 28) + 5
    var = torch.rand(n, dtype=torch.float64, device="cuda")
    out = _silu(sq, var, 2)
    for part in (slice(0, 4099), slice((1 << 28) - 7, n)):
        ref = oimp.e_silu_sq(var[part].cpu().numpy(), 2)
        assert np.allclose(out[part].cpu().numpy(), ref, rtol=1e-12, atol=0)
    assert float(out.min()) >= 0.0   # every channel was written


def test_transposed_product_of_more_columns_than_sixteen_threads_each(sq):  # noqa: F811
    import torch

    from paper_2609_38477_amd import frontend
    n = (1 << 28) + 16
    W = torch.rand(1, n, device="cuda") + 0.5
    got = frontend.sq_gemv(W, torch.full((1,), 3.0, device="cuda"), transpose=True)
    want = W[0].double().square().mul_(3.0).cpu().numpy()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("nodes", [1, 2, 15, 16, 17, 128])
def test_expectation_at_the_line(sq, nodes):  # noqa: F811
    # sixteen threads a channel up to 2048 channels a node, one above: 1e-12 of fp64
    # sums in either order
    for n in (1, 17, 2048 * nodes - 1, 2048 * nodes, 2048 * nodes + 1):
        rng = np.random.default_rng(n + nodes)
        var = np.exp(rng.normal(0, 2, n))
        var[0] = 0.0
        got = _silu(sq, _t(var), nodes).cpu().numpy()
        at = np.unique(np.linspace(0, n - 1, 300).astype(np.int64))
        assert np.allclose(got[at], oimp.e_silu_sq(var[at], nodes), rtol=1e-12, atol=0)
        assert np.all(got >= 0.0)


@pytest.mark.parametrize("ncols", [1, 1 << 17, (1 << 17) + 1])
def test_transposed_product_at_the_line(sq, ncols):  # noqa: F811
    import torch

    from paper_2609_38477_amd import frontend
    nrows = 600   # three row chunks
    W = torch.randn(nrows, ncols, device="cuda", generator=torch.Generator(device="cuda").manual_seed(7))
    v = torch.rand(nrows, device="cuda") + 0.1
    got = frontend.sq_gemv(W, v, transpose=True)
    want = (W.double().square() * v.double()[:, None]).sum(0).cpu().numpy()
    assert np.allclose(got, want, rtol=1e-12, atol=0)
