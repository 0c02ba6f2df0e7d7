"""The search's launch rules on both sides of their lines: how many 32-block tiles a wave owns
(1, 2 or 4, the last one in two kernels) and into how many ranges of seed tiles a rung is cut
follow the count of blocks, and none of it may show in the codes."""
import numpy as np
import pytest

import synthetic
from test_gpu_parity import _dev, check_search, sq, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# count of blocks from which units of 512 blocks x (2^K / 256) ranges reach 6144 workgroups
@pytest.mark.parametrize("K,P,line", [(12, 2, 196608), (12, 3, 196608), (12, 4, 196608),
                                      (15, 4, 24576), (13, 5, 98304), (14, 5, 49152),
                                      (13, 6, 98304)])
def test_search_same_codes_at_every_tile_count(sq, oq, torch, K, P, line):  # noqa: F811
    # one call of a little more than `line` blocks (a ragged last workgroup, an
    # all-zero block) against the same rows in four calls of one tile per wave
    # and more ranges: the codes must be equal bit for bit, and 128 of the
    # blocks are compared with the oracle's exhaustive search
    G = 257
    rows = line // G + 4
    W = synthetic.weights(rows, 8 * G, 0.02, key=40 + 7 * K + P, outlier_frac=0.01)
    W[1, 8 * 5:8 * 6] = 0.0
    b = sq.build_bases(K, P)
    d = _dev(torch, W)
    whole = [t.cpu() for t in sq.compress(d, [b])]
    cuts = [rows * i // 4 for i in range(5)]
    parts = [sq.compress(d[r0:r1], [b]) for r0, r1 in zip(cuts, cuts[1:])]
    for i, a in enumerate(whole):
        assert torch.equal(a, torch.cat([p[i] for p in parts]).cpu()), (K, P, i)
    at = np.linspace(0, rows * G - 1, 128).astype(np.int64)
    seed, e, q, err = (t.numpy()[at] for t in whole)
    check_search(oq, W.reshape(-1, 8)[at], K, P, seed.view(np.uint32), e, q, err, f"K{K}P{P}")
