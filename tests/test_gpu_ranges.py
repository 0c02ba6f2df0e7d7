"""The search's launch rules on both sides of their lines: how many 32-block tiles a wave owns
(1, 2 or 4, the last one in two kernels) and into how many ranges of seed tiles a rung is cut
follow the count of blocks, and none of it may show in the codes."""
import os

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


def _with_ranges(tiles, f):
    saved = os.environ.pop("SEEDQ_SEED_CHUNK_TILES", None)
    try:
        if tiles is not None:
            os.environ["SEEDQ_SEED_CHUNK_TILES"] = tiles
        return [t.cpu() for t in f()]
    finally:
        os.environ.pop("SEEDQ_SEED_CHUNK_TILES", None)
        if saved is not None:
            os.environ["SEEDQ_SEED_CHUNK_TILES"] = saved


@pytest.mark.parametrize("rungs", [[(8, 1)], [(8, 4)], [(9, 5)], [(8, 6)], [(12, 2)], [(12, 3)],
                                   [(13, 4)], [(12, 5)], [(12, 6)], [(8, 2), (12, 3), (15, 4)]])
def test_a_walk_of_one_range_emits_the_same_codes(sq, torch, rungs):  # noqa: F811
    # one range (the walk writes the codes), the rule's ranges and ranges of 8 tiles
    # (a kernel emits from the keys): the same codes and errors, all-zero blocks and
    # blocks without any finite weight among them
    G, rows = 203, 8
    W = synthetic.weights(rows, 8 * G, 0.02, key=60 + len(rungs) + rungs[0][1], outlier_frac=0.01)
    b = W.reshape(-1, 8)
    b[5] = b[700] = 0.0
    b[6] = b[701] = b[1623] = np.nan
    bases = [sq.build_bases(K, P) for K, P in rungs]
    d, rob = _dev(torch, W), None
    if len(rungs) > 1:
        rob = _dev(torch, (np.arange(rows * G) * 7 // 5 % len(rungs)).astype(np.uint8))
    out = {v: _with_ranges(v, lambda: sq.compress(d, bases, rob)) for v in ("0", None, "8")}
    for v in (None, "8"):
        for a, c in zip(out["0"], out[v]):
            assert torch.equal(a, c), (rungs, v)
    seed, e, q, err = (t.numpy() for t in out["8"])
    for i in (5, 700, 6, 701, 1623):   # no seed is better than another: the smallest one
        assert seed[i] == 1 and e[i] == 15 and not q[i].any() and err[i] == 0.0


@pytest.mark.parametrize("K,P", [(12, 1), (12, 3), (13, 4), (16, 4), (12, 5), (12, 6)])
def test_blocks_that_are_not_finite_do_not_depend_on_the_ranges(sq, torch, K, P):  # noqa: F811
    # the contract asks for finite weights; a block without them still gets one code,
    # from the first seed tile, whatever the ranges and the order in which they run
    W = synthetic.weights(4, 8 * 203, 0.02, key=70 + K + P)
    b = W.reshape(-1, 8)
    bad = [3, 40, 41, 300, 555, 811]
    for n, i in enumerate(bad):
        b[i, n] = [np.nan, np.inf, -np.inf][n % 3]
    b[300] = [np.inf, -np.inf] * 4
    big = np.concatenate([W] * 40)   # and in a call of several block tiles a wave
    bases = [sq.build_bases(K, P)]
    first = _with_ranges("0", lambda: sq.compress(_dev(torch, W), bases))
    assert bool((first[0][bad] <= 32).all()) and bool((first[0][bad] >= 1).all())
    for v in (None, "8", "8"):
        for part in (W, big):
            got = _with_ranges(v, lambda: sq.compress(_dev(torch, part), bases))
            for a, c in zip(first[:3], got[:3]):
                n = len(first[0])
                for k in range(0, len(c), n):
                    assert torch.equal(a, c[k:k + n]), (K, P, v)
