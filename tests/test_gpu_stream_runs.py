"""The stream kernels where neighbouring blocks share a rung (wave steps of 128 blocks with one
rung, two packed registers for K <= 16), at the edges of such runs, across blocks without bits, and
with the offsets taken from group sums or from the scan. Packed words, codes and weights are
bit-exact; the decode-GEMV is held to its fp32 bound."""
import numpy as np
import pytest

from oracle import stream as ostream
from test_gpu_stream import _codes, _t, _words, sq  # noqa: F401

pytestmark = pytest.mark.gpu

# every P and the registers at the edges of the packed path (8, 15, 16 | 17, 24)
RUNGS = [(8, 1), (9, 2), (15, 3), (16, 4), (16, 5), (12, 6), (17, 3), (24, 6)]


def _check(sq, oq, rob, rungs, nrows, ncols, nvecs=(1, 4, 8), many=False):
    rng = np.random.default_rng(len(rob) + nrows)
    seed, exp, q = (_many_codes if many else _codes)(rng, rob, rungs)
    valid = rob < len(rungs)
    cnt = np.bincount(rob[valid], minlength=len(rungs))
    d = _t(rob) if len(rungs) > 1 else None
    w = sq.pack(_t(seed.view(np.int32)), _t(exp), _t(q), rungs, nrows, ncols, d, cnt)
    if not many:   # the oracle's packer is slow
        assert np.array_equal(_words(w), ostream.pack(seed[valid], exp[valid], q[valid], rob[valid], rungs))
    s, e, qq = (t.cpu().numpy() for t in sq.unpack(w, rungs, nrows, ncols, d))
    assert np.array_equal(s.view(np.uint32)[valid], seed[valid]) and np.all(s[~valid] == 0)
    assert np.array_equal(e[valid], exp[valid]) and np.array_equal(qq[valid], q[valid])
    Wh = sq.decompress_stream(w, rungs, nrows, ncols, d).cpu().numpy()
    K = np.array([rungs[r][0] if r < len(rungs) else 8 for r in rob])
    P = np.array([rungs[r][1] if r < len(rungs) else 1 for r in rob])
    want, _ = oq.decompress(seed[valid], exp[valid], q[valid], K[valid], P[valid])
    got = Wh.reshape(-1, 8)
    assert np.array_equal(got[valid], np.asarray(want, dtype=np.float32).reshape(-1, 8))
    assert np.isnan(got[~valid]).all()
    G = ncols // 8
    x = rng.normal(0, 1, (8, ncols)).astype(np.float32)
    exact = np.where(np.isnan(Wh), 0, Wh).astype(np.float64) @ x.T.astype(np.float64)
    size = np.abs(np.where(np.isnan(Wh), 0, Wh)).astype(np.float64) @ np.abs(x.T).astype(np.float64)
    bad = np.isnan(Wh).any(1)
    for nv in nvecs:
        y = sq.gemv_stream(w, rungs, nrows, ncols, _t(x[:nv]), d).cpu().numpy().T
        # a lane's chain of at most 8 products a block over every 64th block, the
        # lanes' and the segments' sums; the matrix-core kernel's shares
        n = 8 * -(-G // 64) + 58
        assert np.all(np.abs(y - exact[:, :nv])[~bad] <= n * 2.0 ** -24 * size[:, :nv][~bad])
        assert np.isnan(y[bad]).all()


@pytest.mark.parametrize("nrows,G", [(1, 128), (3, 300), (17, 1031), (2, 2048), (40, 257)])
def test_runs_of_one_rung(sq, oq, nrows, G):  # noqa: F811
    # rungs in runs of 1 to 700 blocks across rows, so that wave steps fall inside
    # a run, on its edge and across several
    rng = np.random.default_rng(G)
    rob = np.concatenate([np.full(int(rng.integers(1, 700)), r % len(RUNGS), np.uint8)
                          for r in rng.permutation(3 * (nrows * G // 100 + 8))])[:nrows * G]
    _check(sq, oq, rob, RUNGS, nrows, 8 * G)


@pytest.mark.parametrize("K,P", RUNGS)
def test_one_rung_without_rung_bytes(sq, oq, K, P):  # noqa: F811
    # offsets are products; 2100 blocks a row: a ragged last step and chunk
    _check(sq, oq, np.zeros(2 * 2100, np.uint8), [(K, P)], 2, 8 * 2100)


def test_words_across_blocks_without_bits(sq, oq):  # noqa: F811
    # a word's codes may lie in chunks far apart: thousands of blocks without bits
    # between two codes, whole chunks of them, and at both ends
    rob = np.full(5 * 2048 + 77, 255, np.uint8)
    rob[[5, 6, 2047, 2048, 2049, 7000, 7001, 7002, 9000, 10239, 10240]] = [0, 1, 0, 1, 0, 1, 1, 0, 1, 0, 0]
    rob[4096:4200] = 1
    _check(sq, oq, rob, [(8, 1), (9, 2)], 1, 8 * len(rob), nvecs=())


def _pack_ms(sq, rob, rungs):
    import torch
    nb = len(rob)
    cnt = np.bincount(rob[rob < len(rungs)], minlength=len(rungs))
    seed, exp = torch.ones(nb, dtype=torch.int32, device="cuda"), torch.ones(nb, dtype=torch.uint8, device="cuda")
    args = (seed, exp, torch.ones(nb, 8, dtype=torch.int8, device="cuda"), rungs, 1, 8 * nb, _t(rob), cnt)
    ms = []
    for _ in range(6):   # the first one warms up
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        sq.pack(*args)
        b.record()
        torch.cuda.synchronize()
        ms.append(a.elapsed_time(b))
    return min(ms[1:])


def test_long_stretch_without_bits_costs_no_more_than_codes(sq, oq):  # noqa: F811
    # hundreds of chunks without bits behind an unaligned code, another code after
    # them: only the word's own chunk looks for its end, and by chunks (38 us against
    # 27 with every block coded; every chunk going through all blocks after it would
    # take milliseconds)
    rungs = [(8, 1), (9, 2)]
    rob = np.full(400 * 2048 + 131, 255, np.uint8)
    rob[[0, 2, 3, len(rob) - 3]] = [0, 1, 0, 1]
    _check(sq, oq, rob, rungs, 1, 8 * len(rob), nvecs=())
    full = np.resize(np.array([0, 1], np.uint8), len(rob))
    assert _pack_ms(sq, rob, rungs) < 10 * _pack_ms(sq, full, rungs)


def _many_codes(rng, rob, rungs):
    """_codes for many blocks."""
    n, r = len(rob), np.minimum(rob, len(rungs))
    K = np.array([k for k, _ in rungs] + [1])[r]
    P = np.array([p for _, p in rungs] + [0])[r]
    seed = np.where(r < len(rungs), rng.integers(0, 1 << 30, n) % ((1 << K) - 1) + 1, 0)
    q = rng.integers(-8, 8, (n, 8)) * (np.arange(8) < P[:, None])
    return seed.astype(np.uint32), rng.integers(0, 16, n).astype(np.uint8), q.astype(np.int8)


# one step of 128 blocks a row, two (the second of 12 blocks), four and nine of them, at
# the row counts where the waves a row change and where a workgroup's last rows are past
# the end
@pytest.mark.parametrize("nrows,G", [(2047, 100), (2047, 140), (2048, 140), (2049, 140),
                                     (2047, 400), (2048, 400), (2049, 400), (4095, 400), (4096, 400),
                                     (4097, 400), (2047, 1030), (2051, 1030), (4099, 300)])
def test_rows_by_several_waves(sq, oq, nrows, G):  # noqa: F811
    rng = np.random.default_rng(nrows)
    rob = np.sort(rng.integers(0, 3, (nrows, G)), axis=1).astype(np.uint8)
    rob[:, G // 3:G // 2] = rng.integers(0, 3, (nrows, G // 2 - G // 3))
    rob[::97, G - 1] = 255    # rows poisoned by a block without a code, the last one
    rob[50::89, 3] = 9
    rob[nrows - 1] = 2
    _check(sq, oq, rob.ravel(), [(12, 2), (16, 3), (20, 4)], nrows, 8 * G, nvecs=(1, 2, 4),
           many=True)


def test_one_wave_for_each_of_very_many_rows(sq):  # noqa: F811
    # two waves for each of 2^25 rows would be more threads than a launch holds
    import torch
    nrows = (1 << 25) + 3
    g = torch.Generator(device="cuda").manual_seed(5)
    seed = torch.randint(1, 256, (nrows,), device="cuda", generator=g, dtype=torch.int32)
    exp = torch.randint(0, 16, (nrows,), device="cuda", generator=g, dtype=torch.uint8)
    q = torch.zeros(nrows, 8, dtype=torch.int8, device="cuda")
    q[:, 0] = torch.randint(-8, 8, (nrows,), device="cuda", generator=g, dtype=torch.int8)
    w = sq.pack(seed, exp, q, [(8, 1)], nrows, 8)
    W = sq.decompress(seed, exp, q, [(8, 1)], nrows, 8)[0].double()
    x = torch.randn(2, 8, device="cuda", generator=g)
    y = sq.gemv_stream(w, [(8, 1)], nrows, 8, x)
    for v in range(2):
        p = W * x[v].double()   # (a matrix product of so many rows comes back cut)
        want, size = p.sum(1), p.abs().sum(1)
        assert bool(((y[v].double() - want).abs() <= 16 * 2.0 ** -24 * size).all())


def test_more_rows_than_group_sums_reach(sq, oq):  # noqa: F811
    # above 1024 groups of 16 rows the decode-GEMV takes its offsets from the scan
    nrows, G = 16 * 1024 + 9, 3
    rng = np.random.default_rng(4)
    _check(sq, oq, rng.integers(0, 3, nrows * G).astype(np.uint8), [(8, 1), (16, 3), (20, 4)], nrows,
           8 * G)


def test_offsets_from_the_scan_of_many_chunks(sq):  # noqa: F811
    # above 16384 chunks (33.5 M blocks) the packer and the parsers take their offsets
    # from the scan; a long stretch without bits lies behind an unaligned code. The same
    # blocks in calls below the line, cut where a word ends
    import torch
    rungs = [(8, 1), (12, 4)]   # 16 and 32 bits
    nb = (1 << 25) + 70001
    g = torch.Generator(device="cuda").manual_seed(6)
    rob = torch.randint(0, 2, (nb,), device="cuda", generator=g, dtype=torch.uint8)
    gap = (9000001, 20000003)
    rob[gap[0]:gap[1]] = 200
    cuts = [0, 8000000, 25000000, nb]
    for c in cuts[1:3]:   # an even number of 16-bit codes before a cut
        rob[c - 1] = 1
        if int((rob[:c] == 0).sum()) % 2:
            rob[c - 2] = 1 - rob[c - 2]
    rob[gap[0] - 1] = 1
    if int((rob[:gap[0]] == 0).sum()) % 2 == 0:
        rob[gap[0] - 2] = 1 - rob[gap[0] - 2]
    if int((rob[:cuts[2]] == 0).sum()) % 2:
        rob[cuts[2] - 2] = 1 - rob[cuts[2] - 2]
    valid = rob < 2
    P = torch.tensor([1, 4, 0], device="cuda")[rob.clamp(max=2).long()]
    top = torch.tensor([255, 4095, 1], device="cuda")[rob.clamp(max=2).long()]
    seed = (torch.randint(1 << 30, (nb,), device="cuda", generator=g) % top + 1).to(torch.int32)
    seed[~valid] = 0
    exp = torch.randint(0, 16, (nb,), device="cuda", generator=g, dtype=torch.uint8) * valid
    q = torch.randint(-8, 8, (nb, 8), device="cuda", generator=g, dtype=torch.int8)
    q *= torch.arange(8, device="cuda") < P[:, None]

    def count(r):
        return [int((r == 0).sum()), int((r == 1).sum())]

    words = sq.pack(seed, exp, q, rungs, 1, 8 * nb, rob, count(rob))
    parts = []
    for a, b in zip(cuts, cuts[1:]):
        c = count(rob[a:b])
        assert c[0] % 2 == 0 or b == nb
        parts.append(sq.pack(seed[a:b], exp[a:b], q[a:b], rungs, 1, 8 * (b - a), rob[a:b], c))
    assert torch.equal(words, torch.cat(parts))
    for x, y in zip(sq.unpack(words, rungs, 1, 8 * nb, rob), (seed, exp, q)):
        assert torch.equal(x, y)
    W = sq.decompress_stream(words, rungs, 1, 8 * nb, rob).view(-1, 8)
    W2 = sq.decompress(seed, exp, q, rungs, 1, 8 * nb, rob)[0].view(-1, 8)
    assert torch.equal(W[valid], W2[valid]) and bool(W[~valid].isnan().all())
