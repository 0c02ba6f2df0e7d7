"""The decoders' stores on both sides of their rule (past the caches where a call reads and writes
more than 256 MiB): the same results, and below it an output that its reader finds in the caches."""
import pytest

from test_gpu_stream import sq  # noqa: F401

pytestmark = pytest.mark.gpu

RUNGS = [(12, 2), (16, 3), (20, 4)]


def _codes(rows, cols, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    nb = rows * cols // 8
    rob = (torch.arange(cols // 8, device="cuda") * 3 // (cols // 8)).to(torch.uint8).repeat(rows)
    K = torch.tensor([k for k, _ in RUNGS], device="cuda")[rob.long()]
    P = torch.tensor([p for _, p in RUNGS], device="cuda")[rob.long()]
    s = (torch.randint(1 << 30, (nb,), device="cuda", generator=g) % ((1 << K) - 1) + 1).to(torch.int32)
    e = torch.randint(0, 16, (nb,), device="cuda", generator=g, dtype=torch.uint8)
    q = torch.randint(-8, 8, (nb, 8), device="cuda", generator=g, dtype=torch.int8)
    q *= torch.arange(8, device="cuda") < P[:, None]
    return rob, s, e, q, torch.bincount(rob.long(), minlength=3).tolist()


def test_same_results_on_both_sides(sq):  # noqa: F811
    # 8192 x 16384 (512 MiB of weights, 208 MiB of codes and 64 of stream) against its
    # quarters, of which only the permutation's read and write no more than 256 MiB
    import torch
    rows, cols = 8192, 16384
    rob, s, e, q, cnt = _codes(rows, cols, 1)
    quarter = rows * cols // 32
    words = sq.pack(s, e, q, RUNGS, rows, cols, rob, cnt)
    W = sq.decompress_stream(words, RUNGS, rows, cols, rob)
    W2, acc = sq.decompress(s, e, q, RUNGS, rows, cols, rob, with_acc=True)
    assert torch.equal(W, W2)
    back = sq.unpack(words, RUNGS, rows, cols, rob)
    assert all(torch.equal(a, b) for a, b in zip(back, (s, e, q)))
    perm = torch.randperm(cols, device="cuda").to(torch.int32)
    out = [torch.empty_like(W) for _ in range(2)]
    for inverse in (0, 1):
        sq.seedq_permute_columns(W, rows, cols, perm, inverse, out[inverse])
    assert torch.equal(out[0], W[:, perm.long()]) and torch.equal(out[1][:, perm.long()], W)
    for i in range(4):
        b, r = slice(i * quarter, (i + 1) * quarter), slice(i * rows // 4, (i + 1) * rows // 4)
        part = sq.decompress(s[b], e[b], q[b], RUNGS, rows // 4, cols, rob[b], with_acc=True)
        assert torch.equal(part[0], W[r]) and torch.equal(part[1], acc[r])
        w = sq.pack(s[b], e[b], q[b], RUNGS, rows // 4, cols, rob[b], [c // 4 for c in cnt])
        assert torch.equal(sq.decompress_stream(w, RUNGS, rows // 4, cols, rob[b]), W[r])
        assert all(torch.equal(x, y[b]) for x, y in
                   zip(sq.unpack(w, RUNGS, rows // 4, cols, rob[b]), (s, e, q)))
        o = torch.empty(rows // 4, cols, device="cuda")
        sq.seedq_permute_columns(W[r], rows // 4, cols, perm, 1, o)
        assert torch.equal(o, out[1][r])


@pytest.mark.parametrize("codes", [False, True])
def test_weights_stay_for_their_reader(sq, codes):  # noqa: F811
    # 128 MiB of weights right after they were decoded and right after torch copied
    # them: the permutation that reads them takes the same time (0.98 times), 1.5 times
    # as long where the decoder stored past the caches
    import torch
    rows, cols = 4096, 8192
    rob, s, e, q, cnt = _codes(rows, cols, 2)
    words = sq.pack(s, e, q, RUNGS, rows, cols, rob, cnt)
    perm = torch.randperm(cols, device="cuda").to(torch.int32)
    src, out = torch.empty(rows, cols, device="cuda"), torch.empty(rows, cols, device="cuda")
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def reader_ms(make):
        ms = []
        for _ in range(9):
            W = make()
            a.record()
            sq.seedq_permute_columns(W, rows, cols, perm, 1, out)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        return sorted(ms)[4]

    W = sq.decompress_stream(words, RUNGS, rows, cols, rob)
    copied = reader_ms(lambda: src.copy_(W))
    decoded = reader_ms(lambda: sq.decompress(s, e, q, RUNGS, rows, cols, rob)[0] if codes
                        else sq.decompress_stream(words, RUNGS, rows, cols, rob))
    assert decoded < 1.15 * copied, (decoded, copied)
