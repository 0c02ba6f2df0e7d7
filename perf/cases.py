"""The calls that a user of this library makes, at the sizes they are made: the seed search of an
encoder (one tensor at a time, from a toy matrix to a 4096 x 14336 layer, one rung or three), the
whole encode and decode of a tensor, the emission of the code stream, and what a decoder does with
it (reconstruction, and products with vectors straight from the stream), and the importance of a
layer from which the rungs are planned.

In a case, ``sorted`` says whether the caller put the channels in order of importance (the encoder
of a layer does), or left them as they were, so that rungs change from block to block.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges, ``prepare`` makes what a
program has in hand, ``run`` is one pass through the public entry points. Sizes are those of
``synthetic.WORKLOADS`` and ``synthetic.synthetic_layer`` and of their projections. Weights are
N(0, 0.02^2) with 0.1 % heavy-tailed outliers, as in ``synthetic.weights``, drawn on the GPU.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2609_38477_amd as sq
from paper_2609_38477_amd import frontend

THREE = "12,2;16,3;20,4"          # the rungs of the multi-rung workloads
DAMAGE = (4.0, 1.0, 0.25)
MASKS = {8: 0xB8, 9: 0x110, 10: 0x240, 11: 0x500, 12: 0x829, 13: 0x100D, 14: 0x2015, 15: 0x6000,
         16: 0xD008, 17: 0x12000, 18: 0x20400, 19: 0x40023, 20: 0x90000}


def listed():
    return [
        # The smallest call: a 256 x 256 matrix at one small rung. Launch and latency bound.
        dict(name="search_tiny", kind="search", rows=256, cols=256, rungs="12,3", bpw=3.5,
             sorted=True),
        # A key or value projection with shared heads, three rungs: the ordinary small tensor.
        dict(name="search_kv", kind="search", rows=1024, cols=4096, rungs=THREE, bpw=4.0,
             sorted=True),
        # An odd shape at a lower rate: few blocks at the widest rung.
        dict(name="search_ragged", kind="search", rows=1001, cols=2056, rungs=THREE, bpw=3.5,
             sorted=True),
        # A uniform build at one of the grid's wide rungs, odd row count.
        dict(name="search_grid", kind="search", rows=1023, cols=4096, rungs="16,5", bpw=5.0,
             sorted=True),
        # The benchmark's step on an attention projection: plan, basis stack, search, decompress.
        dict(name="step_attn", kind="step", rows=4096, cols=4096, rungs="16,3", bpw=4.0,
             sorted=True),
        # The largest: an MLP up-projection at three rungs.
        dict(name="search_mlp", kind="search", rows=4096, cols=14336, rungs=THREE, bpw=4.0,
             sorted=True),
        # One tensor through the encoder and back (channel sort, plan with row factors, basis
        # stacks, search, stream; re-derivation, one-pass decode, inverse sort, FP16 columns).
        dict(name="encode_tensor", kind="tensor", rows=1024, cols=2816, rungs=THREE, bpw=4.0,
             escape=4),
        # The emit step of the encoder on a 4096 x 11008 layer's codes.
        dict(name="pack", kind="pack", rows=4096, cols=11008, rungs=THREE, bpw=3.5, sorted=True),
        # A decoder that loads a layer: the stream to fp32 weights in one pass.
        dict(name="decode", kind="decode", rows=4096, cols=14336, rungs=THREE, bpw=4.0,
             sorted=True),
        # One token against a compressed projection: decode-GEMV with one vector.
        dict(name="gemv_token", kind="gemv", rows=4096, cols=4096, rungs=THREE, bpw=4.0, nvec=1,
             sorted=True),
        # Eight vectors against the largest layer.
        dict(name="gemv_batch", kind="gemv", rows=8192, cols=28672, rungs=THREE, bpw=4.0, nvec=8,
             sorted=True),
        # The data-free importance of a 7B-shaped layer and its head: factors, channel orders,
        # column statistics, outlier columns.
        dict(name="importance", kind="importance", d=4096, f=11008, heads=32, kv=32, vocab=32000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("search", "search", "search", "search", "step", "tensor", "pack", "decode",
                       "gemv", "gemv", "importance"))
    if kind == "importance":
        kv = rng.choice((2, 4, 8))
        heads = kv * rng.choice((1, 2, 4))
        d = heads * 8 * _log(rng, 4, 4096 // (8 * heads))
        return dict(kind=kind, d=d, f=8 * _log(rng, d // 8, 11008 // 8), heads=heads, kv=kv,
                    vocab=_log(rng, 500, 32000))
    if kind == "tensor":
        return dict(kind=kind, rows=_log(rng, 128, 1024), cols=8 * _log(rng, 16, 352), rungs=THREE,
                    bpw=rng.randint(26, 37) / 8, escape=rng.choice((0, 1, 4)))
    if kind in ("search", "step"):
        if kind == "search" and rng.random() < 0.5:
            rungs, bpw = THREE, rng.randint(26, 37) / 8
            rows, cols = _log(rng, 64, 3000), 8 * _log(rng, 16, 1024)
        else:   # one rung of the grid
            K, P = rng.randint(8, 16), rng.randint(2, 6)
            rungs, bpw = "%d,%d" % (K, P), (K + 4 * P + 4) / 8
            rows, cols = _log(rng, 64, 4096), 8 * _log(rng, 16, 512)
        return dict(kind=kind, rows=rows, cols=cols, rungs=rungs, bpw=bpw,
                    sorted=rng.random() < 0.75)
    rungs, bpw = THREE, rng.randint(26, 37) / 8
    if rng.random() < 0.3:
        K, P = rng.randint(8, 16), rng.randint(2, 6)
        rungs, bpw = "%d,%d" % (K, P), (K + 4 * P + 4) / 8
    case = dict(kind=kind, rows=_log(rng, 64, 8192), cols=8 * _log(rng, 32, 3584), rungs=rungs,
                bpw=bpw, sorted=rng.random() < 0.75)
    if kind == "gemv":
        case["nvec"] = rng.choice((1, 1, 2, 4, 8))
    return case


# ---------------------------------------------------------------- inputs

def _rungs(case):
    return [tuple(int(v) for v in r.split(",")) for r in case["rungs"].split(";")]


def _damage(case):
    return DAMAGE if len(_rungs(case)) > 1 else None


def _profile(ncols, order=None):
    """Log-normal column importance in increasing order, or in the given one."""
    p = (torch.arange(ncols, dtype=torch.float64) + 0.5) / ncols
    a = torch.exp(torch.special.ndtri(p)).to(torch.float32)
    return (a if order is None else a[order]).numpy()


def _importance(case):
    if case["sorted"]:
        return _profile(case["cols"])
    g = torch.Generator().manual_seed(case["cols"])   # the order belongs to the case
    return _profile(case["cols"], torch.randperm(case["cols"], generator=g))


def _weights(rows, cols, g):
    w = torch.randn(rows, cols, device="cuda", generator=g).mul_(0.02)
    m = max(1, rows * cols // 1000)   # one outlier at a random place of every 1000 weights
    at = torch.arange(m, device="cuda") * 1000 + torch.randint(1000, (m,), device="cuda", generator=g)
    z = torch.randn(4, m, device="cuda", generator=g)
    w.view(-1)[at.clamp_(max=rows * cols - 1)] = 0.1 * z[0] / (z[1:].square().sum(0) / 3).sqrt()
    return w


def _rung_map(case, a):
    """Rung index per block (host) and the blocks per rung, as an encoder plans them."""
    rob, rep = sq.plan_schedule(case["rows"], case["cols"], _rungs(case), _damage(case),
                                case["bpw"], a)
    return rob, rep["count"]


def _codes(case, g, rob):
    """Random valid codes of the planned rungs: seeds, exponents 7..9, mantissas."""
    rungs = _rungs(case)
    nb = case["rows"] * case["cols"] // 8
    K = torch.tensor([k for k, _ in rungs], device="cuda")[rob]
    P = torch.tensor([p for _, p in rungs], device="cuda")[rob]
    r = torch.randint(1 << 30, (nb,), device="cuda", generator=g)
    seed = (r % ((1 << K) - 1) + 1).to(torch.int32)
    e = torch.randint(7, 10, (nb,), device="cuda", generator=g, dtype=torch.uint8)
    q = torch.randint(-8, 8, (nb, 8), device="cuda", generator=g, dtype=torch.int8)
    q *= torch.arange(8, device="cuda") < P[:, None]
    return seed, e, q


def prepare(case, seed):
    kind = case["kind"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    s = SimpleNamespace(case=case, kind=kind)
    if kind == "importance":
        d, f, hd = case["d"], case["f"], case["d"] // case["heads"]
        shapes = {"q": (d, d), "k": (case["kv"] * hd, d), "v": (case["kv"] * hd, d), "o": (d, d),
                  "gate": (f, d), "up": (f, d), "down": (d, f), "lm_head": (case["vocab"], d)}
        s.dW = {n: _weights(r, c, g) for n, (r, c) in shapes.items()}
        gains = {}
        for norm in ("attn", "mlp"):   # RMSNorm gains around 1, one massive channel
            gains[norm] = torch.randn(d, device="cuda", generator=g).mul_(0.3).exp_().cpu().numpy()
        gains["mlp"][seed % d] = 30.0
        s.dW["down"][seed % d, seed % f] = 20.0   # one super weight
        s.layer = SimpleNamespace(tensors=s.dW, gains=gains, n_heads=case["heads"],
                                  n_kv_heads=case["kv"], vocab=case["vocab"])
        return s
    rows, cols = case["rows"], case["cols"]
    s.rungs = _rungs(case)
    if kind == "tensor":
        s.W = _weights(rows, cols, g)
        s.a = torch.randn(cols, device="cuda", generator=g).exp_().double().cpu().numpy()
        s.rho = torch.randn(rows, device="cuda", generator=g).mul_(0.5).exp_().double().cpu().numpy()
        s.escape = sorted(int(c) for c in np.argsort(-s.a)[:case["escape"]])
        return s
    s.a = _importance(case)
    multi = len(s.rungs) > 1
    if kind in ("search", "step"):
        s.W = _weights(rows, cols, g)
        s.bases = [sq.build_bases(K, P) for K, P in s.rungs] if kind == "search" else None
        s.rob = torch.from_numpy(_rung_map(case, s.a)[0]).cuda() if multi else None
        return s
    rob, s.counts = _rung_map(case, s.a)
    rob = torch.from_numpy(rob).cuda()
    s.rob = rob if multi else None
    s.seed, s.exp, s.q = _codes(case, g, rob.long())
    if kind != "pack":
        s.words = sq.pack(s.seed, s.exp, s.q, s.rungs, rows, cols, s.rob, s.counts)
    if kind == "gemv":
        s.x = torch.randn(case["nvec"], cols, device="cuda", generator=g)
    return s


def run(s):
    kind, case = s.kind, s.case
    if kind == "importance":
        imp = frontend.layer_importance(s.layer, s.dW)
        names = list(frontend.PROJECTIONS)
        outliers = np.full((frontend.OUTLIER_COLUMNS, 2), -1, dtype=np.int64)
        for i, (n, c) in enumerate(imp.outliers):
            outliers[i] = names.index(n), c
        return {"a": imp.a, "rho": imp.rho, "perm": imp.perm,
                "stats": {n: list(v) for n, v in imp.stats.items()},
                "outliers": outliers}
    rows, cols = case["rows"], case["cols"]
    if kind == "tensor":
        enc = frontend.encode_tensor("down", s.W, s.a, s.rho, s.escape, s.rungs, DAMAGE, case["bpw"])
        out = {"words": enc.words, "perm": enc.perm, "rungs": enc.rob,
               "W": frontend.decode_tensor(enc, s.rungs, DAMAGE)}
        if enc.escape_fp16 is not None:
            out["escape"] = enc.escape_fp16
        return out
    if kind == "search":
        seed, exp, q, err = sq.compress(s.W, s.bases, s.rob)
        return {"seed": seed, "exp": exp, "q": q, "err": err}
    if kind == "step":
        rob, _ = sq.plan_schedule(rows, cols, s.rungs, _damage(case), case["bpw"], s.a)
        bases = [sq.build_bases(K, P) for K, P in s.rungs]
        seed, exp, q, err = sq.compress(s.W, bases)
        W_hat, _ = sq.decompress(seed, exp, q, s.rungs, rows, cols)
        return {"rungs": rob, "seed": seed, "exp": exp, "q": q, "err": err, "W": W_hat}
    if kind == "pack":
        return sq.pack(s.seed, s.exp, s.q, s.rungs, rows, cols, s.rob, s.counts)
    if kind == "decode":
        return sq.decompress_stream(s.words, s.rungs, rows, cols, s.rob)
    return sq.gemv_stream(s.words, s.rungs, rows, cols, s.x, s.rob)


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    kind = case["kind"]
    if kind == "importance":
        d, f, kvd = case["d"], case["f"], case["kv"] * (case["d"] // case["heads"])
        once = 2 * d * d + 2 * kvd * d + 3 * d * f + case["vocab"] * d
        products = kvd * d + 2 * d * f + case["vocab"] * d
        return {"bytes": 4 * once, "flops": 3 * products}
    rows, cols = case["rows"], case["cols"]
    n, nb = rows * cols, rows * cols // 8
    rungs = _rungs(case)
    a = _profile(cols) if kind == "tensor" else _importance(case)
    counts = _rung_map(case, a)[1]
    cands = [c * ((1 << K) - 1) * 16 * P for c, (K, P) in zip(counts, rungs)]
    payload = sum(c * (K + 4 * P + 4) for c, (K, P) in zip(counts, rungs)) / 8
    rob = nb if len(rungs) > 1 else 0
    if kind in ("search", "step", "tensor"):   # 2 C P flops a candidate: the least-squares fit
        codes = 17 * nb if kind != "tensor" else payload
        decoded = 0 if kind == "search" else 4 * n
        return {"bytes": 4 * n + rob + codes + decoded, "flops": float(sum(cands))}
    regen = 16.0 * sum(c * P for c, (_, P) in zip(counts, rungs))   # U q of every block
    if kind == "pack":
        return {"bytes": 13 * nb + rob + payload, "flops": 0}
    if kind == "decode":
        return {"bytes": payload + rob + 4 * n, "flops": regen}
    return {"bytes": payload + rob + 4 * case["nvec"] * (rows + cols),
            "flops": regen + 2.0 * case["nvec"] * n}


def tolerance(case):
    if case["kind"] == "gemv":
        # fp32 products and sums over a row (measured against 64 bits: 2e-7 of the result)
        return {"rel": 8e-7, "max": 1e-5}
    if case["kind"] == "importance":
        # 64-bit sums of a row or column in any order (measured: 7e-16 of the result); a channel
        # order may swap neighbours whose factors round to the same or the next fp32 value
        return {"rel": 4e-15, "max": 1e-13, "differ": 1e-3}
    return "exact"   # codes, streams and reconstructed weights are exact by definition


# ---------------------------------------------------------------- 64-bit results

def _states(seed, K, n):
    """The n LFSR states from each seed on: Galois, right shift (int64 [n, ...])."""
    mask = torch.zeros_like(seed)
    for k, m in MASKS.items():
        mask = torch.where(K == k, torch.full_like(mask, m), mask)
    x, out = seed.clone(), []
    for _ in range(n):
        out.append(x)
        x = (x >> 1) ^ ((x & 1) * mask)
    return torch.stack(out)


def _decoded(case, s):
    """U(s) q 2^-e of every block in 64 bits, [rows, cols]."""
    rungs = _rungs(case)
    nb = s.seed.numel()
    rob = s.rob.long() if s.rob is not None else torch.zeros(nb, dtype=torch.long, device="cuda")
    out = torch.empty(nb, 8, dtype=torch.float64, device="cuda")
    table = torch.tensor([k for k, _ in rungs], device="cuda")
    for b0 in range(0, nb, 1 << 21):
        sl = slice(b0, min(nb, b0 + (1 << 21)))
        K, P = table[rob[sl]], max(p for _, p in rungs)
        x = _states(s.seed[sl].long(), K, 8 * P).reshape(P, 8, -1)
        u = x - (1 << (K - 1))                                   # [P, 8, blocks]
        acc = (u * s.q[sl, :P].long().t()[:, None, :]).sum(0)    # [8, blocks]
        out[sl] = (acc.double() * torch.exp2(-(K - 1 + s.exp[sl].long()).double())).t()
    return out.reshape(case["rows"], case["cols"])


def _best_errors(W, K, P):
    """The least quantised error of every block over all seeds, in 64 bits."""
    dev, w = W.device, W.double().reshape(-1, 8)
    S = (1 << K) - 1
    k = torch.full((S,), K, device=dev)
    x = _states(torch.arange(1, S + 1, device=dev), k, 8 * P)
    U = ((x - (1 << (K - 1))).double() * 2.0 ** -(K - 1)).reshape(P, 8, S).permute(2, 1, 0)  # [S, 8, P]
    pinv = torch.from_numpy(np.linalg.pinv(U.cpu().numpy(), rcond=2.0 ** -30)).to(dev)       # [S, P, 8]
    best = torch.full((w.shape[0],), math.inf, dtype=torch.float64, device=dev)
    ex = torch.arange(15, -1, -1, device=dev).double()
    for s0 in range(0, S, 64):
        A, B = pinv[s0:s0 + 64], U[s0:s0 + 64]
        t = (A.reshape(-1, 8) @ w.t()).reshape(-1, P, w.shape[0])            # [s, P, blocks]
        e = torch.zeros_like(t[:, 0])
        for v in ex.flip(0):                                                 # the largest that fits
            r = torch.round(t * 2.0 ** v)
            e = torch.where(((r >= -8) & (r <= 7)).all(1), v, e)
        q = torch.round(t * torch.exp2(e)[:, None]).clamp(-8, 7) * torch.exp2(-e)[:, None]
        err = torch.zeros_like(e)
        for i in range(8):
            d = w[:, i] - (B[:, i, :, None] * q).sum(1)
            err += d * d
        best = torch.minimum(best, err.min(0).values)
    return best


def exact(case, seed):
    kind = case["kind"]
    if kind == "search" and ";" not in case["rungs"]:
        (K, P), = _rungs(case)
        if (case["rows"] * case["cols"] << K) * P > 2 ** 32:
            return None
        s = prepare(case, seed)
        return {"seed": None, "exp": None, "q": None, "err": _best_errors(s.W, K, P)}
    if kind == "decode":
        return _decoded(case, prepare(case, seed))
    if kind == "gemv":
        s = prepare(case, seed)
        return s.x.double() @ _decoded(case, s).t()
    if kind == "importance":
        return _exact_importance(case, prepare(case, seed))
    return None


def _exact_importance(case, s):
    dev = "cuda"
    a_attn, a_mlp = (torch.from_numpy(s.layer.gains[n]).to(dev).double().square()
                     for n in ("attn", "mlp"))

    def product(n, v):
        return torch.cat([c.double().square() @ v for c in s.dW[n].split(2048)])

    v_mlp, v_attn = a_mlp.float().double(), a_attn.float().double()
    group = case["heads"] // case["kv"]
    a_o = product("v", v_attn).reshape(case["kv"], 1, -1).expand(-1, group, -1).reshape(-1)
    x, wt = (torch.from_numpy(t).to(dev) for t in np.polynomial.hermite.hermgauss(128))
    g = (2 * product("gate", v_mlp)).sqrt()[:, None] * x
    silu2 = ((g * torch.sigmoid(g)).square() @ wt) / math.sqrt(math.pi)
    a_down = silu2 * product("up", v_mlp)
    rho = sum(c.double().square().sum(0) for c in s.dW["lm_head"].split(2048))
    a = dict(q=a_attn, k=a_attn, v=a_attn, o=a_o, gate=a_mlp, up=a_mlp, down=a_down)
    stats = {}
    for n in frontend.PROJECTIONS:
        w = s.dW[n].abs()
        r = w.shape[0]
        v = torch.sort(w, dim=0).values
        stats[n] = [v[-1].double(), (v[(r - 1) // 2].double() + v[r // 2].double()) / 2]
    return {"a": a, "rho": {"o": rho, "down": rho}, "perm": None, "stats": stats, "outliers": None}
