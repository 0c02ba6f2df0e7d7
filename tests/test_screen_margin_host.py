"""The margin of the search's quadratic-form screen, restated in numpy: with both operands rounded
to fp16, the form plus the seed's margin must reach the exact form less the block's margin, so that
a seed whose least-squares residual is at most the best error always passes."""
import os
import re

import numpy as np
import pytest

I, J = np.triu_indices(8)
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2609_38477_amd", "csrc")


def _source(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def constant(name):
    """A constexpr of the kernels' header."""
    return float(re.search(r"constexpr \w+ %s = ([0-9.]+)f?;" % name,
                           _source("seedq_internal.h")).group(1))


# the kernels' own constants
SCALE, MARGIN_B, MARGIN_A = (constant(n) for n in ("kOperandScale", "kMarginScale",
                                                   "kMarginSeedScale"))
_c = [float(x) for x in re.search(
    r"constexpr float c = P == 1 \? ([0-9.]+)f : P == 2 \? ([0-9.]+)f : P == 3 \? ([0-9.]+)f : ([0-9.]+)f;",
    _source("seedq_search_mfma.hip")).groups()]
C = {1: _c[0], 2: _c[1], 3: _c[2], 4: _c[3], 5: _c[3]}


@pytest.mark.parametrize("P", [1, 2, 3, 4, 5])
def test_block_constant_is_the_largest_over_ranks(P):
    # sqrt(r - r^2/8), the Frobenius norm of Pi - (r/8) I for a projector of rank r
    want = max(np.sqrt(r - r * r / 8) for r in range(1, P + 1))
    assert want <= C[P] < want * (1 + 1e-4)


def _blocks(rng):
    w = rng.normal(0, 0.02, (160, 8))
    w[20:60] = rng.standard_t(3, (40, 8))
    w[60:80, 1:] *= 1e-4                      # one dominant weight
    w[80:90] = 1.0
    w[90:98] = np.eye(8)
    w[98:120, rng.integers(0, 8, 22)] = 0.0
    w[120:140] *= 1e-12
    w = w.astype(np.float32)
    w = w[np.abs(w).max(1) > 0]
    ex = np.floor(np.log2(np.abs(w).max(1).astype(np.float64)))
    return w.astype(np.float64) * 2.0 ** -ex[:, None]


@pytest.mark.parametrize("P", [1, 2, 3, 4, 5])
def test_form_with_margins_bounds_the_exact_form(oq, P):
    rng = np.random.default_rng(70 + P)
    ws = _blocks(rng)
    seeds = np.concatenate([[0xFE], rng.integers(1, 1 << 11, 300)])   # 0xFE: rank deficient at P = 4
    U = np.stack([oq.basis(11, P, int(s)) for s in seeds])
    u, sv, _ = np.linalg.svd(U, full_matrices=False)
    u = u * (sv > 2.0 ** -30 * sv[:, :1])[:, None, :]
    Pi = u @ u.transpose(0, 2, 1)
    ww = (ws ** 2).sum(1).astype(np.float32).astype(np.float64)
    a = (SCALE * Pi[:, I, J]).astype(np.float16).astype(np.float64)
    E = np.zeros_like(Pi)
    E[:, I, J] = E[:, J, I] = a - SCALE * Pi[:, I, J]
    eps = np.sqrt(np.sqrt(((E @ E) ** 2).sum((1, 2)))) / SCALE
    margin = (MARGIN_A * eps * (1 + 2.0 ** -9) + 2.0 ** -24).astype(np.float16).astype(np.float64)
    z32 = (np.where(I == J, 1.0, 2.0) * ws[:, I] * ws[:, J] * SCALE).astype(np.float32)
    b = z32.astype(np.float16).astype(np.float64)
    d = b - z32
    f2 = (d ** 2 * np.where(I == J, 1.0, 0.5)).sum(1)
    tr = d[:, I == J].sum(1)
    base = (ww * (1 - 2.0 ** -15) * SCALE ** 2
            - SCALE * (C[P] * (1 + 2.0 ** -10) * np.sqrt(f2) + np.maximum(0, -P / 8 * tr)))
    form = a @ b.T + np.outer(margin, (MARGIN_B * ww).astype(np.float16).astype(np.float64))
    exact = np.einsum("bi,sij,bj->sb", ws, Pi, ws) * SCALE ** 2
    # passes whenever exact form >= ww - best: form - base >= exact - ww, with the
    # fp32 evaluation's share (2^-17 of ww) still to come
    slack = (form - base) - (exact - ww * SCALE ** 2)
    assert np.all(slack >= 2.0 ** -17 * ww * SCALE ** 2)
    # and the margin is the smaller one: below half of sqrt(P) 2^-10 on average
    assert np.mean(slack / (ww * SCALE ** 2)) < 0.5 * np.sqrt(P) * 2.0 ** -10
