"""Fixed costs of the host calls, as ratios of calls of the same library measured side by side (the
best of many repetitions each), and the results where the planner's short way is taken."""
import time

import numpy as np
import pytest

from test_decoder_host import sq  # noqa: F401

RUNGS, DAMAGE = [(12, 2), (16, 3), (20, 4)], [4.0, 1.0, 0.25]


def _best(*calls, n=300):
    """The shortest time of each call, the calls taken in turn."""
    out = [1e9] * len(calls)
    for _ in range(n):
        for i, f in enumerate(calls):
            t = time.perf_counter()
            f()
            out[i] = min(out[i], time.perf_counter() - t)
    return out


def _plan(sq, rows, G, rho=False, rungs=RUNGS, damage=DAMAGE, bpw=4.0, f=0.06):
    rng = np.random.default_rng(rows + G)
    a = np.exp(rng.normal(0, 1, 8 * G)).astype(np.float32)
    r = np.exp(rng.normal(0, 0.5, rows)).astype(np.float32) if rho else None
    desc, keep = sq._schedule_desc(rows, 8 * G, rungs, damage, bpw, a, r, f)
    rep, out = sq.ScheduleReport(), np.empty(rows * G, np.uint8)
    sq.seedq_plan_schedule(desc, out, rep)

    def plan():
        sq.seedq_plan_schedule(desc, out, rep)

    def derive(T=None):
        sq.seedq_derive_schedule(desc, rep.lambda_, rep.floor_q, rep.tie_count if T is None else T,
                                 out)
    return plan, derive, rep, keep


@pytest.mark.parametrize("rows,G", [(8, 16), (256, 32)])
def test_a_small_plan_costs_little_more_than_its_derivation(sq, rows, G):  # noqa: F811
    # measured 1.0 and 1.1 times; 4 times with a histogram and a bisection over bit patterns
    plan, derive, _, keep = _plan(sq, rows, G)
    p, d = _best(plan, derive)
    assert p < 2.5 * d, (p, d)
    del keep


def test_row_factors_of_a_small_tensor_cost_nothing_fixed(sq):  # noqa: F811
    # measured 1.0 times; 2.1 times and more when the number of cores is asked for
    _, plain, _, k0 = _plan(sq, 1, 1, bpw=3.0)
    _, rows, _, k1 = _plan(sq, 1, 1, rho=True, bpw=3.0)
    a, b = _best(plain, rows)
    assert b < 1.7 * a, (a, b)
    del k0, k1


def test_deriving_a_tie_pass_is_a_copy_of_rows(sq):  # noqa: F811
    # the tied blocks of whole rows are part of the row that is copied: measured 1.0
    # times the call without a tie; 9 times when every block is looked at
    _, derive, rep, keep = _plan(sq, 4096, 1792)
    assert rep.tie_count > 100000
    a, b = _best(lambda: derive(0), derive, n=20)
    assert b < 4 * a, (a, b)
    del keep


def test_a_rule_of_two_nodes_costs_little_more_than_of_one(sq):  # noqa: F811
    # measured 1.4 times; 1.9 times with the recurrence's factors on the heap each step
    one, two = _best(lambda: sq.seedq_gauss_hermite(1), lambda: sq.seedq_gauss_hermite(2))
    assert two < 1.65 * one, (one, two)


@pytest.mark.parametrize("rows,G,rho", [(1, 1, False), (3, 4096, False), (3, 4097, False),
                                        (17, 240, True), (17, 242, True)])
@pytest.mark.parametrize("f", [0.0, 0.06, 0.999])
def test_one_rung_reports_the_floor(sq, rows, G, rho, f):  # noqa: F811
    # a single rung's plan takes one rank of the importances, on both sides of the
    # count up to which they are kept in a list
    plan, _, rep, (_, _, a, r) = _plan(sq, rows, G, rho, [(16, 3)], None, f=f)
    abar = a.astype(np.float64).reshape(-1, 8)
    s = abar[:, 0].copy()
    for j in range(1, 8):
        s = s + abar[:, j]
    s = s / 8.0
    s = s / (np.cumsum(s)[-1] / G)
    imp = np.tile(s, rows)
    if rho:
        r = r.astype(np.float64)
        imp = np.outer(r / (np.cumsum(r)[-1] / rows), s).ravel()
    k = min(max(int(np.ceil(rows * G * f)) - 1, 0), rows * G - 1)
    assert rep.floor_q == np.sort(imp)[k]
