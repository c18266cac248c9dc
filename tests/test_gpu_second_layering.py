"""Batches and plans layered twice (Sec. 3.2), because the first form leaves a
graph: the instances it finished keep their levels, order, units and
statistics, those it left are the oracle's too, and both fill as one launch
per level does."""
import time

import numpy as np
import pytest

import oracle
import synth
from synth import CGC, CGC_ES, HGC, LAYER2
from synth.workloads import SplitMix64, sh_shape
from test_gpu_build_order import stats_agree
from test_gpu_fill_paths import MIXED, agree
from test_gpu_layering import check, circle, thin
from test_gpu_parity import gcr  # noqa: F401  (the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def wavy(n, k=40, amp=0.03):
    """A star of k waves: with a second layer, two coupled units to a trough."""
    g = synth.Grid(2, (n, n, 1), (-1.0, -1.0, 0.0), (2.0 / n, 2.0 / n, 1.0))
    coef = np.zeros((k + 1, 2))
    coef[k, 0] = amp
    return g, synth.Shape(synth.STAR2D, (0.3 / n, 0.7 / n, 0.0), 0.7, coef.ravel(), k + 1)


@pytest.mark.parametrize("first", [True, False])
def test_batch_keeps_what_the_first_layering_finished(gcr, first):  # noqa: F811
    """The deepest graph, before and behind instances with many cycles, few,
    and none."""
    b = [(wavy(800), HGC | LAYER2), (circle(200), HGC),
         *[((i.grid, i.shape), HGC) for i in synth.stars64(1) if i.grid.n[0] <= 1200][:4]]
    b.insert(0 if first else len(b), (thin(10000, 64), CGC))
    ops = [oracle.OraclePlan(g, s, c) for (g, s), c in b]
    assert max(o.n_levels for o in ops) == 629 and max(o.n_units_coupled for o in ops) >= 80
    B = gcr.Batch([g for (g, _), _ in b], [s for (_, s), _ in b], [c for _, c in b])
    for p, o, ((g, s), c) in zip(B.plans, ops, b):
        check(p, o)
        stats_agree(p, g)
        agree(p, [MIXED], 3)


def harmonic(n, amp, seed=0):
    """A spherical-harmonic body, with coupled units in its folds at amp 0.1
    and above, without at 0.04."""
    g = synth.Grid(3, (n, n, n), (-1.0,) * 3, (2.0 / n,) * 3)
    return g, sh_shape(SplitMix64(seed), (0.3 / n, 0.7 / n, -0.2 / n), 0.3, 4, amp)


# whole GPU first: 2,006, 4,477 and 8,684 interface cells, then one workgroup
# pulling; 18,565, then one pushing
@pytest.mark.parametrize("scheme", [HGC, CGC_ES])
@pytest.mark.parametrize("n,amp", [(64, 0.1), (96, 0.1), (128, 0.15), (192, 0.12)])
def test_plan_with_cycles_3d(gcr, n, amp, scheme):  # noqa: F811
    g, s = harmonic(n, amp)
    op = oracle.OraclePlan(g, s, scheme)
    assert op.n_units_coupled > 0
    p = gcr.Plan(g, s, scheme)
    check(p, op)
    stats_agree(p, g)
    agree(p, [MIXED], 3)
    # a re-plan takes the same way
    p.update(harmonic(n, 0.04)[1])
    p.update(s)
    check(p, op)


# in 2D only when asked for: a cycle, and more levels than the whole GPU's
# table (129 to 629)
@pytest.mark.parametrize("body,scheme", [(wavy(800), HGC | LAYER2), (thin(2048, 64), CGC), (thin(8192, 64), CGC),
                                         (thin(10000, 64), CGC)])
def test_plan_left_by_the_whole_gpu_2d(gcr, body, scheme):  # noqa: F811
    op = oracle.OraclePlan(*body, scheme)
    assert op.n_units_coupled or op.n_levels > 128
    gcr.set_wide_layering(1)
    try:
        p = gcr.Plan(*body, scheme)
    finally:
        gcr.set_wide_layering(0)
    check(p, op)
    stats_agree(p, body[0])
    agree(p, [MIXED, MIXED], 3)


def test_cycles_cost_no_wait(gcr):  # noqa: F811
    """A body with cycles builds in a small multiple of the time of one
    without, of the same size (a wait for them took fourteen times as long)."""
    def build(body):
        times = []
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            gcr.Plan(*body, HGC)
            times.append(time.perf_counter() - t)
        return min(times)
    assert build(harmonic(128, 0.15)) < 5 * build(harmonic(128, 0.04))


# alone: 213 levels, 256 and 257 (the most that every wave ranks), 629
@pytest.mark.parametrize("nx,ny", [(1300, 8), (4064, 64), (4080, 64), (10000, 64)])
def test_deep_plan(gcr, nx, ny):  # noqa: F811
    body = thin(nx, ny)
    check(gcr.Plan(*body, CGC), oracle.OraclePlan(*body, CGC))
