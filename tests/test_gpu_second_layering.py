"""Batches and plans layered twice (Sec. 3.2), because the first form leaves a
graph: the instances it finished keep their levels, order, units and
statistics, those it left are the oracle's too, and both fill as one launch
per level does."""
import numpy as np
import pytest

import oracle
import synth
from synth import CGC, HGC, LAYER2
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
    """A graph of more levels than the first form's table, before and behind
    instances with many cycles, few, and none."""
    b = [(wavy(800), HGC | LAYER2), (circle(200), HGC),
         *[((i.grid, i.shape), HGC) for i in synth.stars64(1) if i.grid.n[0] <= 1200][:4]]
    b.insert(0 if first else len(b), (thin(4096, 64), CGC))
    ops = [oracle.OraclePlan(g, s, c) for (g, s), c in b]
    assert max(o.n_levels for o in ops) > 256 and max(o.n_units_coupled for o in ops) >= 80
    B = gcr.Batch([g for (g, _), _ in b], [s for (_, s), _ in b], [c for _, c in b])
    for p, o, ((g, s), c) in zip(B.plans, ops, b):
        check(p, o)
        stats_agree(p, g)
        agree(p, [MIXED], 3)
