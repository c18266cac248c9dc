"""Layering of the dependency graph (Sec. 3.2) at the sizes where its form
changes (ghosts per thread, workgroup size, depth tables, whole GPU) and
around cycles: levels, canonical order and coupled units against the
oracle."""
import numpy as np
import pytest

import oracle
import synth
from synth import CGC, CGC_ES, HGC, LAYER2
from test_gpu_parity import check_plan, gcr, host  # noqa: F401  (gcr: the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(gp, op):
    check_plan(op, gp)
    st = gp.stats()
    assert st["n_units_coupled"] == op.n_units_coupled and st["max_unit"] == op.max_unit
    # the oracle names a unit by number, the plan by its first ghost's position
    got, want = host(gp.export(["unit"])["unit"]), np.full(op.n_ghost, -1)
    for u in range(op.n_units_coupled):
        mem = np.nonzero(op.unit == u)[0]
        want[mem] = mem[np.argmin(op.ghost_cell[mem])]
    assert np.array_equal(got, want), "units"


def circle(n, r=0.5):
    g = synth.Grid(2, (n, n, 1), (-1.0, -1.0, 0.0), (2.0 / n, 2.0 / n, 1.0))
    return g, synth.Shape(synth.SPHERE, (0.3 / n, 0.7 / n, 0.0), r)


def sphere(n, r=0.4):
    g = synth.Grid(3, (n, n, n), (-1.0,) * 3, (2.0 / n,) * 3)
    return g, synth.Shape(synth.SPHERE, (0.3 / n, 0.7 / n, -0.2 / n), r)


def thin(nx, ny):
    g = synth.Grid(2, (nx, ny, 1), (-2.0, -2.0, 0.0), (4.0 / nx, 4.0 / ny, 1.0))
    return g, synth.Shape(synth.SPHERE, (0.001, 0.003, 0.0), 0.7)


# interface cells on either side of 1024, 4096, 8192 and 16384
@pytest.mark.parametrize("scheme", [CGC, HGC])
@pytest.mark.parametrize("n", [40, 256, 260, 1020, 1028, 2050, 4100])
def test_levels_2d(gcr, n, scheme):  # noqa: F811
    g, s = circle(n)
    check(gcr.Plan(g, s, scheme), oracle.OraclePlan(g, s, scheme))


@pytest.mark.parametrize("scheme", [CGC_ES, HGC, HGC | LAYER2])
@pytest.mark.parametrize("n", [24, 32, 64, 90, 128, 160])
def test_levels_3d(gcr, n, scheme):  # noqa: F811
    g, s = sphere(n)
    check(gcr.Plan(g, s, scheme), oracle.OraclePlan(g, s, scheme))


# levels beyond the depth tables (258 and 515), alone and beside shallow ones
@pytest.mark.parametrize("nx", [4096, 8192])
def test_levels_deep(gcr, nx):  # noqa: F811
    g, s = thin(nx, 64)
    op = oracle.OraclePlan(g, s, CGC)
    assert op.n_levels > 256
    check(gcr.Plan(g, s, CGC), op)
    gs = [circle(200), (g, s), sphere(24)]
    B = gcr.Batch([x[0] for x in gs], [x[1] for x in gs], [HGC, CGC, HGC])
    for p, (gg, ss), sch in zip(B.plans, gs, (HGC, CGC, HGC)):
        check(p, oracle.OraclePlan(gg, ss, sch))


# stars whose graphs hold cycles, with up to 79 ghosts behind one
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_levels_cycles(gcr, seed):  # noqa: F811
    insts = [i for i in synth.stars64(seed) if i.grid.n[0] <= 1200]
    ops = [oracle.OraclePlan(i.grid, i.shape, HGC) for i in insts]
    assert sum(o.n_units_coupled for o in ops) > 0
    B = gcr.Batch([i.grid for i in insts], [i.shape for i in insts], [HGC] * len(insts))
    for p, o in zip(B.plans, ops):
        check(p, o)
