"""Candidates of the second ghost layer (Sec. 7.1) around spheres and circles,
whose search is narrowed to the walk of each candidate's foot point: the plan
must equal the oracle's, which tests every solid cell near a fluid one."""
import numpy as np
import pytest

import oracle
import synth
from synth import CGC, CGC_ES, HGC, LAYER2
from test_gpu_parity import check_plan, gcr  # noqa: F401  (gcr: the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def grid_of(dim, n, lo, hi, ratio=1.0, uneven=False):
    faces = None
    if ratio != 1.0:
        faces = [synth.stretched_faces(n[a], lo[a], hi[a], ratio + 0.003 * a) for a in range(dim)]
    if uneven:   # widths alternating, wide and narrow, so no axis is monotone
        faces = []
        for a in range(dim):
            w = np.where(np.arange(n[a]) % 3 == a % 3, 1.2, 1.0)
            f = lo[a] + np.concatenate([[0.0], np.cumsum(w)]) * (hi[a] - lo[a]) / w.sum()
            f[-1] = hi[a]
            faces.append(f)
    h = [(hi[a] - lo[a]) / n[a] for a in range(dim)]
    pad = (1,) * (3 - dim)
    return synth.Grid(dim, tuple(n) + pad, tuple(lo) + (0.0,) * (3 - dim), tuple(h) + (1.0,) * (3 - dim),
                      None if faces is None else tuple(faces) + (None,) * (3 - dim))


CASES = {
    "uniform3d_odd": (grid_of(3, (63, 58, 61), (-1, -1, -1), (1, 1, 1)), (0.013, -0.021, 0.008), 0.4),
    "anisotropic3d": (grid_of(3, (90, 40, 56), (-1, -1, -1), (1, 1, 1)), (0.003, 0.017, -0.012), 0.45),
    "stretched3d": (grid_of(3, (72, 70, 66), (-1, -1, -1), (1, 1, 1), 1.03), (0.011, 0.006, -0.004), 0.3),
    "stretched3d_off_centre": (grid_of(3, (64, 64, 64), (-1, -1, -1), (1, 1, 1), 1.02), (0.31, -0.27, 0.2), 0.3),
    "uneven3d": (grid_of(3, (60, 66, 57), (-1, -1, -1), (1, 1, 1), uneven=True), (0.02, 0.01, -0.03), 0.4),
    "uniform2d": (grid_of(2, (201, 187), (-2, -2), (2, 2)), (0.013, 0.004), 0.5),
    "stretched2d": (grid_of(2, (150, 131), (-2, -2), (2, 2), 1.025), (0.4, -0.3), 0.5),
    "uneven2d": (grid_of(2, (120, 133), (-2, -2), (2, 2), uneven=True), (0.05, -0.02), 0.6),
    # the walk's room does not fit beside the body: the whole box is searched
    "near_edge2d": (grid_of(2, (96, 96), (-1, -1), (1, 1)), (0.41, 0.013), 0.5),
}


@pytest.mark.parametrize("scheme", [CGC, CGC_ES, HGC])
@pytest.mark.parametrize("name", sorted(CASES))
def test_second_layer_candidates(gcr, name, scheme):  # noqa: F811
    grid, c, r = CASES[name]
    shape = synth.Shape(synth.SPHERE, tuple(c) + (0.0,) * (3 - len(c)), r)
    op = oracle.OraclePlan(grid, shape, scheme | LAYER2)
    print(name, scheme, op.n_ghost, flush=True)
    gp = gcr.Plan(grid, shape, scheme | LAYER2)
    assert gp.n_interface == op.n_interface
    check_plan(op, gp)
    # a re-plan counts marks in listed chunks only
    moved = synth.Shape(synth.SPHERE, (shape.center[0] - 0.01, shape.center[1] + 0.013) + shape.center[2:], r)
    check_plan(oracle.OraclePlan(grid, moved, scheme | LAYER2), gp.update(moved))
