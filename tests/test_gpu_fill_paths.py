"""The automatic fill (Sec. 3.2) at the sizes where its form changes: 2D in
LDS by one workgroup per field (four or sixteen waves, coupled units), 2D and
3D by ghosts waiting for their corners.  Its values are those of one launch
per level, bit for bit (which the parity tests hold to the oracle)."""
import numpy as np
import pytest

import synth
from synth import CGC, CGC_ES, HGC, LAYER2, DIRICHLET, NEUMANN
from test_gpu_layering import circle, sphere, thin
from test_gpu_parity import gcr  # noqa: F401  (the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
MIXED = 2


def inputs(plan, nf, seed, nan=False):
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = [torch.randn(plan.n_cells, dtype=torch.float64, device="cuda", generator=g) for _ in range(nf)]
    if nan:
        # a NaN of any payload in fluid cells, that of the fill's own mark among them
        at = torch.randint(plan.n_cells, (plan.n_cells // 50,), device="cuda", generator=g)
        bits = torch.tensor([0x7ff85eed0f11e57a, 0x7ff8000000000000, 0x7ff0000000000000],
                            dtype=torch.int64, device="cuda")
        for x in u:
            x.view(torch.int64)[at] = bits[torch.arange(len(at), device="cuda") % 3]
    b = [torch.randn(plan.n_ghost, dtype=torch.float64, device="cuda", generator=g) for _ in range(nf)]
    t = [(torch.rand(plan.n_ghost, device="cuda", generator=g) < 0.5).to(torch.uint8) for _ in range(nf)]
    return u, b, t


def agree(plan, kinds, seed, nan=False):
    u, b, t = inputs(plan, len(kinds), seed, nan)
    want, got = [x.clone() for x in u], [x.clone() for x in u]
    plan.set_schedule(1)
    plan.fill(want, kinds, b, t)
    plan.set_schedule(0)
    plan.fill(got, kinds, b, t)
    torch.cuda.synchronize()
    for f, (x, y) in enumerate(zip(got, want)):
        if nan:   # which of several NaNs comes out of a sum is not the fill's to say
            assert torch.equal(x.isnan(), y.isnan()), f
            x, y = x.nan_to_num(0.0), y.nan_to_num(0.0)
        assert torch.equal(x, y), f
    return got


CASES = {   # about 99 to 1,030 ghosts, 4,080 and 4,110 (the LDS form's most), beyond
    "circle128": (circle(128), HGC), "circle640": (circle(640), HGC), "circle660": (circle(660), HGC),
    "circle2590": (circle(2590), HGC), "circle2630": (circle(2630), HGC), "circle700_l2": (circle(700), HGC | LAYER2),
    "circle_es": (circle(301), CGC_ES), "thin": (thin(2048, 64), CGC), "thin_long": (thin(8192, 64), CGC),
    "sphere24": (sphere(24), HGC), "sphere63": (sphere(63), HGC | LAYER2), "sphere96_es": (sphere(96), CGC_ES),
}


@pytest.mark.parametrize("kinds", [[DIRICHLET], [NEUMANN, MIXED, DIRICHLET], [MIXED] * 8])
@pytest.mark.parametrize("name", sorted(CASES))
def test_fill_agrees_with_levels(gcr, name, kinds):  # noqa: F811
    (grid, shape), scheme = CASES[name]
    plan = gcr.Plan(grid, shape, scheme)
    print(name, plan.n_ghost, plan.n_levels, flush=True)
    agree(plan, kinds, 7)


@pytest.mark.parametrize("name", ["circle128", "circle2630", "sphere63"])
def test_fill_passes_nan_through(gcr, name):  # noqa: F811
    (grid, shape), scheme = CASES[name]
    agree(gcr.Plan(grid, shape, scheme), [MIXED, NEUMANN], 11, nan=True)


def test_fill_coupled_units(gcr):  # noqa: F811
    seen = 0
    for inst in synth.stars64(1):
        if inst.grid.n[0] > 1200:
            continue
        plan = gcr.Plan(inst.grid, inst.shape, HGC)
        if plan.stats()["n_units_coupled"]:
            seen += 1
            agree(plan, [MIXED, DIRICHLET, NEUMANN], 3)
    assert seen


@pytest.mark.parametrize("name", ["sphere63", "circle2630"])
def test_fill_waits_that_give_up(gcr, name):  # noqa: F811
    """A wait bounded to its first poll gives up: the plan's levels are then
    swept again, in this and every later fill."""
    (grid, shape), scheme = CASES[name]
    plan = gcr.Plan(grid, shape, scheme)
    gcr.set_batch_spin(1)
    try:
        first = agree(plan, [DIRICHLET, MIXED], 5)
    finally:
        gcr.set_batch_spin(0)
    again = agree(plan, [DIRICHLET, MIXED], 5)
    assert all(torch.equal(x, y) for x, y in zip(first, again))


@pytest.mark.parametrize("name", ["circle128", "sphere96_es"])
def test_fill_on_two_streams_and_captured(gcr, name):  # noqa: F811
    (grid, shape), scheme = CASES[name]
    plan = gcr.Plan(grid, shape, scheme)
    kinds = [NEUMANN, DIRICHLET]
    want = [agree(plan, kinds, s) for s in (1, 2)]
    sets = [inputs(plan, 2, s) for s in (1, 2)]
    streams = [torch.cuda.Stream() for _ in sets]
    torch.cuda.synchronize()
    for _ in range(20):
        for (u, b, t), st in zip(sets, streams):
            plan.fill(u, kinds, b, t, stream=st)
    torch.cuda.synchronize()
    for (u, _, _), w in zip(sets, want):
        assert all(torch.equal(x, y) for x, y in zip(u, w))
    u, b, t = inputs(plan, 2, 1)
    start = [x.clone() for x in u]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.fill(u, kinds, b, t)
    for _ in range(3):
        for x, s in zip(u, start):
            x.copy_(s)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(u, want[0]))


@pytest.mark.parametrize("kind", [DIRICHLET, NEUMANN])
@pytest.mark.parametrize("name", ["sphere63", "circle2630"])
def test_mark_in_a_field_is_not_waited_for(gcr, name, kind):  # noqa: F811
    """The waiting fill's own mark as an input NaN in every cell: level 1 comes
    out NaN, and the levels behind it do not take that for a value to come (a
    wait for one runs to its bound, half a second)."""
    import time
    (grid, shape), scheme = CASES[name]
    plan = gcr.Plan(grid, shape, scheme)
    u = torch.empty(plan.n_cells, dtype=torch.float64, device="cuda")
    u.view(torch.int64).fill_(0x7ff85eed0f11e57a)
    b = torch.ones(plan.n_ghost, dtype=torch.float64, device="cuda")
    cell = plan.export(("cell",))["cell"].long()

    def timed(f):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        return time.perf_counter() - t
    run = lambda: plan.fill([u], [kind], [b])
    assert min(timed(run) for _ in range(3)) < 0.05
    assert u[cell].isnan().all()
    assert not (u.view(torch.int64)[cell] == 0x7ff85eed0f11e57a).any()
    if plan.dim == 3:
        B = gcr.Batch([grid], [shape], [scheme])
        u.view(torch.int64).fill_(0x7ff85eed0f11e57a)
        run = lambda: B.forward(1, [u], [kind], [b])
        assert min(timed(run) for _ in range(3)) < 0.05
        assert u[cell].isnan().all()
