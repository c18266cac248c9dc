"""The automatic adjoints (Sec. 3.2, Sec. 6 transposed) where their form
changes: the fill's by ghosts waiting for their readers, with coupled units,
one to eight fields, and after a wait that gave up; the surface's with many
points to an anchor, and the force's without cotangent arrays.  The fill's
values are those of one launch per level, bit for bit (which the parity tests
hold to the oracle); the force's those of the surface adjoint on the
cotangents it stands for, bit for bit."""
import pytest

import synth
from synth import HGC
from test_gpu_fill_paths import CASES, MIXED, circle
from synth import DIRICHLET, NEUMANN
from test_gpu_parity import gcr  # noqa: F401  (the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rand(*shape, seed):
    return torch.randn(*shape, dtype=torch.float64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(seed))


def agree(plan, kinds, seed):
    nf = len(kinds)
    lam0 = rand(nf, plan.n_cells, seed=seed)
    t = [(rand(plan.n_ghost, seed=seed + 1 + f) < 0).to(torch.uint8) for f in range(nf)]
    out = []
    for schedule in (1, 2, 0):
        plan.set_schedule(schedule)
        lam = [x.clone() for x in lam0]
        bc = [torch.empty(plan.n_ghost, dtype=torch.float64, device="cuda") for _ in kinds]
        plan.fill_adjoint(lam, kinds, bc, t)
        out.append(lam + bc)
    torch.cuda.synchronize()
    for got in out[1:]:
        for f, (x, y) in enumerate(zip(got, out[0])):
            assert torch.equal(x, y), f


@pytest.mark.parametrize("kinds", [[NEUMANN], [NEUMANN, MIXED], [NEUMANN, MIXED, DIRICHLET], [MIXED] * 5,
                                   [MIXED] * 8])
@pytest.mark.parametrize("name", ["circle128", "circle640", "circle700_l2", "thin", "sphere24", "sphere63",
                                  "sphere96_es"])
def test_fill_adjoint_agrees_with_levels(gcr, name, kinds):  # noqa: F811
    (grid, shape), scheme = CASES[name]
    agree(gcr.Plan(grid, shape, scheme), kinds, 5)


def test_fill_adjoint_coupled_units(gcr):  # noqa: F811
    seen = 0
    for inst in synth.stars64(1):
        if inst.grid.n[0] > 1200:
            continue
        plan = gcr.Plan(inst.grid, inst.shape, HGC)
        if plan.stats()["n_units_coupled"]:
            seen += 1
            agree(plan, [MIXED, DIRICHLET, NEUMANN], 3)
    assert seen


def test_fill_adjoint_after_a_wait_that_gave_up(gcr):  # noqa: F811
    (grid, shape), scheme = CASES["sphere63"]
    gcr.set_batch_spin(1)   # no polls: every wait gives up at once
    try:
        agree(gcr.Plan(grid, shape, scheme), [DIRICHLET, MIXED], 9)
    finally:
        gcr.set_batch_spin(0)


@pytest.mark.parametrize("nq", [1, 63, 257, 5000])
@pytest.mark.parametrize("name", ["circle128", "sphere24"])
def test_force_adjoint_is_the_surface_adjoint_of_its_cotangents(gcr, name, nq):  # noqa: F811
    (grid, shape), scheme = CASES[name]
    plan = gcr.Plan(grid, shape, scheme)
    d = plan.dim
    # points about the body: up to hundreds of them to an anchor
    S = plan.foot_points()[0][:, torch.arange(nq, device="cuda") % plan.n_ghost % 17].contiguous()
    x = S + 1e-3 * rand(d, nq, seed=1) / grid.n[0]
    n, w, gF, mu = rand(d, nq, seed=2), rand(nq, seed=3), rand(d, seed=4), 0.7
    got = torch.zeros(1 + d, plan.n_cells, dtype=torch.float64, device="cuda")
    plan.forces_adjoint(x, n, w, mu, gF, got[0], list(got[1:]))
    gn = gF[0] * n[0]
    for a in range(1, d):
        gn = gn + gF[a] * n[a]
    gval = torch.zeros(1 + d, nq, dtype=torch.float64, device="cuda")
    ggrad = torch.zeros(1 + d, d, nq, dtype=torch.float64, device="cuda")
    gval[0] = -w * gn
    for i in range(d):
        for j in range(d):
            ggrad[1 + i, j] = mu * w * (gF[i] * n[j] + gF[j] * n[i])
    want = torch.zeros_like(got)
    plan.surface_adjoint(x, gval, ggrad, list(want))
    torch.cuda.synchronize()
    assert want.abs().sum() > 0
    assert torch.equal(got, want)
    # each point by itself, in ascending order, summed in double: the same to
    # the rounding of a sum of nq terms
    if nq <= 63:
        one = torch.zeros_like(got)
        for q in range(nq):
            plan.surface_adjoint(x[:, q:q + 1].contiguous(), gval[:, q:q + 1].contiguous(),
                                 ggrad[:, :, q:q + 1].contiguous(), list(one))
        mag = torch.zeros_like(got)
        for q in range(nq):
            t = torch.zeros_like(got)
            plan.surface_adjoint(x[:, q:q + 1].contiguous(), gval[:, q:q + 1].contiguous(),
                                 ggrad[:, :, q:q + 1].contiguous(), list(t))
            mag += t.abs()
        assert ((got - one).abs() <= 4 * (nq + 16) * 2.0 ** -52 * mag).all()


def test_one_array_for_several_fields(gcr):  # noqa: F811
    """The fields' sums then follow each other in that array."""
    (grid, shape), scheme = CASES["sphere24"]
    plan = gcr.Plan(grid, shape, scheme)
    x = plan.foot_points()[0]
    gval, start = rand(5, x.shape[1], seed=1), rand(plan.n_cells, seed=2)
    got, want = start.clone(), start.clone()
    plan.surface_adjoint(x, gval, None, [got] * 5)
    for f in range(5):
        plan.surface_adjoint(x, gval[f:f + 1].contiguous(), None, [want])
    torch.cuda.synchronize()
    assert not torch.equal(want, start)
    assert torch.equal(got, want)


@pytest.mark.parametrize("body", ["star", "harmonic"])
def test_fill_adjoint_with_units_after_a_wait_that_gave_up(gcr, body):  # noqa: F811
    """Waits that give up at once in a plan with coupled units: the same
    values, then and from the next call on, which takes no longer than that of
    a plan where none gave up (a second sweep by one workgroup, kept up for the
    plan's life, took five times as long)."""
    import time

    from test_gpu_second_layering import harmonic
    if body == "star":
        inst = next(i for i in synth.stars64(1) if i.grid.n[0] <= 1200 and
                    gcr.Plan(i.grid, i.shape, HGC).stats()["n_units_coupled"])
        make = lambda: gcr.Plan(inst.grid, inst.shape, HGC)
    else:
        make = lambda: gcr.Plan(*harmonic(128, 0.15), HGC)
    plan, other = make(), make()
    kinds = [DIRICHLET, MIXED, NEUMANN, MIXED]
    gcr.set_batch_spin(1)
    try:
        agree(plan, kinds, 9)
    finally:
        gcr.set_batch_spin(0)
    agree(plan, kinds, 9)

    def best(p):
        lam = [rand(p.n_cells, seed=f) for f in range(4)]
        bc = [torch.empty(p.n_ghost, dtype=torch.float64, device="cuda") for _ in kinds]
        t = [torch.zeros(p.n_ghost, dtype=torch.uint8, device="cuda")] * 4
        p.fill_adjoint(lam, kinds, bc, t)
        times = []
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                p.fill_adjoint(lam, kinds, bc, t)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        return min(times)
    other.set_schedule(0)
    assert best(plan) < 2 * best(other)


@pytest.mark.parametrize("name", ["circle128", "sphere24"])
def test_points_of_one_anchor_in_ascending_order(gcr, name):  # noqa: F811
    """Points at one anchor, few and many (33 on, ranked first): its seeds are
    the points' own, summed in ascending order, bit for bit."""
    (grid, shape), scheme = CASES[name]
    plan = gcr.Plan(grid, shape, scheme)
    d = plan.dim
    sizes = [1, 2, 31, 32, 33, 64, 65, 256, 257, 700]
    S = plan.foot_points()[0]
    x = S[:, 5:6] + 1e-6 * rand(d, sizes[-1], seed=1) / grid.n[0]
    gval, ggrad = rand(2, sizes[-1], seed=2), rand(2, d, sizes[-1], seed=3)
    cut = lambda a, i, j: a[..., i:j].contiguous()
    total = torch.zeros(2, plan.n_cells, dtype=torch.float64, device="cuda")
    for q in range(sizes[-1]):
        one = torch.zeros_like(total)
        plan.surface_adjoint(cut(x, q, q + 1), cut(gval, q, q + 1), cut(ggrad, q, q + 1), list(one))
        total += one
        if q + 1 in sizes:
            got = torch.zeros_like(total)
            plan.surface_adjoint(cut(x, 0, q + 1), cut(gval, 0, q + 1), cut(ggrad, 0, q + 1), list(got))
            torch.cuda.synchronize()
            assert got.abs().sum() > 0 and torch.equal(got, total), q + 1


def test_many_points_of_one_anchor_cost_their_number(gcr):  # noqa: F811
    """Eight times the points at an anchor: not sixty-four times the time."""
    import time
    (grid, shape), scheme = CASES["sphere24"]
    plan = gcr.Plan(grid, shape, scheme)
    lam = [torch.zeros(plan.n_cells, dtype=torch.float64, device="cuda")]

    def best(nq):
        x = (plan.foot_points()[0][:, 5:6] + 1e-6 * rand(3, nq, seed=1) / 24).contiguous()
        gval, times = rand(1, nq, seed=2), []
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            plan.surface_adjoint(x, gval, None, lam)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
        return min(times[1:])
    assert best(4096) < 24 * best(512)


@pytest.mark.parametrize("n", [24, 128, 300])
def test_fill_adjoint_of_few_ghosts(gcr, n):  # noqa: F811
    # the last fields that one workgroup sweeps, the first that wait, and one
    plan = gcr.Plan(*circle(n), HGC)
    most = 512 // plan.n_ghost
    for nf in {1, min(most, 8), min(most + 1, 8)}:
        agree(plan, ([MIXED, DIRICHLET, NEUMANN] * 3)[:nf], n)
