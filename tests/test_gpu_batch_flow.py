"""The forward of a batch (Sec. 3.2 fill, Sec. 6 surface values and forces) by
ghosts waiting for their corners (3D) or in LDS (2D), and by chunks of points:
one point, a chunk's edge, none; one to eight fields; instances of one
workgroup and many, without ghosts, with coupled units, beyond LDS; and after a
wait that gave up.  Fields and surface values are those
of each plan's own calls with one launch per level, bit for bit; the force
differs from theirs by the order of its sum."""
import numpy as np
import pytest

import synth
from synth import CGC, CGC_ES, HGC, LAYER2, DIRICHLET, NEUMANN
from test_gpu_parity import gcr  # noqa: F401  (the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
MIXED = 2


def rand(*shape, seed):
    return torch.randn(*shape, dtype=torch.float64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(seed))


def agree(gcr, ns, schemes, kinds, nqs, forces=True):
    insts = [synth.sphere256(seed=k, n=n) for k, n in enumerate(ns)]
    return agree_on(gcr, [i.grid for i in insts], [i.shape for i in insts], schemes, kinds, nqs, forces)


def agree_on(gcr, grids, shapes, schemes, kinds, nqs, forces=True):
    ns, d = grids, grids[0].dim
    B = gcr.Batch(grids, shapes, schemes)
    nf = len(kinds)
    clean = [rand(p.n_cells, seed=10 + f) for p in B.plans for f in range(nf)]
    bcv = [rand(p.n_ghost, seed=50 + f) for p in B.plans for f in range(nf)]
    bct = [(rand(p.n_ghost, seed=90 + f) < 0).to(torch.uint8) for p in B.plans for f in range(nf)]
    S = [p.foot_points()[0] for p in B.plans]
    x = [s[:, torch.arange(q, device="cuda") * 7 % max(s.shape[1], 1)].contiguous()[:d] if s.shape[1] else
         rand(d, q, seed=8) for s, q in zip(S, nqs)]
    n = [rand(d, q, seed=3) for q in nqs]
    w = [rand(q, seed=4).abs() for q in nqs]
    mu, u = 0.7, [c.clone() for c in clean]
    F = torch.full((len(ns), 3), 7.0, dtype=torch.float64, device="cuda")
    val = [torch.empty(q, dtype=torch.float64, device="cuda") for q in nqs for _ in range(nf)]
    grad = [torch.empty((d, q), dtype=torch.float64, device="cuda") for q in nqs for _ in range(nf)]
    for _ in range(2):   # every value again from the clean fields
        for a, c in zip(u, clean):
            a.copy_(c)
        if forces:
            B.forward(nf, u, kinds, bcv, bct, nq=nqs, xq=x, nrm=n, wq=w, p_field=nf - 1, u_first=0,
                      mu=mu, F=F, sval=val, sgrad=grad)
        else:
            B.forward(nf, u, kinds, bcv, bct)
    B.status()
    for i, p in enumerate(B.plans):
        s = slice(i * nf, (i + 1) * nf)
        want = [c.clone() for c in clean[s]]
        p.set_schedule(1)
        p.fill(want, kinds, bcv[s], bct[s])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(u[s], want)), i
        p.set_schedule(0)
        if not forces:
            continue
        if nqs[i] == 0:
            assert (F[i] == 0).all()
            continue
        v, g, _ = p.surface(x[i], want)
        if p.n_ghost == 0:
            assert v.isnan().all() and all(a.isnan().all() for a in val[s] + grad[s])
            continue
        assert all(torch.equal(a, b) for a, b in zip(val[s], v)), i
        assert all(torch.equal(a, b) for a, b in zip(grad[s], g)), i
        # each point's share, in the terms of the sum; 40 roundings on a term
        # and the sum's own bound the difference
        if nf >= d + 1:
            G = g[:d]
            t = -w[i] * v[nf - 1] * n[i] + mu * w[i] * (torch.einsum("caq,aq->cq", G, n[i])
                                                         + torch.einsum("caq,cq->aq", G, n[i]))
            mag = (w[i] * v[nf - 1] * n[i]).abs() + mu * w[i] * (
                torch.einsum("caq,aq->cq", G.abs(), n[i].abs()) + torch.einsum("caq,cq->aq", G.abs(), n[i].abs()))
            assert (F[i, d:] == 0).all()
            assert ((F[i, :d] - t.sum(1)).abs() <= (40 + nqs[i]) * 2.0 ** -53 * mag.sum(1)).all(), i
    return B


@pytest.mark.parametrize("kinds", [[DIRICHLET], [NEUMANN, DIRICHLET, MIXED, DIRICHLET], [MIXED] * 8])
def test_batch_waiting_fill(gcr, kinds):  # noqa: F811
    agree(gcr, [16, 64, 33, 90], [HGC, CGC_ES, CGC, HGC | LAYER2], kinds, [1, 256, 257, 0])


def test_batch_waiting_fill_one_instance(gcr):  # noqa: F811
    agree(gcr, [120], [HGC], [DIRICHLET, NEUMANN, DIRICHLET, MIXED], [1000])
    agree(gcr, [120], [HGC], [DIRICHLET, NEUMANN], [0], forces=False)


def test_batch_waiting_fill_many_instances(gcr):  # noqa: F811
    ns = [int(n) for n in np.random.default_rng(3).integers(16, 40, 70)]
    agree(gcr, ns, [HGC] * 70, [DIRICHLET] * 4, [k % 5 * 64 for k in range(70)])


def test_batch_wait_that_gives_up_is_swept_again(gcr):  # noqa: F811
    gcr.set_batch_spin(1)   # no polls: every wait gives up at once
    try:
        agree(gcr, [64, 33], [HGC, CGC], [DIRICHLET, MIXED, NEUMANN, DIRICHLET], [300, 5])
    finally:
        gcr.set_batch_spin(0)

def test_batch_in_lds(gcr):  # noqa: F811
    from test_gpu_layering import circle
    b = [circle(n) for n in (128, 40, 700, 330, 128)]
    b[3] = (b[3][0], synth.Shape(synth.SPHERE, (9.0, 9.0, 0.0), 0.5))   # no ghosts
    g, s = [x for x, _ in b], [y for _, y in b]
    for kinds in ([DIRICHLET], [NEUMANN, MIXED, DIRICHLET], [MIXED] * 8):
        B = agree_on(gcr, g, s, [HGC, CGC, HGC | LAYER2, CGC, CGC_ES], kinds, [1, 256, 257, 300, 0])
        assert B.tiled() == 1 and B.shape() == (0, 0)
    agree_on(gcr, g[:1], s[:1], [HGC], [NEUMANN, DIRICHLET], [0], forces=False)


def test_batch_in_lds_coupled_units(gcr):  # noqa: F811
    insts = [i for i in synth.stars64(1) if i.grid.n[0] <= 1200]
    B = agree_on(gcr, [i.grid for i in insts], [i.shape for i in insts], [HGC] * len(insts),
                 [MIXED, DIRICHLET, NEUMANN], [64] * len(insts))
    assert sum(p.stats()["n_units_coupled"] for p in B.plans) and B.shape() == (0, 0)


def test_batch_beyond_lds(gcr):  # noqa: F811
    from test_gpu_layering import circle
    b = [circle(2630), circle(64)]
    B = agree_on(gcr, [g for g, _ in b], [s for _, s in b], [HGC] * 2, [MIXED, DIRICHLET, NEUMANN], [300, 5])
    assert B.shape() != (0, 0)


def test_anchors_at_the_edges_of_their_workgroups(gcr):  # noqa: F811
    """Points of an instance: none, one, and around the 4 (3D) and 32 (2D) that
    an anchor workgroup takes, instances without any between."""
    nqs = [0, 1, 3, 4, 5, 0, 255, 256, 257, 0, 0, 9]
    agree(gcr, [20 + k for k in range(12)], [HGC] * 12, [DIRICHLET] * 4, nqs)
    from test_gpu_layering import circle
    b = [circle(24 + 3 * k) for k in range(12)]
    nqs = [0, 1, 31, 32, 33, 0, 255, 256, 257, 0, 64, 0]
    agree_on(gcr, [g for g, _ in b], [s for _, s in b], [HGC] * 12, [DIRICHLET, NEUMANN, MIXED], nqs)
