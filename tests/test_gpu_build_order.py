"""The ghosts of a build put in order by counts that workgroups post to each
other (Sec. 3.1): workgroups of either size, instances that begin and end
within a wave, instances without ghosts at either end and between.  Every plan
against the oracle, and its statistics with its arrays.  Likewise the chunks
of a grid too large for one workgroup's scan, and a move's fresh cells."""
import numpy as np
import pytest

import oracle
import synth
from synth import CGC, CGC_ES, HGC, LAYER2
from test_gpu_layering import check, circle, sphere
from test_gpu_parity import gcr, host  # noqa: F401  (gcr: the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def stats_agree(p, g):
    st, d = p.stats(), p.dim
    a = {k: host(v) for k, v in p.export(("psi", "normal", "r")).items()}
    assert st["n_ghost_fluid_side"] == int((a["psi"] < 0).sum())
    for k in range(d):
        # a displacement over its stencil's length: a few roundings
        al = np.maximum(a["psi"] * np.abs(a["normal"][k]) / (a["r"][k] * g.h[k]), 0.0)
        assert abs(st["max_alpha"][k] - al.max(initial=0.0)) <= 1e-12, k


def away(n):
    """A body far outside its grid."""
    g, s = circle(n)
    return g, synth.Shape(synth.SPHERE, (9.0, 9.0, 0.0), 0.5)


@pytest.mark.parametrize("case", ["tiny", "mixed", "empty", "many"])
def test_batch_order(gcr, case):  # noqa: F811
    if case == "tiny":      # a few ghosts each: several instances in a wave
        b = [(circle(n, 0.4), HGC) for n in (6, 8, 7, 9, 6, 12, 33, 8)]
    elif case == "mixed":
        b = [(circle(n), s) for n, s in ((64, CGC), (300, HGC), (41, CGC_ES), (700, HGC | LAYER2), (64, HGC))]
    elif case == "empty":
        b = [(away(20), HGC), (circle(90), HGC), (away(64), CGC), (away(8), CGC), (circle(16, 0.4), CGC),
             (away(300), HGC)]
    else:                   # more instances than a wave compares at once
        b = [(circle(10 + k % 7, 0.4) if k % 5 else away(9), CGC) for k in range(150)]
    B = gcr.Batch([g for (g, _), _ in b], [s for (_, s), _ in b], [c for _, c in b])
    for p, ((g, s), c) in zip(B.plans, b):
        check(p, oracle.OraclePlan(g, s, c))
        stats_agree(p, g)


def test_large_workgroups(gcr):  # noqa: F811
    """More interface cells than workgroups of 256 are used for."""
    g, s = sphere(168, 0.95)
    op = oracle.OraclePlan(g, s, HGC)
    p = gcr.Plan(g, s, HGC)
    assert p.stats()["n_interface"] > 65536
    check(p, op)
    stats_agree(p, g)


def test_more_instances_than_a_workgroup(gcr):  # noqa: F811
    """Offsets of more instances than the workgroup that finds them has
    threads, the last ones beyond it among several sizes."""
    b = [circle(6 + k % 3, 0.4) if k % 11 else away(9) for k in range(1030)]
    B = gcr.Batch([g for g, _ in b], [s for _, s in b], [CGC] * len(b))
    for k in list(range(5)) + list(range(1015, 1030)):
        check(B.plans[k], oracle.OraclePlan(*b[k], CGC))
    assert [p.n_ghost for p in B.plans[:990:33]] == [B.plans[0].n_ghost] * 30


@pytest.mark.parametrize("n", [322, 340])   # 8,151 chunks and 9,596
def test_chunks_beyond_one_workgroup(gcr, n):  # noqa: F811
    g, s = sphere(n)
    p = gcr.Plan(g, s, HGC)
    tags, cell = (p.export((k,))[k] for k in ("tags", "cell"))
    x = [torch.arange(n, dtype=torch.float64, device="cuda").add(0.5).mul(g.h[a]).add(g.lo[a]).sub(s.center[a])
         for a in range(3)]
    solid = (x[2] ** 2)[:, None, None] + (x[1] ** 2)[None, :, None] + (x[0] ** 2)[None, None, :] <= 0.4 ** 2
    iface = torch.zeros_like(solid)
    for a in range(3):
        d = solid.narrow(a, 0, n - 1) != solid.narrow(a, 1, n - 1)
        iface.narrow(a, 0, n - 1).logical_or_(d)
        iface.narrow(a, 1, n - 1).logical_or_(d)
    t = tags.view(n, n, n)
    assert torch.equal(t > 0, solid)
    assert p.stats()["n_interface"] == int(iface.sum())
    assert not (t.abs() == 2).logical_and(~iface).any()
    assert torch.equal(cell.long().sort()[0], (tags.abs() == 2).nonzero()[:, 0])


@pytest.mark.parametrize("n", [40, 41, 130])   # one workgroup's cells (65,536), a little more, many
def test_fresh_cells_counted_and_listed(gcr, n):  # noqa: F811
    from test_gpu_layering import sphere
    g, s = sphere(n)
    a = gcr.Plan(g, s, HGC)
    b = gcr.Plan(g, synth.Shape(synth.SPHERE, tuple(c - 0.11 for c in s.center), 0.33), HGC)
    ta, tb = (p.export(("tags",))["tags"] for p in (a, b))
    want = ((ta > 0) & ((tb == 0) | (tb == -2))).nonzero()[:, 0]
    unc = int(((ta == 1) & ((tb == 0) | (tb == -2))).sum())
    assert len(want) > 10
    for cap in (len(want) + 5, len(want) // 2, 0):
        counts = torch.full((2,), -1, dtype=torch.int64, device="cuda")
        lst = torch.full((max(cap, 1) + 1,), -7, dtype=torch.int32, device="cuda")
        import ctypes
        e = gcr.lib().gcr_plan_fresh_cells(a._h, b._h, ctypes.c_void_p(counts.data_ptr()),
                                           ctypes.c_void_p(lst.data_ptr()), ctypes.c_int64(cap), None)
        torch.cuda.synchronize()
        assert e == 0 and counts.tolist() == [len(want), unc]
        k = min(cap, len(want))
        assert torch.equal(lst[:k].long(), want[:k]) and (lst[k:] == -7).all()
