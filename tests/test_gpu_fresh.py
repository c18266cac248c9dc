"""GPU parity of gcr_plan_fresh_cells: the cells a moved body exposes (Sec.
7.1), bit-exact against the oracle's list and counts."""
import numpy as np
import pytest

import oracle
import synth
from synth import CGC, HGC, LAYER2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_10165_amd as g
    g.lib()
    return g


def moved(shape, v):
    return synth.Shape(shape.kind, tuple(c + d for c, d in zip(shape.center, v)), shape.r0)


def check(gcr, inst, flag, v, cap=None):
    a_o = oracle.OraclePlan(inst.grid, inst.shape, flag)
    b_o = oracle.OraclePlan(inst.grid, moved(inst.shape, v), flag)
    want, unc = a_o.fresh_cells(b_o)
    a = gcr.Plan(inst.grid, inst.shape, flag)
    b = gcr.Plan(inst.grid, moved(inst.shape, v), flag)
    lst, counts = a.fresh_cells(b, cap=cap)
    torch.cuda.synchronize()
    c = counts.cpu().numpy()
    assert c[0] == len(want) and c[1] == unc, (c, len(want), unc)
    k = min(len(want), lst.numel())
    assert np.array_equal(lst[:k].cpu().numpy().astype(np.int64), want[:k])
    return len(want), unc


@pytest.mark.parametrize("scheme", [CGC, HGC])
@pytest.mark.parametrize("layer2", [False, True])
def test_fresh_cells_circle(gcr, scheme, layer2):
    inst = synth.circle128(seed=3)
    h = inst.grid.h[0]
    for v in ((0.7 * h, 0.2 * h, 0.0), (-1.3 * h, 0.9 * h, 0.0), (0.05 * h, -1.9 * h, 0.0)):
        nf, unc = check(gcr, inst, scheme | (LAYER2 if layer2 else 0), v)
        assert nf > 0
        if layer2 and np.hypot(v[0], v[1]) < 1.5 * h:
            assert unc == 0


def test_fresh_cells_sphere256_full_size(gcr):
    inst = synth.sphere256(seed=0)
    h = inst.grid.h[0]
    nf, unc = check(gcr, inst, HGC | LAYER2, (0.6 * h, -0.5 * h, 0.8 * h))
    assert nf > 1000 and unc == 0
    nf, unc = check(gcr, inst, CGC, (1.2 * h, 0.3 * h, -0.4 * h))
    assert unc > 0


def test_fresh_cells_stretched_and_truncated(gcr):
    inst = synth.circle_stretched(seed=1)
    check(gcr, inst, HGC | LAYER2, (0.01, -0.02, 0.0))
    nf, _ = check(gcr, inst, CGC, (0.03, 0.01, 0.0), cap=7)   # list cut at 7, counts whole
    assert nf > 7


def test_fresh_cells_refuses_other_grids(gcr):
    a_inst = synth.circle128(seed=0)
    big = synth.Grid(2, (130, 128, 1), a_inst.grid.lo, a_inst.grid.h)
    a = gcr.Plan(a_inst.grid, a_inst.shape, HGC)
    b = gcr.Plan(big, a_inst.shape, HGC)
    with pytest.raises(gcr.GcrError):
        a.fresh_cells(b)


def test_fresh_cells_on_two_streams_and_captured(gcr):
    """Calls that share the scratch of `after` overlap on two streams, then are
    replayed from a graph."""
    inst = synth.sphere256(seed=1, n=160)
    h = inst.grid.h[0]
    shape = moved(inst.shape, (0.6 * h, -0.5 * h, 0.8 * h))
    want, unc = oracle.OraclePlan(inst.grid, inst.shape, HGC).fresh_cells(
        oracle.OraclePlan(inst.grid, shape, HGC))
    a, b = gcr.Plan(inst.grid, inst.shape, HGC), gcr.Plan(inst.grid, shape, HGC)
    n = len(want)
    counts = torch.zeros(40, 2, dtype=torch.int64, device="cuda")
    lst = torch.zeros(40, n, dtype=torch.int32, device="cuda")
    streams = [torch.cuda.Stream() for _ in range(2)]
    call = lambda k, st: gcr.lib().gcr_plan_fresh_cells(a._h, b._h, counts[k].data_ptr(), lst[k].data_ptr(),
                                                        n, st.cuda_stream)
    def right():
        torch.cuda.synchronize()
        assert counts[:, 0].eq(n).all() and counts[:, 1].eq(unc).all()
        assert np.array_equal(lst.cpu().numpy(), np.broadcast_to(want, lst.shape))
    torch.cuda.synchronize()
    assert all(call(k, streams[k % 2]) == 0 for k in range(40))
    right()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert all(call(k, torch.cuda.current_stream()) == 0 for k in range(40))
    for _ in range(3):
        counts.zero_()
        lst.zero_()
        graph.replay()
        right()


# tiles of 16,384 cells: 512 (one to a workgroup), 513 and 1024 (two), 1025 (one
# again), 2048, 2049 and 4097 (two and three); the last one whole and half
@pytest.mark.parametrize("tiles", [512, 513, 1024, 1025, 2048, 2049, 4097])
@pytest.mark.parametrize("whole", [True, False])
def test_fresh_cells_by_several_tiles(gcr, tiles, whole):
    h = 2.0 / 8192
    ny = 2 * tiles - (0 if whole else 1)
    g = synth.Grid(2, (8192, ny, 1), (-1.0, -1.0, 0.0), (h, h, 1.0))
    # a body among the first tiles, and one across all of them
    for y, r in ((60.3 * h, 40.0 * h), (0.5 * ny * h, 0.47 * min(ny * h, 2.0))):
        c = (0.01, -1.0 + y, 0.0)
        a = gcr.Plan(g, synth.Shape(synth.SPHERE, c, r), CGC)
        b = gcr.Plan(g, synth.Shape(synth.SPHERE, (c[0] + 0.7 * h, c[1] - 0.4 * h, 0.0), r), CGC)
        ta, tb = (p.export(("tags",))["tags"] for p in (a, b))
        want = ((ta > 0) & ((tb == 0) | (tb == -2))).nonzero()[:, 0]
        lst, counts = a.fresh_cells(b, cap=len(want) + 3)
        torch.cuda.synchronize()
        unc = int(((ta == 1) & ((tb == 0) | (tb == -2))).sum())
        assert len(want) > 50 and counts.tolist() == [len(want), unc]
        assert torch.equal(lst[:len(want)].long(), want)
