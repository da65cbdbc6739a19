"""The one-launch step of small shots (the automatic variant) against the
naive kernel, bit for bit: every point goes through the same operations in the
same order, so nothing may differ, in any storage, at any edge of a box
(32 x 8 x 4 points), with layers that meet no, one, two or three axes of it,
eager and as a graph, over a save, a change of plan, and in the adjoint's
recomputation.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

AUTO, NAIVE, ZMARCH = 0, 1, 2

# n, layers: whole boxes; one point over and one under; the smallest grid; layers wider than a box,
# on one axis only, on one face only, almost meeting in the middle; no layer
GEOMETRIES = [
    ((64, 32, 24), (10, 10, 8, 8, 6, 6)),
    ((65, 33, 25), (10, 7, 5, 8, 6, 3)),
    ((63, 31, 23), (3, 12, 12, 3, 2, 9)),
    ((9, 9, 9), (4, 4, 4, 4, 4, 4)),
    ((100, 41, 38), (36, 40, 0, 0, 0, 0)),
    ((37, 58, 30), (0, 0, 20, 25, 0, 0)),
    ((34, 19, 61), (0, 0, 0, 0, 29, 28)),   # z layers too close for the tile kernel
    ((34, 19, 61), (0, 0, 0, 0, 25, 24)),   # just far enough
    ((40, 24, 20), (0, 6, 0, 0, 1, 0)),
    ((33, 47, 29), (0,) * 6),
]


def _workload(n, cpml, nt, seed=3):
    rng = np.random.default_rng(seed)
    nx, ny, nz = n
    v = 1800.0 + 900.0 * rng.uniform(size=(nz, ny, nx))
    dt = synth.dt_from_courant(v.max(), (10.0, 11.0, 9.0)) * 0.9
    u = [rng.standard_normal((nz, ny, nx)).astype(np.float32) * 1e-3 for _ in range(2)]
    src = (nx // 3, ny // 2, nz // 2)
    rec = np.stack([rng.integers(0, m, 12) for m in n], 1).astype(np.int32)
    return v.astype(np.float32), dt, u, src, synth.ricker(nt, dt, 30.0).astype(np.float32), rec


def _prop(cases, nt, variants, storage=0):
    import torch

    from paper_2606_06910_amd import Propagator, Shot

    ws = [_workload(n, cpml, nt) for n, cpml in cases]
    p = Propagator([Shot(n=n, h=(10.0, 11.0, 9.0), dt=w[1], cpml=cpml, variant=var, storage=storage,
                         field_scale=1024.0 if storage else 0.0)
                    for (n, cpml), w, var in zip(cases, ws, variants)])
    traces = []
    for i, (v, _, _, src, wav, rec) in enumerate(ws):
        p.set_velocity(i, torch.from_numpy(v).cuda())
        p.inject_source(i, src, torch.from_numpy(wav).cuda())
        p.set_receivers(i, rec)
        traces.append(p.record(i, nt))
    return p, ws, traces


def _start(p, ws):
    """Both levels seeded noise over the whole grid, layers included."""
    import torch

    p.reset()
    for i, w in enumerate(ws):
        p.set_field(i, 0, torch.from_numpy(w[2][0]).cuda())
        p.set_field(i, 1, torch.from_numpy(w[2][1]).cuda())


def _out(p, traces):
    import torch

    torch.cuda.synchronize()
    return [x.cpu().numpy().copy() for i in range(len(traces)) for x in (traces[i], p.get_field(i, 0), p.get_field(i, 1))]


def _same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("case", GEOMETRIES, ids=lambda c: "x".join(map(str, c[0])))
def test_tile_step_equals_naive(case, storage):
    nt = 15
    got = []
    for variant in (AUTO, NAIVE):
        p, ws, tr = _prop([case], nt, [variant], storage)
        _start(p, ws)
        p.step(7)       # two calls, an odd number of steps in each
        p.step(8)
        got.append(_out(p, tr))
        p.close()
    assert np.abs(got[0][1]).max() > 0
    _same(*got)


# 1.2e7 points or more: the inner region in a launch of its own (boxes of 8 planes); faces without a layer, where it
# reaches the grid's edge; an inner region of a few boxes
LARGE = [
    ((261, 243, 197), (10, 12, 9, 20, 15, 11)),
    ((256, 240, 200), (0, 20, 20, 0, 0, 20)),
    ((225, 233, 230), (0,) * 6),
    ((97, 200, 640), (20, 20, 90, 90, 20, 20)),
]


@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("case", LARGE, ids=lambda c: "x".join(map(str, c[0])))
def test_inner_launch_equals_naive(case, storage):
    nt = 5
    got = []
    for variant in (AUTO, NAIVE):
        p, ws, tr = _prop([case], nt, [variant], storage)
        _start(p, ws)
        p.step(3)
        p.step(2)
        got.append(_out(p, tr))
        p.close()
    assert np.isfinite(got[0][1]).all() and np.abs(got[0][1]).max() > 0
    _same(*got)


# 1.6e7 points or more, where 16-bit storage takes it too: boxes of two points to a lane; regions of a few boxes, of one
# along x, at the grid's edge, and none
LARGE16 = [
    ((283, 243, 237), (10, 12, 9, 20, 15, 11)),
    ((256, 256, 257), (0, 20, 20, 0, 0, 20)),
    ((320, 229, 230), (0,) * 6),
    ((160, 170, 640), (20, 20, 70, 70, 20, 20)),
    ((129, 250, 512), (20, 2, 20, 20, 20, 20)),
]


@pytest.mark.parametrize("storage", [1, 2])
@pytest.mark.parametrize("case", LARGE16, ids=lambda c: "x".join(map(str, c[0])))
def test_inner_launch_of_pairs_equals_naive(case, storage):
    test_inner_launch_equals_naive(case, storage)


def test_inner_launch_in_a_batch_and_of_16_planes():
    """Two shots that reach the size together, eager and as a graph, and one large enough for boxes of 16 planes."""
    for cases, graphs in (([((180, 190, 200), (15,) * 6), ((200, 170, 180), (15, 10, 0, 9, 20, 15))], (False, True)),
                          ([((480, 460, 456), (20, 20, 20, 20, 0, 20))], (False,))):
        nt = 4
        single = []
        for c in cases:
            p, ws, tr = _prop([c], nt, [NAIVE])
            _start(p, ws)
            p.step(nt)
            single += _out(p, tr)
            p.close()
        for graph in graphs:
            p, ws, tr = _prop(cases, nt, [AUTO] * len(cases))
            _start(p, ws)
            p.step(nt, graph=graph)
            _same(_out(p, tr), single)
            p.close()


def test_tile_batch_equals_single_shots():
    """All geometries in one context (one launch over every shot), and beside shots of the other variants."""
    nt = 12
    single = []
    for c in GEOMETRIES:
        p, ws, tr = _prop([c], nt, [NAIVE])
        _start(p, ws)
        p.step(nt)
        single += _out(p, tr)
        p.close()
    for variants in ([AUTO] * len(GEOMETRIES), [(AUTO, NAIVE, ZMARCH)[i % 3] for i in range(len(GEOMETRIES))]):
        p, ws, tr = _prop(GEOMETRIES, nt, variants)
        _start(p, ws)
        p.step(5)
        p.step(nt - 5)
        _same(_out(p, tr), single)
        p.close()


def test_tile_graph_replays_equal_eager():
    """A small shot's graph, replayed with eager work between, against the eager steps."""
    nt = 9
    p, ws, tr = _prop([GEOMETRIES[1]], 3 * nt, [AUTO])
    _start(p, ws)
    for _ in range(3):
        p.step(nt)
    ref = _out(p, tr)
    for _ in range(3):
        tr[0].zero_()
        _start(p, ws)
        for _ in range(3):
            p.step(nt, graph=True)
            p.check_finite()
        _same(_out(p, tr), ref)
    p.close()


def test_tile_state_and_change_of_plan():
    """Saved and restored at an odd step, and handed over to the other variants at one."""
    nt, k = 16, 7
    case = GEOMETRIES[1]
    p, ws, tr = _prop([case], nt, [AUTO])
    _start(p, ws)
    p.step(k)
    blob = p.save_state()
    p.step(nt - k)
    ref = _out(p, tr)
    q, _, tq = _prop([case], nt, [AUTO])
    q.step(2)
    q.load_state(blob)
    q.step(nt - k)
    got = _out(q, tq)
    assert np.array_equal(got[0][k:], ref[0][k:])
    _same(got[1:], ref[1:])
    for variant in (NAIVE, ZMARCH):
        r, wr, trr = _prop([case], nt, [AUTO])
        _start(r, wr)
        r.step(k)
        r.set_plan(0, variant, 2, 64)
        r.step(nt - k)
        _same(_out(r, trr), ref)
        r.close()
    p.close()
    q.close()


@pytest.mark.parametrize("every", [4, 7])
def test_tile_gradient_equals_naive(every):
    """Checkpoints, recomputation and gradient of two shots, batched and one by one."""
    import torch

    nt = 17
    cases = [GEOMETRIES[1], GEOMETRIES[0]]
    got = []
    for variant in (AUTO, NAIVE):
        p, ws, tr = _prop(cases, nt, [variant] * 2)
        for i in range(2):
            p.set_checkpointing(i, every, nt)
        p.reset()
        p.step(nt)
        g = torch.Generator().manual_seed(1)
        resid = [torch.randn(nt, 12, generator=g) for _ in range(2)]
        grads = p.adjoint_all(nt, resid) + [p.adjoint(i, nt, resid[i]) for i in (1, 0)]
        got.append([x.cpu().numpy() for x in tr + grads])
        p.close()
    assert np.abs(got[0][2]).max() > 0
    assert np.array_equal(got[0][2], got[0][5]) and np.array_equal(got[0][3], got[0][4])
    _same(*got)


# z layers (where there are two) at least 20 planes apart: the reverse step in one launch
ADJOINT_GEOMETRIES = [
    ((64, 32, 33), (10, 10, 8, 8, 6, 6)),
    ((65, 33, 30), (10, 7, 5, 8, 6, 3)),
    ((63, 31, 31), (3, 12, 12, 3, 2, 9)),
    ((100, 41, 38), (36, 40, 0, 0, 0, 0)),
    ((37, 58, 30), (0, 0, 20, 25, 0, 0)),
    ((40, 24, 20), (0, 6, 0, 0, 1, 0)),
    ((20, 19, 60), (9, 9, 9, 9, 15, 25)),
    ((33, 47, 29), (0,) * 6),
]


@pytest.mark.parametrize("case", ADJOINT_GEOMETRIES, ids=lambda c: "x".join(map(str, c[0])))
def test_adjoint_in_one_launch_equals_passes(case):
    """The one-launch reverse step against the three passes, bit for bit: a shot whose z layers are too close for
    the one launch puts every sweep of its context on the passes."""
    import torch

    nt = 13
    close = ((24, 20, 30), (4, 4, 4, 4, 8, 8))
    got = []
    for cases in ([case], [case, close]):
        p, ws, tr = _prop(cases, nt, [ZMARCH] * len(cases))
        for i in range(len(cases)):
            p.set_checkpointing(i, 5, nt)
        p.reset()
        for i, w in enumerate(ws):
            p.set_field(i, 0, torch.from_numpy(w[2][0]).cuda())
            p.set_field(i, 1, torch.from_numpy(w[2][1]).cuda())
        p.step(nt)
        g = torch.Generator().manual_seed(2)
        grad = p.adjoint(0, nt, torch.randn(nt, 12, generator=g))
        got.append(grad.cpu().numpy())
        p.close()
    assert np.abs(got[0]).max() > 0
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("rec", ["dense", "corners"])
def test_residuals_in_the_reverse_step(rec):
    """Residuals added by the one-launch reverse step against the pass of their own: more receiver locations in a box
    than threads, with repeated ones, and receivers on the corners of boxes and of the grid."""
    import torch

    nt, n, lay = 9, (65, 33, 34), (10, 7, 5, 8, 6, 3)
    if rec == "dense":
        g = np.stack(np.meshgrid(np.arange(28, 65), np.arange(7, 10), np.arange(3, 9), indexing="ij"), -1).reshape(-1, 3)
        r = np.concatenate([g, g[::7], g[:5]])
        r = r[np.random.default_rng(0).permutation(len(r))]
    else:
        r = np.array([(x, y, z) for x in (0, 31, 32, 64) for y in (0, 7, 8, 32) for z in (0, 3, 4, 33)])
    close = ((24, 20, 30), (4, 4, 4, 4, 8, 8))
    got = []
    for cases in ([(n, lay)], [(n, lay), close]):
        p, ws, _ = _prop(cases, nt, [ZMARCH] * len(cases))
        p.set_receivers(0, r.astype(np.int32))
        tr = p.record(0, nt)
        for i in range(len(cases)):
            p.set_checkpointing(i, 4, nt)
        p.reset()
        p.step(nt)
        g = torch.Generator().manual_seed(3)
        got.append([tr.cpu().numpy(), p.adjoint(0, nt, torch.randn(nt, len(r), generator=g)).cpu().numpy()])
        p.close()
    assert np.abs(got[0][1]).max() > 0
    _same(*got)


def test_increments_of_the_inner_launch():
    """A gradient whose recomputed steps take two launches, against one recomputed by the naive kernel."""
    import torch

    nt = 5
    got = []
    for variant in (AUTO, NAIVE):
        p, ws, _ = _prop([LARGE[0]], nt, [variant])
        p.set_checkpointing(0, 3, nt)
        _start(p, ws)
        p.step(nt)
        g = torch.Generator().manual_seed(4)
        got.append([p.adjoint(0, nt, torch.randn(nt, 12, generator=g)).cpu().numpy()])
        p.close()
    assert np.abs(got[0][0]).max() > 0
    _same(*got)


@pytest.mark.parametrize("case", [
    ((9, 9, 9), (4, 4, 4, 4, 4, 4)),
    ((64, 32, 24), (10, 10, 8, 8, 6, 6)),
    ((65, 33, 25), (10, 7, 5, 8, 6, 3)),
    ((63, 31, 23), (3, 12, 12, 3, 2, 9)),
    ((100, 41, 38), (36, 40, 0, 0, 20, 17)),
    ((34, 45, 61), (0, 1, 20, 24, 0, 0)),
    ((33, 47, 29), (0,) * 6),
    ((200, 180, 172), (12,) * 6),      # large enough for the non-temporal accesses
], ids=lambda c: "x".join(map(str, c[0])))
def test_pv_in_one_launch_equals_stages(case):
    """The first-order step in one launch (the automatic variant) against the two stages, bit for bit: sources in
    and outside the layers, receivers, several calls of odd step counts, a pressure set in between."""
    import torch

    from paper_2606_06910_amd import PVPropagator

    n, cpml = case
    rng = np.random.default_rng(5)
    p0 = torch.from_numpy(rng.standard_normal(n[::-1]).astype(np.float32))
    rec = np.stack([rng.integers(0, m, 300) for m in n], 1).astype(np.int32)
    wav = torch.from_numpy(synth.ricker(14, 0.3, 0.2).astype(np.float32))
    got = []
    for variant in (0, 1):
        s = PVPropagator(n, cpml, 0.3, variant=variant)
        s.set_pressure(p0)
        s.set_source((n[0] - 1, n[1] // 2, 1), wav)
        tr = s.record(rec, 12)      # the last steps are not recorded
        out = []
        for k in (5, 1, 8):
            s.step(k)
            p = s.get_pressure()
            out.append(p.cpu().numpy())
            s.set_pressure(p + 0.5 * p0.cuda())
        torch.cuda.synchronize()
        got.append(out + [tr.cpu().numpy()])
        s.close()
    assert np.isfinite(got[0][2]).all() and np.abs(got[0][2]).max() > 0
    _same(*got)


@pytest.mark.parametrize("case", [
    ((361, 343, 257), (10, 12, 9, 20, 15, 11)),
    ((320, 320, 300), (0, 20, 20, 0, 0, 20)),
    ((321, 313, 310), (0,) * 6),
    ((320, 312, 312), (1,) * 6),
    ((100, 480, 640), (28, 29, 90, 80, 3, 5)),     # one box along x
], ids=lambda c: "x".join(map(str, c[0])))
def test_pv_inner_launch_equals_stages(case):
    """Large enough for a launch of its own for the boxes out of every layer's reach."""
    test_pv_in_one_launch_equals_stages(case)


@pytest.mark.parametrize("cases", [GEOMETRIES[:1], GEOMETRIES[:2]], ids=["one", "two"])
def test_graph_replays_take_a_new_source_and_model(cases):
    """A survey's loop on one context: new source, new model, or both, reset, the same graph; each pass against eager
    steps of a context made for it."""
    import torch

    nt = 12
    p, ws, tr = _prop(cases, nt, [AUTO] * len(cases))

    def model(q, i, k):
        q.set_velocity(i, torch.from_numpy(ws[i][0] * np.float32(1.0 - 0.02 * k)).cuda())

    def source(q, i, k):
        q.inject_source(i, (2 + k, 3, 4 + k), torch.from_numpy(ws[i][4] * np.float32(1 + k)).cuda())

    for k, (new_source, new_model) in enumerate([(0, 0), (1, 0), (0, 1), (1, 1), (0, 0)]):
        ks = k if new_source else (ks if k else 0)
        km = k if new_model else (km if k else 0)
        q, _, tq = _prop(cases, nt, [AUTO] * len(cases))
        for i in range(len(cases)):
            if new_source:
                source(p, i, ks)
            if new_model:
                model(p, i, km)
            if ks:
                source(q, i, ks)
            if km:
                model(q, i, km)
            tr[i].zero_()
        p.reset()
        p.step(nt, graph=True)
        q.reset()
        q.step(nt)
        got = _out(p, tr)
        assert np.abs(got[0]).max() > 0
        _same(got, _out(q, tq))
        q.close()
    p.close()


@pytest.mark.parametrize("first", [0, 1])
def test_captured_first_order_steps_replay(first):
    """Steps captured by the caller, replayed with eager steps of odd counts between, against eager steps alone; the
    state lies in the first (0) or second (1) buffers when captured."""
    import torch

    from paper_2606_06910_amd import PVPropagator

    n, cpml = (65, 33, 25), (10, 7, 5, 8, 6, 3)
    p0 = torch.from_numpy(np.random.default_rng(8).standard_normal(n[::-1]).astype(np.float32)).cuda()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s, ref = PVPropagator(n, cpml, 0.3, stream=st), PVPropagator(n, cpml, 0.3, stream=st)
        for q in (s, ref):
            q.set_pressure(p0)
            q.step(first)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            s.step(3)
        for eager in (0, 1, 2, 5):
            g.replay()
            s.step(eager)
            ref.step(3 + eager)
            torch.cuda.synchronize()
            a, b = s.get_pressure().cpu().numpy(), ref.get_pressure().cpu().numpy()
            assert np.abs(b).max() > 0 and np.array_equal(a, b)
        del g
        s.close()
        ref.close()


def _tight(monkeypatch, least):
    """Allocations of more bytes than `least` (a workspace, with its alignment) fail."""
    import torch

    empty = torch.empty

    def tight(*size, **kw):
        if kw.get("dtype") == torch.uint8 and size[0] > least:
            raise torch.OutOfMemoryError("no room")
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", tight)


def test_first_order_grid_where_seventeen_fields_do_not_fit(monkeypatch):
    """The automatic variant falls back to the stages' ten fields, with the same bits."""
    import torch

    from paper_2606_06910_amd import PVPropagator

    n, cpml = (65, 33, 25), (10, 7, 5, 8, 6, 3)
    p0 = torch.from_numpy(np.random.default_rng(9).standard_normal(n[::-1]).astype(np.float32)).cuda()
    wav = torch.from_numpy(synth.ricker(14, 0.3, 0.2).astype(np.float32))
    got = []
    least = PVPropagator(n, cpml, 0.3, variant=1).ws_bytes
    for tight in (False, True):
        if tight:
            _tight(monkeypatch, least + 256)
        s = PVPropagator(n, cpml, 0.3)
        assert (s.ws_bytes == least) == tight
        s.set_pressure(p0)
        s.set_source((3, 4, 5), wav)
        tr = s.record(np.array([[5, 6, 7], [60, 30, 20]], np.int32), 9)
        s.step(4)
        s.step(5)
        torch.cuda.synchronize()
        got.append([s.get_pressure().cpu().numpy(), tr.cpu().numpy()])
        s.close()
    assert np.abs(got[0][0]).max() > 0
    _same(*got)


@pytest.mark.parametrize("cases", [GEOMETRIES[1:2], GEOMETRIES[:2]], ids=["one", "two"])
def test_shots_where_a_second_psi_does_not_fit(monkeypatch, cases):
    """The automatic variant falls back to the kernels of its reported plan, with the same bits."""
    nt, got = 9, []
    p, _, _ = _prop(cases, nt, [NAIVE if len(cases) == 1 else ZMARCH] * len(cases))
    least = p.ws_bytes
    p.close()
    for tight in (False, True):
        if tight:
            _tight(monkeypatch, least + 256)
        p, ws, tr = _prop(cases, nt, [AUTO] * len(cases))
        assert (p.ws_bytes == least) == tight
        _start(p, ws)
        p.step(4)
        p.step(5, graph=True)
        got.append(_out(p, tr))
        p.close()
    assert np.abs(got[0][1]).max() > 0
    _same(*got)


def _single_naive(cases, nt, storage):
    out = []
    for c in cases:
        p, ws, tr = _prop([c], nt, [NAIVE], storage)
        _start(p, ws)
        p.step(nt)
        out += _out(p, tr)
        p.close()
    return out


@pytest.mark.parametrize("storage", [1, 2])
@pytest.mark.parametrize("cases", [
    GEOMETRIES,                                                                               # k_tile alone
    [((220, 190, 200), (15,) * 6), ((240, 200, 180), (15, 10, 0, 9, 20, 15))],                # all three launches
    LARGE16[:1],                                                                              # a lone shot's graph
], ids=["small", "large", "lone"])
def test_sixteen_bit_batch_equals_single_shots(cases, storage):
    """16-bit shots of one context (descriptors by the items' shot), eager and as a graph that is replayed, against each
    alone on the naive kernel."""
    nt = 4
    single = _single_naive(cases, nt, storage)
    p, ws, tr = _prop(cases, nt, [AUTO] * len(cases), storage)
    for graph in (False, True, True):
        for t in tr:
            t.zero_()
        _start(p, ws)
        p.step(nt, graph=graph)
        _same(_out(p, tr), single)
    p.close()


def test_gradients_of_a_context_with_tile_and_other_shots():
    """Batched sweep over tile, naive and z-march shots (their increments in a pass of its own, the tile shots stepped by
    k_tile all the same) and each shot's own sweep, against a context of naive shots."""
    import torch

    nt = 13
    cases = [GEOMETRIES[0], GEOMETRIES[1], GEOMETRIES[4], GEOMETRIES[9]]
    got = []
    for variants in ([AUTO, NAIVE, ZMARCH, AUTO], [NAIVE] * 4):
        p, ws, tr = _prop(cases, nt, variants)
        for i in range(4):
            p.set_checkpointing(i, 5, nt)
        p.reset()
        p.step(nt)
        g = torch.Generator().manual_seed(6)
        resid = [torch.randn(nt, 12, generator=g) for _ in cases]
        grads = p.adjoint_all(nt, resid) + [p.adjoint(i, nt, resid[i]) for i in range(4)]
        got.append([x.cpu().numpy() for x in tr + grads])
        p.close()
    assert all(np.abs(x).max() > 0 for x in got[0])
    for i in range(4):
        assert np.array_equal(got[0][4 + i], got[0][8 + i])
    _same(*got)
