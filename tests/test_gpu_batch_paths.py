"""The launches a batch can take, each reached on purpose: a launch shape of
the caller's keeps a small grid off the tile kernel, so that the work list and
the launches per order run on grids the oracle can follow; batches of small
and larger grids split by the rule on their nodes (small: up to 1.75 million;
apart if they hold at least half), in groups of at most 250 MB."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import elastic as E

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 2e-5}  # as in test_gpu_boundary.py
SMALL, GROUP_BYTES = 1750000, 250e6


def rel_l2(got, want):
    return max(np.linalg.norm(g - w) / max(np.linalg.norm(w), 1e-300) for g, w in zip(got, want))


def make(i, shape, order, dtype, steps, march):
    from paper_2011_02600_amd import sbp
    ns, nr, nq = shape
    xyz = W.warped_mesh(nq, nr, ns, seed=30 + i)
    med = W.random_medium(shape, 40 + i)
    s = sbp.Solver(xyz, order=order, dtype=dtype, gamma=[0.0, 1.0, 0.5, 0.0, -1.0, 1.0])
    s.set_material(*med)
    if i % 3 < 2:
        s.add_source((0.35 + 0.02 * i, 0.5, 0.45), (0.1, 0.0, 0.0, 1.0, 0.2 * i, 0.0), 0, 5.0 + i, 0.1)
    rec = np.array([[2, 3, ns - 1], [nq - 1, nr - 4, ns - 1], [nq // 2, nr - 1, ns // 2]], dtype=np.int64)
    if i % 2 == 0:
        s.record(rec, steps)
    Q0 = W.random_state(shape, 50 + i, smooth=True) * 1e-3
    s.set_state(Q0)
    if march:
        s.set_launch(8, 0)
    dt = W.cfl_dt(xyz, med[1], 0.25 if order == 8 else 0.4)
    return s, dict(xyz=xyz, med=med, rec=rec, Q0=Q0, dt=dt, order=order, i=i)


def state(s):
    return s.get_state().cpu().numpy().astype(np.float64)


# (ns, nr, nq), order: the orders the work list serves, with tiles of 64 k + 1
# columns and 8 k + 1 rows, whose last column and row are edge blocks; then
# orders that send the batch to launches per order
CASES = {
    "list": [((19, 17, 21), 2), ((23, 25, 18), 6), ((17, 25, 65), 3), ((21, 19, 24), 5), ((14, 33, 33), 4)],
    "list7": [((19, 17, 21), 7), ((15, 17, 65), 7), ((23, 21, 18), 2)],
    "per order 8": [((19, 17, 21), 4), ((17, 18, 65), 8), ((17, 25, 19), 5), ((16, 17, 20), 8)],
    "per order 7": [((19, 17, 21), 2), ((15, 18, 19), 7), ((17, 25, 65), 3)],
}


@pytest.mark.parametrize("dtype,kind", [("f32", "list"), ("f64", "list"), ("f32", "list7"), ("f32", "per order 8"),
                                        ("f64", "per order 8"), ("f64", "per order 7")])
def test_batches_off_the_tile_kernel_against_oracle(dtype, kind):
    from paper_2011_02600_amd import sbp
    print("case: batch %s %s" % (kind, dtype), flush=True)
    steps = 40
    made = [make(i, shape, order, dtype, steps, True) for i, (shape, order) in enumerate(CASES[kind])]
    sbp.sbp_step_batch([s.h for s, _ in made], steps, [c["dt"] for _, c in made])
    tiles = [make(i, shape, order, dtype, steps, False) for i, (shape, order) in enumerate(CASES[kind])]
    sbp.sbp_step_batch([s.h for s, _ in tiles], steps, [c["dt"] for _, c in tiles])
    for (s, c), (t, _) in zip(made, tiles):
        got = state(s)
        assert not np.array_equal(got, state(t))  # (another kernel)
        blk = E.Block(c["xyz"], c["order"]).set_material(*c["med"])
        i = c["i"]
        srcs = [E.Source(blk, (0.35 + 0.02 * i, 0.5, 0.45), (0.1, 0.0, 0.0, 1.0, 0.2 * i, 0.0), E.STF_RICKER, 5.0 + i,
                         0.1)] if i % 3 < 2 else []
        want, _, wtr = E.run(blk, c["Q0"], steps, c["dt"], [0.0, 1.0, 0.5, 0.0, -1.0, 1.0], sources=srcs,
                             receivers=c["rec"])
        err = rel_l2(got, want)
        print("  shot %d order %d: state %.1e" % (i, c["order"], err), flush=True)
        assert err <= TOL[dtype] and s.time()[1] == steps
        if i % 2 == 0:
            tr = s.traces.cpu().numpy().astype(np.float64)
            assert np.linalg.norm(tr - wtr) <= TOL[dtype] * np.linalg.norm(wtr)
        s.close()
        t.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_work_list_graph_replay_equals_eager(dtype):
    """Over two calls and several chunks of the source-time table."""
    from paper_2011_02600_amd import sbp
    print("case: work list, graphs against eager %s" % dtype, flush=True)
    runs = []
    for graphs in (True, False):
        made = [make(i, shape, order, dtype, 200, True) for i, (shape, order) in enumerate(CASES["list"][:3])]
        made[0][0].set_graphs(graphs)
        for n in (17, 183):
            sbp.sbp_step_batch([s.h for s, _ in made], n, [c["dt"] for _, c in made])
        runs.append([(state(s), s.traces.cpu().numpy() if c["i"] % 2 == 0 else 0, s.time()) for s, c in made])
        for s, _ in made:
            s.close()
    for (qa, ta, tma), (qb, tb, tmb) in zip(*runs):
        assert np.isfinite(qa).all() and np.abs(qa).max() > 0
        assert np.array_equal(qa, qb) and np.array_equal(ta, tb) and tma == tmb


SMALLS = [((84, 85, 86), 4), ((40, 33, 20), 6), ((85, 86, 84), 4), ((86, 84, 85), 6), ((37, 65, 25), 6), ((88, 84, 85), 4),
          ((85, 85, 85), 3), ((84, 84, 89), 4), ((97, 82, 81), 6)]
LARGES = [((121, 121, 121), 4), ((120, 122, 121), 6)]


@pytest.mark.parametrize("nlarge", [2, 1])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_small_grids_beside_larger_ones(dtype, nlarge):
    """Small grids that hold most of the nodes run as they do without the
    larger ones, bit for bit: in groups, with two larger grids on the work
    list as those do alone, and a single one as sbp_step runs it."""
    from paper_2011_02600_amd import sbp
    print("case: %d larger grids beside small ones %s" % (nlarge, dtype), flush=True)
    grids = SMALLS + LARGES[:nlarge]
    nodes = [int(np.prod(shape)) for shape, _ in grids]
    ns = len(SMALLS)
    assert max(nodes[:ns]) <= SMALL < min(nodes[ns:]) and 2 * sum(nodes[:ns]) >= sum(nodes)
    assert 39 * (4 if dtype == "f32" else 8) * sum(nodes[:ns]) > 2 * GROUP_BYTES  # (several groups)
    steps = 7
    order = [1, 9, 0, 2, 3, 4, 10, 5, 6, 7, 8] if nlarge == 2 else [1, 0, 9, 2, 3, 4, 5, 6, 7, 8]

    def run(which):
        made = {i: make(i, *grids[i], dtype, steps, False) for i in which}
        if len(which) == 1:
            s, c = made[which[0]]
            s.step(steps, c["dt"])
        else:
            sbp.sbp_step_batch([made[i][0].h for i in which], steps, [made[i][1]["dt"] for i in which])
        out = {}
        for i, (s, c) in made.items():
            out[i] = (state(s), s.traces.cpu().numpy() if i % 2 == 0 else 0, s.time())
            s.close()
        return out

    got = run(order)
    want = run(list(range(ns)))
    want.update(run([i for i in range(ns, len(grids))]))
    for i in order:
        assert np.isfinite(got[i][0]).all() and np.abs(got[i][0]).max() > 0
        assert np.array_equal(got[i][0], want[i][0]) and np.array_equal(got[i][1], want[i][1]), grids[i]
        assert got[i][2] == want[i][2]
        s, c = make(i, *grids[i], dtype, steps, False)
        s.step(steps, c["dt"])
        alone = state(s)
        e = max(np.abs(a - b).max() / np.abs(b).max() for a, b in zip(got[i][0], alone))
        assert e <= (1e-5 if dtype == "f32" else 1e-12), (grids[i], e)
        s.close()
