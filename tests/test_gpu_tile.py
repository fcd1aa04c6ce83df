"""The tile stage kernel (one launch per stage, grids of up to 1.75 million
nodes) against the stage kernel's march, which a caller's launch shape selects:
right-hand side and Runge-Kutta steps agree to rounding at the sizes where
tiles end -- 32 k, 32 k + 1 (a last tile of 33 columns), a remainder smaller
than a closure, 8 k and 7 k rows, the smallest grids -- for every order."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [  # order, (ns, nr, nq)
    (2, (4, 4, 4)), (2, (9, 17, 64)), (2, (5, 9, 33)),
    (3, (6, 6, 6)), (3, (7, 16, 34)), (3, (13, 15, 65)),
    (4, (8, 8, 8)), (4, (17, 64, 32)), (4, (9, 29, 35)), (4, (11, 22, 129)),
    (5, (10, 10, 10)), (5, (12, 16, 36)), (5, (21, 14, 97)),
    (6, (12, 12, 12)), (6, (13, 17, 33)), (6, (15, 15, 37)), (6, (12, 65, 65)), (6, (30, 31, 70)),
    (7, (14, 14, 14)), (7, (15, 17, 38)), (7, (14, 21, 65)),
    (8, (16, 16, 16)), (8, (17, 17, 39)), (8, (16, 23, 65)),
]


def rel_max(x, y):
    """largest difference per field over the field's largest value"""
    ax = tuple(range(1, x.ndim))
    return float((np.abs(x - y).max(axis=ax) / np.maximum(np.abs(y).max(axis=ax), 1e-300)).max())


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("order,shape", SHAPES)
def test_tile_kernel_equals_the_march(order, shape, dtype):
    from paper_2011_02600_amd import sbp
    print("case: tile kernel order %d shape %s %s" % (order, shape, dtype), flush=True)
    ns, nr, nq = shape
    xyz = W.warped_mesh(nq, nr, ns, seed=order + nq, amp=0.02)
    med = W.random_medium(shape, 3)
    Q = W.random_state(shape, 5, smooth=(dtype == "f32"))
    out = {}
    for path in ("tile", "march"):
        s = sbp.Solver(xyz, order=order, dtype=dtype, gamma=[1.0, 0.0, -1.0, 0.4, 0.0, 1.0], sat_variant=order % 2)
        s.set_material(*med)
        s.add_source((0.1, 0.52, 0.61), (0.3, -0.1, 0.2, 1.0, -0.5, 0.25), 0, 2.0, 0.1)
        s.add_source((0.97, 0.98, 0.03), (0.0, 0.5, 0.2, 0.0, 1.0, 0.0), 1, 0.1, 0.0)
        if path == "march":
            s.set_launch(8, 0)
        s.set_state(Q, 0.05)
        r = s.rhs(0.13).cpu().numpy().astype(np.float64)
        traces = s.record([(0, 0, 0), (nq - 1, nr - 1, ns - 1), (nq // 2, nr // 2, ns // 2)], 3)
        s.fill_scratch(float("nan"))
        s.step(3, 1e-4)
        out[path] = (r, s.get_state().cpu().numpy().astype(np.float64),
                     traces.cpu().numpy().astype(np.float64).transpose(2, 0, 1))
        s.close()
    tol = 1e-5 if dtype == "f32" else 1e-12
    errs = [rel_max(a, b) for a, b in zip(out["tile"], out["march"])]
    print("  rel max: rhs %.1e, state %.1e, traces %.1e" % tuple(errs), flush=True)
    assert all(e <= tol for e in errs)


def test_autotune_considers_the_tile_kernel():
    """A small grid keeps the tile kernel, and a caller's shape replaces it."""
    from paper_2011_02600_amd import sbp
    print("case: autotune with the tile kernel", flush=True)
    s = sbp.Solver(W.unit_cube(65, 41, 29), order=4, dtype="f32")
    s.set_material(2.7, 6.0, 3.464)
    s.set_state(W.random_state((29, 41, 65), 1, smooth=True))
    _, _, ms = s.autotune(5)
    a = s.rhs().clone()
    s.set_launch(8, 0)
    b = s.rhs()
    assert ms > 0 and torch.allclose(a, b, rtol=1e-4, atol=1e-4 * float(b.abs().max()))
    s.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_batch_of_small_and_large_grids(dtype):
    """A batch of grids on both sides of the tile kernel's limit (a group of
    small ones over two orders, several launches of a group, the larger ones
    over the work list) against the same handles stepped one by one."""
    from paper_2011_02600_amd import sbp
    print("case: batch of small and large grids %s" % dtype, flush=True)
    grids = [(4, (40, 33, 20)), (6, (121, 122, 120)), (6, (37, 65, 25)), (4, (33, 21, 128)), (4, (121, 121, 121)),
             (3, (101, 99, 97))]

    def solvers():
        out = []
        for n, (order, shape) in enumerate(grids):
            ns, nr, nq = shape
            s = sbp.Solver(W.warped_mesh(nq, nr, ns, seed=n, amp=0.02), order=order, dtype=dtype,
                           gamma=[1, 0, 0.5, 0, -1, 1])
            s.set_material(*W.random_medium(shape, 60 + n))
            s.set_state(W.random_state(shape, 70 + n, smooth=True))
            if n % 2 == 0:
                s.add_source((0.31 + 0.05 * n, 0.5, 0.47), (0.2, 0.1, -0.3, 1.0, 0.0, 0.4), 0, 8.0, 0.05)
            s.record([(1, 2, 3), (nq - 1, nr // 2, ns - 1)], 8)
            out.append(s)
        return out

    dts = [1e-4 * (1 + 0.1 * n) for n in range(len(grids))]
    alone, together = solvers(), solvers()
    for s, d in zip(alone, dts):
        s.step(5, d)
    sbp.sbp_step_batch([s.h for s in together], 5, dts)
    tol = 1e-5 if dtype == "f32" else 1e-12
    for n, (a, b) in enumerate(zip(alone, together)):
        e = rel_max(b.get_state().double().cpu().numpy(), a.get_state().double().cpu().numpy())
        t = rel_max(b.traces.double().cpu().numpy().transpose(2, 0, 1), a.traces.double().cpu().numpy().transpose(2, 0, 1))
        print("  grid %d: state %.1e traces %.1e" % (n, e, t), flush=True)
        assert e <= tol and t <= tol and a.time() == b.time()
    for s in alone + together:
        s.close()


def test_refused_batch_advances_no_handle():
    """Two grids whose stage tiles exceed the work list (4 x 8 x 4 of a tile's
    nodes used) beside small grids that hold half of the nodes: the batch is
    refused, and no handle of it has moved."""
    from paper_2011_02600_amd import sbp
    print("case: refused batch", flush=True)
    grids = [(4, 262144, 4)] * 2 + [(97, 128, 121)] * 6  # (nq, nr, ns)
    assert 2 * 6 * 97 * 128 * 121 >= sum(a * b * c for a, b, c in grids)
    ss = []
    for nq, nr, ns in grids:
        s = sbp.Solver(W.unit_cube(nq, nr, ns), order=2, dtype="f32")
        s.set_material(2.7, 6.0, 3.464)
        ss.append(s)
        print("  handle", len(ss), flush=True)
    with pytest.raises(sbp.SBPError) as e:
        sbp.sbp_step_batch([s.h for s in ss], 2, [1e-6] * len(ss))
    assert e.value.code == sbp.SBP_EINVAL and "blocks of work" in str(e.value)
    for s in ss:
        assert s.time() == (0.0, 0)
        s.close()


def test_grids_the_march_serves_better():
    """Order 8 in single precision on 65 x 65 columns, which leave 39 % of the
    tiles' lanes idle: stages are the march's, bit for bit those of a caller's
    shape; its neighbour of 64 x 64 columns stays on the tile kernel."""
    from paper_2011_02600_amd import sbp
    print("case: grids the march serves better", flush=True)
    for shape, march in (((200, 65, 65), True), ((200, 64, 64), False)):
        ns, nr, nq = shape
        xyz, med = W.warped_mesh(nq, nr, ns, seed=3, amp=0.02), W.random_medium(shape, 4)
        Q = W.random_state(shape, 5, smooth=True)
        out = []
        for shaped in (False, True):
            s = sbp.Solver(xyz, order=8, dtype="f32", gamma=[1, 0, 0.5, 0, -1, 1])
            s.set_material(*med)
            s.set_state(Q)
            if shaped:
                s.set_launch(8, 0)
            s.step(2, 1e-4)
            out.append(s.get_state().cpu().numpy())
            s.close()
        assert np.array_equal(*out) == march
        assert rel_max(*(o.astype(np.float64) for o in out)) <= 1e-5


@pytest.mark.parametrize("nrec", [1, 256, 257, 640, 641, 5000])
def test_receivers_in_one_block_and_in_several(nrec):
    """The recorded values are the state's, step after step, and the steps go on
    with their own source-time factors, on both sides of the receivers' launch
    that also ticks the step clock."""
    from paper_2011_02600_amd import sbp
    print("case: %d receivers" % nrec, flush=True)
    nq, nr, ns = 33, 24, 21
    rec = np.random.default_rng(nrec).integers(0, (nq, nr, ns), size=(nrec, 3))
    s = sbp.Solver(W.warped_mesh(nq, nr, ns, seed=2, amp=0.02), order=4, dtype="f32", gamma=[1, 0, 0.5, 0, -1, 1])
    s.set_material(*W.random_medium((ns, nr, nq), 3))
    s.add_source((0.4, 0.5, 0.5), (1.0, 0.5, 0.2, 0.1, 0.0, 0.3), 0, 30.0, 0.002)
    q = W.random_state((ns, nr, nq), 4, smooth=True)
    s.set_state(q, 0.0)
    tr = s.record(rec, 4)
    s.step(4, 1e-3)
    got, end = tr.cpu().numpy(), s.get_state().cpu().numpy()
    s.set_state(q, 0.0)
    s.record(rec, 4)
    for n in range(4):
        s.step(1, 1e-3)
        q1 = s.get_state().cpu().numpy()
        want = q1[:3, rec[:, 2], rec[:, 1], rec[:, 0]].T
        # (a single step's source time is n dt summed up, not multiplied: one rounding)
        assert np.abs(got[n] - want).max() <= 1e-6 * np.abs(q1[:3]).max(), n
    assert np.abs(q1 - end).max() <= 1e-6 * np.abs(end).max()
    s.close()
