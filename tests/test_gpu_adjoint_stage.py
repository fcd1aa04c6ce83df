"""The pass between two right-hand sides of the reverse sweep, on grids where
its surface and interior blocks end: the transposed operator against the
operator itself, <l, L q> = <L^T l, q> in double precision, and the gradient
against a central difference along one direction."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GAMMA = (0.25, -1.0, 1.0, 0.0, 0.5, -0.5)


# smallest grids of an order (few interior nodes), surfaces and interiors below
# and above a block of 256, grids above the tile kernel's
@pytest.mark.parametrize("order,shape,variant,gamma", [
    (2, (4, 4, 4), 0, GAMMA), (2, (5, 4, 6), 1, GAMMA), (4, (8, 8, 8), 1, (1.0,) * 6), (4, (8, 8, 17), 0, (1.0,) * 6),
    (6, (12, 13, 129), 0, GAMMA), (5, (124, 122, 118), 1, (1.0, 0.0, 1.0, -1.0, 0.5, 1.0))])
def test_transposed_operator_and_gradient(order, shape, variant, gamma):
    from paper_2011_02600_amd import sbp
    ns, nr, nq = shape
    xyz = W.warped_mesh(nq, nr, ns, seed=order, amp=0.02)
    med = W.random_medium(shape, 3)
    s = sbp.Solver(xyz, order=order, dtype="f64", gamma=gamma, sat_variant=variant)
    s.set_material(*med)
    q, lam = W.random_state(shape, 1), W.random_state(shape, 2)
    s.set_state(q, 0.0)
    lq = s.rhs(0.0).cpu().numpy()
    ltl = s.adjoint_rhs(torch.from_numpy(lam).cuda()).cpu().numpy()
    a, b = (lam * lq).ravel(), (ltl * q).ravel()
    # the transposed operator is within 4e-13 of the explicit transpose per
    # field (test_gpu_adjoint.py): 1e-12 of the terms' sum
    assert abs(a.sum() - b.sum()) <= 1e-12 * (np.abs(a).sum() + np.abs(b).sum())
    if np.prod(shape) > 1e5:
        s.close()
        return
    # gradient of chi = 1/2 |traces|^2 along one direction of every parameter
    nsteps = 3
    dt = W.cfl_dt(xyz, med[1], 0.2)
    rec = np.array([[0, 0, ns - 1], [nq - 1, nr // 2, ns // 2], [nq // 2, nr // 2, 1]], dtype=np.int64)

    def traces(r, la, m):
        s.set_material(r, np.sqrt((la + 2 * m) / r), np.sqrt(m / r))
        s.set_state(q, 0.0)
        tr = s.record(rec, nsteps)
        s.step(nsteps, dt)
        return tr.double().cpu()

    mu = med[0] * med[2] ** 2
    base = [med[0], med[0] * med[1] ** 2 - 2 * mu, mu]
    rng = np.random.default_rng(5)
    dirs = [p * rng.uniform(-1, 1, size=shape) for p in base]
    tr = traces(*base)
    s.set_state(q, 0.0)
    terms = s.gradient(nsteps, dt, tr, 2).cpu().numpy() * np.stack(dirs)
    eps = 1e-5
    chi = [0.5 * float((traces(*(p + sg * eps * d for p, d in zip(base, dirs))) ** 2).sum()) for sg in (1, -1)]
    # central difference: eps^2 and 2^-53 / eps, both about 1e-10
    assert abs(terms.sum() - (chi[0] - chi[1]) / (2 * eps)) <= 1e-6 * np.abs(terms).sum()
    s.close()


# one block for the whole run, a last block shorter than the others, blocks of
# one step; grids of the tile kernel and of the march, and single-precision
# right-hand sides on the tile kernel where the stages march (2.1 million nodes)
@pytest.mark.parametrize("order,n,dtype,nsteps,every", [
    (4, 17, "f64", 6, 9), (4, 17, "f32", 7, 3), (3, 18, "f64", 4, 1), (6, 128, "f32", 5, 2)])
def test_checkpointed_run_keeps_its_last_block(order, n, dtype, nsteps, every):
    from paper_2011_02600_amd import sbp
    shape = (n, n, n + 1)
    xyz = W.warped_mesh(n + 1, n, n, seed=2, amp=0.02)
    med = W.random_medium(shape, 4)
    dt = W.cfl_dt(xyz, med[1], 0.2)
    rec = np.array([[n, 0, 1], [n // 2, n // 2, n - 1]], dtype=np.int64)
    s = sbp.Solver(xyz, order=order, dtype=dtype, gamma=GAMMA)
    s.set_material(*med)
    s.add_source((0.4, 0.6, 0.5), (1.0, 0.9, 0.8, 0.1, 0.2, 0.3), sbp.SBP_STF_RICKER, 0.3 / dt / nsteps, 2 * dt)
    q = 0.1 * W.random_state(shape, 5, smooth=True)
    s.set_state(q, 0.0)
    tr = s.record(rec, 2 * nsteps)
    s.step(nsteps, dt)
    want = tr[:nsteps].clone()
    s.step(nsteps, dt)
    after, want2 = s.get_state().clone(), tr[nsteps:].clone()
    # the checkpointed run records and ends as the plain one, also in the middle of a recording
    s.set_state(q, 0.0)
    tr = s.record(rec, 2 * nsteps)
    s.step_checkpointed(nsteps, dt, every)
    tol = 1e-12 if dtype == "f64" else 1e-5
    res = tr[:nsteps].clone()
    assert float((res - want).abs().max()) <= tol * float(want.abs().max())
    g1 = s.gradient_from_checkpoints(res)
    g2 = s.gradient_from_checkpoints(res)  # (the kept block is gone if there were several)
    assert torch.equal(g1, g2)
    s.step(nsteps, dt)
    assert float((s.get_state() - after).abs().max()) <= tol * float(after.abs().max())
    assert float((tr[nsteps:] - want2).abs().max()) <= tol * float(want2.abs().max())
    s.set_state(q, 0.0)
    g3 = s.gradient(nsteps, dt, res, every)
    assert float((g3 - g1).abs().max()) <= 10 * tol * float(g1.abs().max())
    s.close()


def test_autotune_leaves_the_reverse_sweeps_kernel():
    """Above 1.75 million nodes sbp_autotune times the march's shapes alone, so
    its choice does not take the penalty-free right-hand sides off the tile
    kernel: the transposed operator keeps its bits.  A shape of the caller's
    does select the march, which rounds differently."""
    from paper_2011_02600_amd import sbp
    shape = (121, 121, 122)
    s = sbp.Solver(W.unit_cube(122, 121, 121), order=4, dtype="f32", gamma=GAMMA)
    s.set_material(*W.random_medium(shape, 4))
    lam = torch.from_numpy(W.random_state(shape, 6, smooth=True)).cuda()
    want = s.adjoint_rhs(lam).clone()
    s.autotune(1)
    assert torch.equal(s.adjoint_rhs(lam), want)
    s.set_launch(8, 0)
    march = s.adjoint_rhs(lam)
    assert not torch.equal(march, want)
    # single precision, sums of some 60 terms in another order
    assert float((march - want).abs().max()) <= 1e-5 * float(want.abs().max())
    s.autotune(1)
    assert torch.equal(s.adjoint_rhs(lam), want)
    s.close()


# single precision on the march (a caller's launch shape): tiles with edge
# blocks, an order without work-list kernels
@pytest.mark.parametrize("order,shape,variant", [(4, (11, 17, 65), 0), (6, (13, 12, 40), 1), (3, (9, 25, 70), 1),
                                                 (8, (16, 17, 65), 0)])
def test_single_precision_reverse_sweep_on_the_march(order, shape, variant):
    from oracle import adjoint as ADJ
    from oracle import elastic as E
    from paper_2011_02600_amd import sbp
    ns, nr, nq = shape
    xyz = W.warped_mesh(nq, nr, ns, seed=order + nq, amp=0.02)
    med = W.random_medium(shape, 7)
    lam = W.random_state(shape, 9, smooth=True)
    q, nsteps = 0.1 * W.random_state(shape, 5, smooth=True), 6
    dt = W.cfl_dt(xyz, med[1], 0.2)
    rec = np.array([[nq - 1, 0, 1], [nq // 2, nr // 2, ns - 1]], dtype=np.int64)
    want = ADJ.adjoint_rhs(E.Block(xyz, order).set_material(*med), lam, GAMMA, variant)
    rhs, grads = {}, {}
    for name, dtype in (("march", "f32"), ("tile", "f32"), ("double", "f64")):
        s = sbp.Solver(xyz, order=order, dtype=dtype, gamma=GAMMA, sat_variant=variant)
        s.set_material(*med)
        if name == "march":
            s.set_launch(8, 0)
        rhs[name] = s.adjoint_rhs(torch.from_numpy(lam).cuda()).double().cpu().numpy()
        s.set_state(q, 0.0)
        tr = s.record(rec, nsteps)
        s.step_checkpointed(nsteps, dt, 4)
        if name == "march":
            res = tr.clone()
        grads[name] = s.gradient_from_checkpoints(res.to(tr.dtype)).double().cpu().numpy()
        s.close()
    assert not np.array_equal(rhs["march"], rhs["tile"])  # (another kernel)
    # the bars of test_gpu_adjoint.py
    for got, ref, tol in ((rhs["march"], want, 1e-5), (grads["march"], grads["double"], 1e-4)):
        for g, w in zip(got, ref):
            assert np.abs(g - w).max() <= tol * np.abs(w).max()


def test_right_hand_sides_the_march_serves_better():
    """Order 8 in single precision on 65 x 65 columns: the reverse sweep's
    right-hand sides are the march's, bit for bit those of a caller's shape; on 64
    x 64 columns the tile kernel's."""
    from paper_2011_02600_amd import sbp
    for shape, march in (((400, 65, 65), True), ((400, 64, 64), False)):
        ns, nr, nq = shape
        s = sbp.Solver(W.unit_cube(nq, nr, ns), order=8, dtype="f32", gamma=GAMMA)
        s.set_material(*W.random_medium(shape, 4))
        lam = torch.from_numpy(W.random_state(shape, 6, smooth=True)).cuda()
        auto = s.adjoint_rhs(lam).clone()
        s.set_launch(8, 0)
        shaped = s.adjoint_rhs(lam)
        assert torch.equal(auto, shaped) == march
        assert float((auto - shaped).abs().max()) <= 1e-5 * float(shaped.abs().max())
        s.close()
