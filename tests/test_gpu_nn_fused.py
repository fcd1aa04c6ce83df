"""The surrogate network's fused layers against its separate calls."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# remainders of the 16-row and 16-column tiles (channels, modes, points), two
# k steps of the pointwise product (C > 32) and of the transforms (n > 32),
# fewer lines than a block's waves, receivers that share a point or a line
@pytest.mark.parametrize("S,n,m,C,L,R,same", [
    (1, 4, 2, 1, 2, 3, True), (2, 16, 4, 8, 2, 5, True), (3, 24, 7, 24, 3, 40, True), (1, 32, 16, 64, 2, 9, False),
    (2, 36, 9, 33, 2, 20, True), (8, 40, 5, 16, 2, 33, False), (1, 64, 8, 32, 4, 64, False), (2, 64, 12, 48, 2, 7, True)])
def test_fused_layers_equal_separate_calls(S, n, m, C, L, R, same):
    import torch
    from paper_2011_02600_amd import nn
    rng = np.random.default_rng(n + C)
    pos = rng.integers(0, n ** 3, size=R) if same else rng.choice(n * n, size=R, replace=False)
    if same:
        pos[1] = pos[0]
        pos[-1] = pos[0] - pos[0] % n  # (the same line)
    T = 50
    x = torch.tensor(rng.standard_normal((S, n, n, n)).astype(np.float32), device="cuda")
    ref = torch.tensor(rng.standard_normal((S, R, T)).astype(np.float32), device="cuda")
    res = []
    for fused in (False, True):
        net = nn.SpectralOperator(n, m, C, L, pos, T, seed=1)
        gen = np.random.default_rng(2)
        for l in range(L):
            net.params["b%d" % l].copy_(torch.tensor(0.1 * gen.standard_normal(C).astype(np.float32)))
        if not fused:
            net.fused = False
        for _ in range(2):  # (the second pass reuses every buffer)
            y = net.forward(x)
            _, dy = net.loss(y, ref, 1.0 / S)
            net.backward(dy)
        assert net.was_fused == fused
        res.append((y.clone(), {k: g.clone() for k, g in net.grads.items()}))
    (y0, g0), (y1, g1) = res
    assert torch.equal(y0, y1)
    for k in g0:
        if k[0] in "DR" or k == "b_out":  # the same products in the same order
            assert torch.equal(g0[k], g1[k]), k
        else:  # sums over the grid in another order: 1e-5 is about 100 float roundings
            d, r = (g1[k] - g0[k]).double().norm(), g0[k].double().norm()
            assert d <= 1e-5 * r, (k, float(d / r))


def test_layers_outside_the_fused_shapes_take_the_separate_calls():
    import torch
    from paper_2011_02600_amd import nn
    for n, m, C, L in ((18, 4, 8, 2), (16, 4, 65, 2), (16, 4, 8, 1), (68, 4, 2, 2)):
        net = nn.SpectralOperator(n, m, C, L, [0, n ** 3 - 1], 10)
        y = net.forward(torch.ones((1, n, n, n), device="cuda"))
        assert not net.was_fused and bool(torch.isfinite(y).all())
    net = nn.SpectralOperator(16, 4, 8, 2, [0, 5], 10)
    x = torch.ones((1, 16, 16, 17), device="cuda")[..., 1:]  # rows that are not 16-byte aligned
    net.forward(x.contiguous())
    assert net.was_fused


# a grid of the fused layers and one of the separate calls
@pytest.mark.parametrize("n", [16, 18])
def test_strided_and_misaligned_inputs(n):
    """A strided view of the media gives what its dense copy gives, forward and
    backward; a dense view off the 16-byte grid takes the separate calls."""
    import torch
    from paper_2011_02600_amd import nn
    rng = np.random.default_rng(n)
    pos, T, S = [3, n ** 3 - 2, n * n], 20, 2
    ref = torch.tensor(rng.standard_normal((S, len(pos), T)).astype(np.float32), device="cuda")
    wide = torch.tensor(rng.standard_normal((S, n, n, n + 1)).astype(np.float32), device="cuda")
    flat = torch.zeros(S * n ** 3 + 1, device="cuda")
    off = flat[1:].view(S, n, n, n)
    views = {"dense": wide[..., 1:].contiguous(), "strided": wide[..., 1:],
             "transposed": wide[..., 1:].transpose(1, 3).contiguous().transpose(1, 3), "offset": off}
    off.copy_(views["dense"])
    want = {}
    for name, x in views.items():
        net = nn.SpectralOperator(n, 4, 8, 2, pos, T, seed=1)
        y = net.forward(x)
        _, dy = net.loss(y, ref, 0.5)
        net.backward(dy)
        assert net.was_fused == (n == 16 and name != "offset"), name
        got = dict(net.grads, y=y)
        if name == "dense":
            want = {k: v.clone() for k, v in got.items()}
        for k, v in got.items():
            if name == "offset" and n == 16 and k not in ("y", "D", "b_out") and k[0] != "R":
                # the separate calls sum over the grid in another order
                assert (v - want[k]).double().norm() <= 1e-5 * want[k].double().norm(), (name, k)
            else:
                assert torch.equal(v, want[k]), (name, k)
