"""The relaxed forward from states of the caller's, of few steps: its first
state is kept for the adjoint and tells which tiles hold burning mass, in envs
of one strip of columns and of several.  Across the plans the same states to
the bit and the same gradient but for the order of its sums; and the gradient
against differences of the forward.
"""
import numpy as np
import pytest
import torch

import firegen

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")

SMALL = [(1, 1), (1, 63), (2, 64), (3, 65), (31, 20), (32, 64), (33, 63), (64, 3), (65, 64), (40, 129), (97, 200)]
# (alone they are below the 8 tiles per env from which the sparse plan skips any)
LARGE = SMALL + [(520, 700)]


def _params(seed):
    return firegen.Params(p_base=0.5, p_continue=0.55,
                          veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(seed))))


@pytest.mark.parametrize("sizes", [SMALL, LARGE])
@pytest.mark.parametrize("T,k", [(1, 1), (3, 2), (5, 1)])
def test_states_of_the_callers(T, k, sizes):
    batch = firegen.landscape_batch(104, sizes)
    params = _params(104)
    rng = np.random.default_rng(9)
    U0 = rng.uniform(0.0, 1.0, batch.n_cells)
    B0 = np.where(rng.random(batch.n_cells) < 0.02 * (np.arange(batch.n_cells) < 60000), rng.uniform(0.0, 1.0, batch.n_cells), 0.0)
    seed_u = rng.normal(size=batch.n_cells)
    got = {}
    for fwd in (0, 1):
        for bwd in (0, 1):
            sim = fs.FireSim.from_batch(batch, params, seed=0)
            p = fs.make_params(params)
            p.unburnable_mask = batch.unburnable_mask
            sim.set_plan(sparse=fwd)
            U, B = torch.from_numpy(U0.copy()).cuda(), torch.from_numpy(B0.copy()).cuda()
            ws = sim.relaxed_workspace(T, k)
            ws.fill_(0xFF)
            sim.relaxed_fwd(p, U, B, T, k, ws, "product")
            sim.set_plan(sparse=bwd)
            grads = [sim.relaxed_bwd(p, torch.from_numpy(seed_u).cuda(), None, T, k, ws, "product").cpu().numpy()
                     for _ in range(2)]
            assert np.array_equal(grads[0], grads[1])
            got[fwd, bwd] = U.cpu().numpy(), B.cpu().numpy(), grads[0]
    # the directional derivative along theta by central differences of the dense forward
    sim = fs.FireSim.from_batch(batch, params, seed=0)
    sim.set_plan(sparse=0)
    base = fs.make_params(params)
    base.unburnable_mask = batch.unburnable_mask
    theta = np.array([base.p_base, base.alpha_w1, base.alpha_w2, base.alpha_s, base.alpha_gamma, base.p_continue] +
                     list(base.veg))
    d = np.zeros(17)
    d[4] = 1.0  # alpha_gamma

    def value(t):
        p = fs.params_with_theta(base, t)
        U, B = torch.from_numpy(U0.copy()).cuda(), torch.from_numpy(B0.copy()).cuda()
        ws = sim.relaxed_workspace(T, k)
        sim.relaxed_fwd(p, U, B, T, k, ws, "product")
        return float((U.cpu().numpy() * seed_u).sum())

    h = 2.0 ** -9
    lo, hi = theta - h * d, theta + h * d
    numeric = (value(hi) - value(lo)) / (2 * h)
    U, B, g = got[0, 0]
    # 32-bit rates: 1e-6 of each; the difference quotient's own error h^2
    assert abs(numeric - g @ d) <= 1e-3 * max(1.0, np.abs(g).max())
    for key, (U1, B1, g1) in got.items():
        assert np.array_equal(U1, U) and np.array_equal(B1, B), key
        assert np.max(np.abs(g1 - g)) <= 1e-11 * np.max(np.abs(g)), key


@pytest.mark.parametrize("n", [99, 100, 127, 128])
def test_gradient_on_both_sides_of_the_band_lines(n):
    """n envs of 8 tiles, around the numbers of tiles at which the adjoint and
    the forward change their row bands: the sum of the envs' own gradients,
    whose sums only run in another order."""
    batch = firegen.landscape_batch(105, [(128, 128)] * n)
    params = _params(105)
    rng = np.random.default_rng(10)
    seed_u = rng.normal(size=batch.n_cells)
    T, k = 6, 3

    def gradient(sub, cells):
        sim = fs.FireSim.from_batch(sub, params, seed=0)
        p = fs.make_params(params)
        p.unburnable_mask = sub.unburnable_mask
        U, B = sim.relaxed_init()
        ws = sim.relaxed_workspace(T, k)
        sim.relaxed_fwd(p, U, B, T, k, ws, "product")
        return U.cpu().numpy(), sim.relaxed_bwd(p, torch.from_numpy(seed_u[cells]).cuda(), None, T, k, ws,
                                                "product").cpu().numpy()

    U, g = gradient(batch, slice(0, batch.n_cells))
    whole = np.zeros(17)
    for a in range(0, n, 50):
        cells = slice(a * 128 * 128, min(n, a + 50) * 128 * 128)
        part, gp = gradient(batch.subset(range(a, min(n, a + 50))), cells)
        assert np.array_equal(part, U[cells])
        whole += gp
    assert np.max(np.abs(whole - g)) <= 1e-11 * np.max(np.abs(g))


@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("name", ["p_base", "alpha_gamma", "alpha_w1", "alpha_w2", "alpha_s", "veg"])
def test_parameters_that_are_not_finite(name, value):
    """Under such a parameter (a calibration that has diverged) edges without
    burning mass are no longer 0: the states are those of the dense forward,
    far from the fire too."""
    batch = firegen.landscape_batch(106, [(200, 300), (40, 70)], ign_range=(1, 1))
    params = _params(106)
    got = []
    for sparse in (0, 1):
        sim = fs.FireSim.from_batch(batch, params, seed=0)
        sim.set_plan(sparse=sparse)
        p = fs.make_params(params)
        p.unburnable_mask = batch.unburnable_mask
        if name == "veg":
            p.veg[1] = value
        else:
            setattr(p, name, value)
        U, B = sim.relaxed_init()
        sim.relaxed_fwd(p, U, B, 6, 3, sim.relaxed_workspace(6, 3), "product")
        got.append((U.cpu().numpy(), B.cpu().numpy()))
    for a, b in zip(*got):
        assert np.array_equal(a, b, equal_nan=True)
