"""GPU parity of the relaxed kernels where a tile is walked by several waves
(row bands that meet in LDS) and where only the tiles within reach of the fire
run: against the fp64 oracle (tolerances of test_gpu_relaxed.py: U, B 1e-5,
gradient 1e-4 of its largest entry) and against the dense sweep (the same
states to the bit; the gradient's sums run in another order, so 1e-11 of its
largest entry)."""
import numpy as np
import pytest
import torch

import firegen
import oracle
from oracle import relaxed64

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")


def _params(seed, **kw):
    base = dict(p_base=0.5, alpha_w1=0.05, alpha_w2=0.12, alpha_s=3.0, alpha_gamma=1.1, p_continue=0.55,
                veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(seed))))
    base.update(kw)
    return firegen.Params(**base)


def _run(batch, params, Y, T, k, form, fwd_sparse, bwd_sparse, loss="iou"):
    sim = fs.FireSim.from_batch(batch, params, seed=0)
    p = fs.make_params(params)
    p.unburnable_mask = batch.unburnable_mask
    sim.set_plan(sparse=fwd_sparse)
    U, B = sim.relaxed_init()
    ws = sim.relaxed_workspace(T, k)
    ws.fill_(0xFF)  # NaNs: a state that is read without having been written shows
    sim.relaxed_fwd(p, U, B, T, k, ws, form)
    _, gU, _ = sim.relaxed_loss_any(loss, U, torch.from_numpy(Y).cuda(), scale=1.0 / batch.n_env)
    sim.set_plan(sparse=bwd_sparse)
    grad = sim.relaxed_bwd(p, gU, None, T, k, ws, form)
    return U.cpu().numpy(), B.cpu().numpy(), grad.cpu().numpy()


def _scar(batch, params, T):
    ref = oracle.Sim(batch, params, seed=5)
    ref.step(T, threads=8)
    return ((ref.states == firegen.BURNING) | (ref.states == firegen.BURNT)).astype(np.uint8)


@pytest.mark.parametrize("form", ["product", "exp"])
@pytest.mark.parametrize("per_cell", [False, True])
def test_bands_of_a_tile(form, per_cell):
    """Heights around the 2- and 4-row bands and the 32-row tile, widths around the 64-column strip."""
    sizes = [(1, 70), (2, 5), (4, 64), (5, 65), (8, 63), (31, 9), (32, 130), (33, 66), (36, 40), (67, 20)]
    batch = firegen.landscape_batch(91, sizes, per_cell_wind=per_cell, elev_max=60.0)
    params = _params(91)
    T, k = 18, 5
    Y = _scar(batch, params, T)
    U, B, grad = _run(batch, params, Y, T, k, form, 1, 1)
    Ys = [batch.env_view(Y, e).astype(bool) for e in range(batch.n_env)]
    theta = relaxed64.theta_from_params(params).astype(np.float32).astype(np.float64)
    _, g64, finals = relaxed64.loss_and_grad(batch, theta, T, Ys, cell_size=params.cell_size, form=form)
    for e in range(batch.n_env):
        assert np.max(np.abs(batch.env_view(U, e) - finals[e][0])) <= 1e-5
        assert np.max(np.abs(batch.env_view(B, e) - finals[e][1])) <= 1e-5
    assert np.max(np.abs(grad - g64)) <= 1e-4 * np.max(np.abs(g64))


@pytest.mark.parametrize("size,per_cell", [((700, 900), True), ((2048, 1100), False), ((64, 130), False)])
def test_reach_of_the_fire(size, per_cell):
    """States and gradient with only the tiles in reach against the dense
    sweep, and the plan changed between forward and backward."""
    batch = firegen.landscape_batch(92, [size, (40, 40)], per_cell_wind=per_cell, ign_range=(2, 2), elev_max=200.0)
    params = _params(92)
    T, k = 70, 8
    Y = _scar(batch, params, T)
    U0, B0, g0 = _run(batch, params, Y, T, k, "product", 0, 0)
    for fwd, bwd in ((1, 1), (1, 0), (0, 1)):
        U, B, g = _run(batch, params, Y, T, k, "product", fwd, bwd)
        assert np.array_equal(U, U0) and np.array_equal(B, B0), (fwd, bwd)
        assert np.max(np.abs(g - g0)) <= 1e-11 * np.max(np.abs(g0)), (fwd, bwd)


@pytest.mark.parametrize("p_continue,u", [(float("inf"), None), (float("nan"), None), (0.5, float("inf")),
                                          (0.5, float("nan"))])
def test_values_that_are_not_finite(p_continue, u):
    """0 times such a value is no 0: the sparse forward gives what the dense one gives, far from the fire too."""
    batch = firegen.landscape_batch(95, [(200, 300), (40, 70)], ign_range=(1, 1))
    params = _params(95, p_continue=p_continue)
    got = []
    for sparse in (0, 1):
        sim = fs.FireSim.from_batch(batch, params, seed=0)
        p = fs.make_params(params)
        p.unburnable_mask = batch.unburnable_mask
        sim.set_plan(sparse=sparse)
        U, B = sim.relaxed_init()
        if u is not None:
            U[7] = u
            U[200 * 300 - 9] = u
        ws = sim.relaxed_workspace(6, 3)
        sim.relaxed_fwd(p, U, B, 6, 3, ws, "product")
        got.append((U.cpu().numpy(), B.cpu().numpy()))
    for a, b in zip(*got):
        assert np.array_equal(a, b, equal_nan=True)
