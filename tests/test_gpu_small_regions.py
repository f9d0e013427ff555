"""GPU parity of the bit-plane step kernel where an env is small enough that
every lane has one 4-cell group: no list is made, and the waves of a workgroup
meet once per step.  States, counts and history are bit-exact against the CPU
oracle.
"""
import numpy as np
import pytest
import torch

import firegen
import oracle

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")

# env and workgroup size; widths whose rows are whole 32-cell words and not
SHAPES = [((28, 28), 256), ((16, 60), 256), ((32, 60), 512), ((30, 52), 512), ((60, 60), 1024), ((64, 64), 1024)]
T = 120


def _pair(size, threads, mode, series, n_env=48):
    batch = firegen.landscape_batch(91, [size] * n_env)
    params = firegen.Params(p_base=0.7, p_continue=0.8,
                            veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(91))))
    act = None if mode is None else firegen.random_actions(44, batch, T, p_none=0.8)
    wind = firegen.wind_series(10, batch, T, speed_step=1.0, turn_step=0.3) if series else None
    sim = fs.FireSim.from_batch(batch, params, seed=12)
    sim.set_plan(resident=threads, sparse=1)
    sim.set_drop(mode or 0, 2)
    if series:
        sim.set_wind_series(env_series=torch.from_numpy(wind).cuda())
    ref = oracle.Sim(batch, params, seed=12)
    kw = dict(actions=act, counts=True, threads=8, drop_mode=mode or 0, drop_radius=2)
    if series:
        kw["wind_env_series"] = wind
    return sim, ref, None if act is None else torch.from_numpy(act).cuda(), kw


@pytest.mark.parametrize("series", [False, True])
@pytest.mark.parametrize("mode", [None, 1])
@pytest.mark.parametrize("size,threads", SHAPES)
def test_counts_of_every_step(size, threads, mode, series):
    """A fire that a few waves of many carry on: no wave's burning cells go
    uncounted, so no env stops before its fire is out."""
    sim, ref, act, kw = _pair(size, threads, mode, series)
    want = ref.step(T, **kw)
    got = sim.step(T, actions=act, counts=True)
    assert np.array_equal(got.cpu().numpy(), want)
    assert np.array_equal(sim.states.cpu().numpy(), ref.states)


@pytest.mark.parametrize("series", [False, True])
@pytest.mark.parametrize("mode", [None, 1])
@pytest.mark.parametrize("size,threads", SHAPES)
def test_history_of_every_step(size, threads, mode, series):
    """Row k is the state after step k, whichever wave steps the group that
    another one stores; and the counts beside it."""
    sim, ref, act, kw = _pair(size, threads, mode, series)
    rows, want = ref.step(T, history=True, **kw)
    hist, got = sim.step_history(T, actions=act, counts=True)
    assert np.array_equal(hist.cpu().numpy(), rows)
    assert np.array_equal(got.cpu().numpy(), want)
    assert np.array_equal(sim.states.cpu().numpy(), rows[-1])


@pytest.mark.parametrize("size,threads", [((136, 36), 1024), ((132, 52), 512), ((100, 200), 256), ((65, 33), 64)])
def test_lists_dealt_out_without_the_table(size, threads):
    """Envs just too large for that, under a series: the listed groups go to the
    waves several at a time, with fewer waves than lists and more."""
    batch = firegen.landscape_batch(94, [size] * 6, ign_range=(1, 6))
    params = firegen.Params(p_base=0.8, p_continue=0.7,
                            veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(94))))
    wind = firegen.wind_series(12, batch, T, speed_step=1.0, turn_step=0.3)
    ref = oracle.Sim(batch, params, seed=15)
    want = ref.step(T, counts=True, threads=8, wind_env_series=wind)
    sim = fs.FireSim.from_batch(batch, params, seed=15)
    if sim.n_cells // 6 <= 92 * 92 and size[1] % 4 == 0:
        sim.set_plan(resident=threads, sparse=1)
    sim.set_wind_series(env_series=torch.from_numpy(wind).cuda())
    got = sim.step(T, counts=True)
    assert np.array_equal(got.cpu().numpy(), want)
    assert np.array_equal(sim.states.cpu().numpy(), ref.states)
