"""The stochastic step around the lines where a call changes from one launch
per step over tiles to the bit-plane kernel, and from whole envs to parts: the
same bits on both sides, and no call much slower than the plain tiled plan.
"""
import numpy as np
import pytest
import torch

import firegen
import oracle

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")


def _params(seed, **kw):
    return firegen.Params(veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(seed))), **kw)


# every size alone and mixed: below and above 160 x 160 cells, whole envs, parts
@pytest.mark.parametrize("p_continue", [0.6, 0.95])
@pytest.mark.parametrize("sizes", [[(160, 160)], [(161, 160)], [(130, 200), (31, 33)], [(340, 331)],
                                   [(520, 512)], [(700, 644), (64, 64), (200, 208)]])
def test_calls_of_few_steps(sizes, p_continue):
    batch = firegen.landscape_batch(95, sizes, ign_range=(12, 12))
    params = _params(95, p_base=0.9, p_continue=p_continue)
    splits = [1, 2, 3, 4, 5, 7, 8, 9, 1, 16]
    act = firegen.random_actions(45, batch, sum(splits), p_none=0.5)
    ref = oracle.Sim(batch, params, seed=16)
    want = ref.step(sum(splits), actions=act, counts=True, threads=8, drop_mode=0, drop_radius=2)
    sim = fs.FireSim.from_batch(batch, params, seed=16)
    sim.set_drop(0, 2)
    got, t = [], 0
    for n in splits:
        got.append(sim.step(n, actions=torch.from_numpy(np.ascontiguousarray(act[t:t + n])), counts=True).cpu().numpy())
        t += n
    assert np.array_equal(np.concatenate(got), want)
    assert np.array_equal(sim.states.cpu().numpy(), ref.states)


@pytest.mark.parametrize("sizes", [[(150, 170)], [(170, 170)], [(340, 331)]])
def test_history_of_few_steps(sizes):
    batch = firegen.landscape_batch(96, sizes, ign_range=(12, 12))
    params = _params(96, p_base=0.9)
    ref = oracle.Sim(batch, params, seed=17)
    rows, want = ref.step(12, counts=True, threads=8, history=True)
    sim = fs.FireSim.from_batch(batch, params, seed=17)
    t = 0
    for n in (1, 3, 8):
        hist, cnt = sim.step_history(n, counts=True)
        assert np.array_equal(hist.cpu().numpy(), rows[t:t + n])
        assert np.array_equal(cnt.cpu().numpy(), want[t:t + n])
        t += n
    assert np.array_equal(sim.states.cpu().numpy(), rows[-1])


def _ms(sim, states, T, reps=5):
    best = float("inf")
    for _ in range(reps):
        sim.states.copy_(states)
        sim.t = 0
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        sim.step(T)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


# (one step of a large env took 30 times the tiled plan's time where its one
# workgroup copied the cells back, 100 steps of a long fire 2.7 times where one
# workgroup stepped it; half as much again leaves room for the clock)
@pytest.mark.parametrize("n,size,T,p_continue", [(1, (4096, 4096), 1, 0.5), (16, (1000, 1000), 1, 0.5),
                                                 (4, (512, 512), 100, 0.95), (64, (331, 331), 100, 0.95)])
def test_no_call_much_slower_than_tiles(n, size, T, p_continue):
    batch = firegen.landscape_batch(97, [size] * n, ign_range=(20, 20))
    sim = fs.FireSim.from_batch(batch, _params(97, p_base=0.9, p_continue=p_continue), seed=18)
    sim.step(40)
    states = sim.states.clone()
    took = _ms(sim, states, T)
    sim.set_plan(tile_rows=4, tile_width=64, skip_static=1, sparse=0)
    tiled = _ms(sim, states, T)
    assert took < 1.5 * tiled, (took, tiled)
