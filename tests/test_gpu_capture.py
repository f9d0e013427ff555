"""sim_step captured into a caller's graph: nothing is allocated, copied or
waited for in the call, whatever plan was set before it.  Every replay, with
eager work between them, gives the oracle's states and counts.
"""
import numpy as np
import pytest
import torch

import firegen
import oracle

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")

T = 30


def _params(seed):
    return firegen.Params(p_base=0.9, veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(seed))))


def _replays(sim, batch, params, seed, n=3):
    ref = oracle.Sim(batch, params, seed=seed)
    want = ref.step(T, counts=True, threads=8)
    init = sim.states.clone()
    other = fs.FireSim.from_batch(firegen.landscape_batch(5, [(64, 64)]), params, seed=1)
    counts = torch.zeros((T, batch.n_env), dtype=torch.int32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    sim.t = 0
    with torch.cuda.graph(graph):
        counts.copy_(sim.step(T, counts=True))
    for _ in range(n):
        sim.states.copy_(init)
        counts.zero_()
        other.step(3)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(sim.states.cpu().numpy(), ref.states)
        assert np.array_equal(counts.cpu().numpy(), want)


@pytest.mark.parametrize("plan", [dict(resident=256, sparse=1), dict(tile_rows=8, tile_width=128, skip_static=1),
                                  dict(tile_rows=4, tile_width=64, skip_static=1, sparse=0),
                                  dict(tile_rows=4, tile_width=64, skip_static=1, sparse=1)])
def test_first_step_after_set_plan(plan):
    batch = firegen.landscape_batch(98, [(64, 64), (40, 52), (20, 88)])
    params = _params(98)
    sim = fs.FireSim.from_batch(batch, params, seed=19)
    sim.set_plan(**plan)
    _replays(sim, batch, params, 19)


def test_first_step_of_mixed_envs():
    batch = firegen.landscape_batch(99, [(700, 644), (64, 64), (200, 208)], ign_range=(20, 20))
    params = _params(99)
    _replays(fs.FireSim.from_batch(batch, params, seed=20), batch, params, 20)
