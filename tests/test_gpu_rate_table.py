"""The stochastic and RL steps under static wind without the table of ignition
rates: the same bits, from the rates worked out in the step.
"""
import numpy as np
import pytest
import torch

import firegen
import oracle

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")


def _params(seed, **kw):
    return firegen.Params(p_base=0.9, veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(seed))), **kw)


# one group per lane, scanned whole envs, parts; aligned and not; several kinds beside each other
@pytest.mark.parametrize("mode", [None, 0])
@pytest.mark.parametrize("per_cell", [False, True])
@pytest.mark.parametrize("sizes", [[(64, 64), (28, 28)], [(128, 160), (37, 53)], [(700, 644), (64, 64)]])
def test_steps_without_the_table(sizes, per_cell, mode):
    T = 40
    batch = firegen.landscape_batch(100, sizes, per_cell_wind=per_cell, ign_range=(12, 12))
    params = _params(100)
    act = None if mode is None else firegen.random_actions(46, batch, 2 * T, p_none=0.5)
    ref = oracle.Sim(batch, params, seed=21)
    want = ref.step(2 * T, actions=act, counts=True, threads=8, drop_mode=mode or 0, drop_radius=2)
    sim = fs.FireSim.from_batch(batch, params, seed=21)
    sim.set_drop(mode or 0, 2)
    got = []
    for k, on in enumerate((False, True)):  # and with it again for the second half
        sim.set_rate_table(on)
        a = None if act is None else torch.from_numpy(np.ascontiguousarray(act[k * T:(k + 1) * T]))
        got.append(sim.step(T, actions=a, counts=True).cpu().numpy())
    assert np.array_equal(np.concatenate(got), want)
    assert np.array_equal(sim.states.cpu().numpy(), ref.states)


@pytest.mark.parametrize("size,threads", [((28, 28), 256), ((60, 60), 1024)])
def test_history_without_the_table(size, threads):
    batch = firegen.landscape_batch(101, [size] * 8)
    params = _params(101)
    ref = oracle.Sim(batch, params, seed=22)
    rows, want = ref.step(40, counts=True, threads=8, history=True)
    sim = fs.FireSim.from_batch(batch, params, seed=22)
    sim.set_plan(resident=threads, sparse=1)
    sim.set_rate_table(False)
    hist, got = sim.step_history(40, counts=True)
    assert np.array_equal(hist.cpu().numpy(), rows)
    assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("single", [True, False])
@pytest.mark.parametrize("per_cell", [False, True])
def test_rl_steps_without_the_table(per_cell, single):
    sizes = [(20, 20)] * 5 + [(64, 64), (9, 36), (33, 32)]
    batch = firegen.landscape_batch(102, sizes, per_cell_wind=per_cell)
    rng = np.random.default_rng(4)
    acts = torch.from_numpy((rng.integers(0, 9, (20, len(sizes))) | (rng.integers(0, 2, (20, len(sizes))) << 4))
                            .astype(np.int32)).cuda()
    got = []
    for on in (True, False):
        sim = fs.FireSim.from_batch(batch, _params(102), seed=23)
        sim.set_rate_table(on)
        env = fs.RLEnv(sim, obs_radius=3, drop_radius=1, max_steps=15, single_launch=single)
        env.reset(episode=2)
        out = []
        for t in range(20):
            o, r, d = env.step(acts[t])
            out += [o.clone(), r.clone(), d.clone(), sim.states.clone(), env.agents.clone()]
        got.append([x.cpu().numpy() for x in out])
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_the_table_is_given_back(monkeypatch):
    """On request, and where a calibration's workspace would not fit beside it."""
    batch = firegen.landscape_batch(103, [(2048, 2048)])
    table = 32 * batch.n_cells

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    sim = fs.FireSim.from_batch(batch, _params(103), seed=24)
    held = free()
    sim.set_rate_table(False)
    assert free() >= held + table // 2
    sim.set_rate_table(True)
    assert free() <= held + table // 2
    empty, refused = torch.empty, []

    def first_refused(*args, **kw):
        if not refused:
            refused.append(args)
            raise torch.OutOfMemoryError("refused")
        return empty(*args, **kw)

    monkeypatch.setattr(torch, "empty", first_refused)
    ws = sim.relaxed_workspace(1, 1)
    monkeypatch.undo()
    assert refused and ws.numel() == refused[0][0]
    del ws
    torch.cuda.empty_cache()
    assert free() >= held + table // 2


@pytest.mark.parametrize("rl_step", [False, True])
def test_a_captured_step_keeps_the_table(rl_step, monkeypatch):
    """Its graph holds the table's address: it is not given back, neither on
    request nor for a workspace, and the replays stay right."""
    batch = firegen.landscape_batch(108, [(64, 64)] * 4)
    params = _params(108)
    sim = fs.FireSim.from_batch(batch, params, seed=25)
    env = fs.RLEnv(sim)
    acts = torch.zeros(4, dtype=torch.int32, device="cuda")
    if rl_step:
        env.reset(episode=1)
        env.step(acts)
    init = sim.states.clone()
    sim.t = 0
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        env.step(acts) if rl_step else sim.step(20)
    with pytest.raises(fs.SimError):
        sim.set_rate_table(False)
    empty = torch.empty

    def refused(*args, **kw):
        raise torch.OutOfMemoryError("refused")

    monkeypatch.setattr(torch, "empty", refused)
    with pytest.raises(torch.OutOfMemoryError):
        sim.relaxed_workspace(1, 1)
    monkeypatch.undo()
    assert torch.empty is empty
    if not rl_step:
        ref = oracle.Sim(batch, params, seed=25)
        ref.step(20, threads=4)
        for _ in range(3):
            sim.states.copy_(init)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(sim.states.cpu().numpy(), ref.states)
