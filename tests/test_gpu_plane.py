"""GPU parity of the bit-plane step kernel (the default plans): whole envs at
the edges of its 32-cell words and 4-cell groups, envs cut into parts with a
halo, full group lists, and steps across the 32-step staging of drops and
counts.  States, counts and history are bit-exact against the CPU oracle.
"""
import numpy as np
import pytest
import torch

import firegen
import oracle

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")

PLAN = dict(tile_rows=4, tile_width=64, skip_static=1, sparse=1)


def _veg(seed):
    return tuple(float(v) for v in firegen.veg_table(np.random.default_rng(seed)))


def _run(batch, params, T, mode, splits=(), seed=5, series=None):
    """T steps on the GPU (split into calls) and on the oracle; drops of `mode`, or None."""
    act = None if mode is None else firegen.random_actions(41, batch, T, p_none=0.3)
    kw = {} if series is None else {"wind_env_series": series}
    ref = oracle.Sim(batch, params, seed=seed)
    want = ref.step(T, actions=act, counts=True, threads=8, drop_mode=mode or 0, drop_radius=3, **kw)
    sim = fs.FireSim.from_batch(batch, params, seed=seed)
    sim.set_plan(**PLAN)
    sim.set_drop(mode or 0, 3)
    if series is not None:
        sim.set_wind_series(env_series=torch.from_numpy(series).cuda())
    got, t = [], 0
    for n in list(splits) + [T - sum(splits)]:
        a = None if act is None else torch.from_numpy(np.ascontiguousarray(act[t:t + n]))
        got.append(sim.step(n, actions=a, counts=True).cpu().numpy())
        t += n
    assert np.array_equal(sim.states.cpu().numpy(), ref.states)
    assert np.array_equal(np.concatenate(got), want)


WORDS = [(33, 31), (1, 1), (64, 65), (5, 32), (70, 96), (40, 127), (9, 129), (256, 4), (3, 260)]


@pytest.mark.parametrize("mode", [None, 0, 1])
@pytest.mark.parametrize("sizes", [WORDS, [(64, 64), (64, 32), (128, 160)]])
def test_word_edges(sizes, mode):
    batch = firegen.landscape_batch(81, sizes)
    _run(batch, firegen.Params(p_base=0.9, veg=_veg(81)), 70, mode, splits=(1, 32))


@pytest.mark.parametrize("mode,splits", [(None, ()), (None, (1, 16)), (0, (17,)), (1, ())])
@pytest.mark.parametrize("size", [(700, 640), (130, 4100), (601, 603)])
def test_parts_with_halo(size, mode, splits):
    """Envs too large for one workgroup: parts step 24 at a time with a halo."""
    batch = firegen.landscape_batch(82, [size, (65, 129)], ign_range=(40, 40))
    _run(batch, firegen.Params(p_base=1.0, p_continue=0.7, veg=_veg(82)), 60, mode, splits=splits)


@pytest.mark.parametrize("sizes", [[(128, 128)], [(90, 61), (61, 90)], [(700, 660)]])
def test_more_groups_than_the_list(sizes):
    """A checkerboard of fire: every group needs work, more than a list holds."""
    batch = firegen.landscape_batch(83, sizes)
    params = firegen.Params(p_base=0.05, p_continue=0.95, veg=_veg(83))
    st = firegen.dense_front_states(batch)
    ref = oracle.Sim(batch, params, seed=6)
    ref.states[:] = st
    want = ref.step(9, counts=True, threads=8)
    sim = fs.FireSim.from_batch(batch, params, seed=6)
    sim.set_plan(**PLAN)
    sim.states.copy_(torch.from_numpy(st))
    got = sim.step(9, counts=True).cpu().numpy()
    assert np.array_equal(sim.states.cpu().numpy(), ref.states)
    assert np.array_equal(got, want)


def test_wind_series_without_the_table():
    batch = firegen.landscape_batch(84, [(128, 128), (45, 67), (640, 644)], ign_range=(8, 8))
    series = firegen.wind_series(9, batch, 50, speed_step=1.0, turn_step=0.3)
    _run(batch, firegen.Params(p_base=0.8, veg=_veg(84)), 50, 1, splits=(33,), series=series)


@pytest.mark.parametrize("mode", [None, 0, 1])
def test_history_rows(mode):
    """Every state of 40 steps from one launch, odd widths included."""
    batch = firegen.landscape_batch(85, [(64, 64), (37, 53), (128, 128)])
    params = firegen.Params(p_base=0.9, veg=_veg(85))
    act = None if mode is None else firegen.random_actions(42, batch, 40, p_none=0.5)
    ref = oracle.Sim(batch, params, seed=7)
    rows, want = ref.step(40, actions=act, counts=True, threads=8, drop_mode=mode or 0, drop_radius=2, history=True)
    sim = fs.FireSim.from_batch(batch, params, seed=7)
    sim.set_plan(**PLAN)
    sim.set_drop(mode or 0, 2)
    hist, cnt = sim.step_history(40, actions=None if act is None else torch.from_numpy(act), counts=True)
    assert np.array_equal(hist.cpu().numpy(), rows)
    assert np.array_equal(cnt.cpu().numpy(), want)
    assert np.array_equal(sim.states.cpu().numpy(), rows[-1])


@pytest.mark.parametrize("per_cell", [False, True])
def test_rl_step_shapes(per_cell):
    """The one-launch RL step against the separate launches on envs whose
    planes leave room for fewer waves per workgroup, a last workgroup that is
    not full, and envs of one word and of several."""
    sizes = [(1400, 4), (20, 20), (4, 1000), (64, 64), (9, 36), (33, 32), (1, 4)]
    batch = firegen.landscape_batch(86, sizes, per_cell_wind=per_cell)
    params = firegen.Params(p_base=0.9, veg=_veg(86))
    rng = np.random.default_rng(3)
    acts = torch.from_numpy((rng.integers(0, 9, (25, len(sizes))) | (rng.integers(0, 2, (25, len(sizes))) << 4))
                            .astype(np.int32)).cuda()
    got = []
    for single in (True, False):
        sim = fs.FireSim.from_batch(batch, params, seed=9)
        env = fs.RLEnv(sim, obs_radius=4, drop_radius=2, water_capacity=9, max_steps=20, single_launch=single)
        env.reset(episode=2)
        out = []
        for t in range(25):
            o, r, d = env.step(acts[t])
            out += [o.clone(), r.clone(), d.clone(), sim.states.clone(), env.agents.clone()]
        got.append([x.cpu().numpy() for x in out])
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("mode", [None, 0])
def test_launches_beside_each_other(mode, graph):
    """Envs of two kinds, which step beside each other, on a stream of the
    caller's: calls of few and of many steps without a wait in between (with
    `graph`, from captures, where they step in order)."""
    splits = (3, 4, 5, 4, 30)
    batch = firegen.landscape_batch(87, [(700, 640), (65, 129), (40, 33)], ign_range=(40, 40))
    params = firegen.Params(p_base=1.0, p_continue=0.7, veg=_veg(87))
    act = None if mode is None else firegen.random_actions(43, batch, sum(splits), p_none=0.3)
    ref = oracle.Sim(batch, params, seed=8)
    want = ref.step(sum(splits), actions=act, counts=True, threads=8, drop_mode=0, drop_radius=3)
    sim = fs.FireSim.from_batch(batch, params, seed=8)
    sim.set_plan(**PLAN, graph=graph)
    sim.set_drop(0, 3)
    acts = None if act is None else torch.from_numpy(act).cuda()
    got, t = [], 0
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        for n in splits:
            got.append(sim.step(n, actions=None if acts is None else acts[t:t + n], counts=True).clone())
            t += n
        states = sim.states.clone()
    stream.synchronize()
    assert np.array_equal(states.cpu().numpy(), ref.states)
    assert np.array_equal(torch.cat(got).cpu().numpy(), want)
