"""What the RL layer takes from the caller's memory: agents set off the grid
(in one launch as in the separate ones, such an agent spends its water, wets no
cell and sees only what lies on the grid), and states at any address.
"""
import numpy as np
import pytest
import torch

import firegen

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")

H, W = 20, 24
# on the grid, next to it, and far off it on one side, two sides and both ends of the types
POSITIONS = [(3, 5), (19, 23), (-1, 4), (4, -1), (-1, -1), (20, 3), (3, 24), (20, 24), (-100, -100), (-100, 500),
             (500, -100), (500, 500), (40000, 2), (2, 70000), (2, 65540), (70000, 70000), (-70000, 3)]


@pytest.mark.parametrize("drop_radius", [1, 30, 255])
def test_agents_off_the_grid(drop_radius):
    batch = firegen.landscape_batch(93, [(H, W)] * len(POSITIONS), ign_range=(8, 8))
    params = firegen.Params(p_base=0.9, p_continue=0.8,
                            veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(93))))
    got = []
    for single in (True, False):
        sim = fs.FireSim.from_batch(batch, params, seed=14)
        env = fs.RLEnv(sim, obs_radius=3, drop_radius=drop_radius, water_capacity=9, max_steps=20,
                       single_launch=single)
        env.reset(episode=1)
        out = []
        for t in range(6):
            env.agents[:, :2] = torch.tensor(POSITIONS, dtype=torch.int32, device="cuda")
            # valve open, no move; the last step moves onto the grid
            act = torch.full((len(POSITIONS),), 16 + (1 if t == 5 else 0), dtype=torch.int32, device="cuda")
            o, r, d = env.step(act)
            out += [o.clone(), r.clone(), d.clone(), sim.states.clone(), env.agents.clone()]
        got.append([x.cpu().numpy() for x in out])
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_reset_of_states_at_any_address(shift):
    """Envs of a multiple of 4 cells whose widths are none: byte steps, and a
    reset that must not assume 4-byte words either."""
    batch = firegen.landscape_batch(94, [(8, 6), (20, 10), (4, 3)])
    params = firegen.Params(p_base=0.9, veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(94))))
    got = []
    for at in (0, shift):
        sim = fs.FireSim.from_batch(batch, params, seed=15)
        store = torch.full((sim.n_cells + 8,), 9, dtype=torch.uint8, device="cuda")
        store[at:at + sim.n_cells].copy_(sim.states)
        sim.states = store[at:at + sim.n_cells]
        env = fs.RLEnv(sim, obs_radius=2, drop_radius=1)
        obs, _ = env.reset(episode=4)
        out = [obs.clone(), sim.states.clone()]
        o, r, d = env.step(torch.zeros(3, dtype=torch.int32, device="cuda"))
        out += [o.clone(), r.clone(), d.clone(), sim.states.clone()]
        assert int((store == 9).sum()) == 8
        got.append([x.cpu().numpy() for x in out])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
