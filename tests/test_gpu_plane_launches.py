"""GPU parity of the bit-plane step kernel over batches whose envs differ so
much in shape that their launches have to be kept apart.
"""
import numpy as np
import pytest
import torch

import firegen
import oracle

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")


@pytest.mark.parametrize("series", [False, True])
@pytest.mark.parametrize("sizes", [[(6150, 4), (512, 512)], [(512, 512), (6150, 3), (31, 30)]])
def test_strip_and_square(sizes, series):
    """A strip (large planes, short list) and a square (long list) each fit a
    workgroup's LDS; the larger planes with the longer list do not (168140 of
    162304 bytes with 512 lanes)."""
    T = 40
    batch = firegen.landscape_batch(92, sizes, ign_range=(20, 20))
    params = firegen.Params(p_base=0.9, veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(92))))
    wind = firegen.wind_series(11, batch, T, speed_step=1.0, turn_step=0.3) if series else None
    ref = oracle.Sim(batch, params, seed=13)
    want = ref.step(T, counts=True, threads=8, **({"wind_env_series": wind} if series else {}))
    sim = fs.FireSim.from_batch(batch, params, seed=13)
    if series:
        sim.set_wind_series(env_series=torch.from_numpy(wind).cuda())
    got = sim.step(T, counts=True)
    assert np.array_equal(got.cpu().numpy(), want)
    assert np.array_equal(sim.states.cpu().numpy(), ref.states)


@pytest.mark.parametrize("mode", [None, 0])
@pytest.mark.parametrize("size", [(1, 32767), (1, 4100), (2, 9000), (3, 2500), (8000, 1), (4100, 2), (700, 33), (565, 565)])
def test_one_env_wide_or_tall(size, mode):
    """More groups or words per row than lanes, and more rows than lanes: the
    ends of the divisions that deal cells out to them; and a square that just
    fits a workgroup's LDS."""
    T = 40
    batch = firegen.landscape_batch(93, [size], ign_range=(30, 30))
    params = firegen.Params(p_base=0.9, veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(93))))
    act = None if mode is None else firegen.random_actions(47, batch, T, p_none=0.3)
    ref = oracle.Sim(batch, params, seed=14)
    want = ref.step(T, actions=act, counts=True, threads=8, drop_mode=mode or 0, drop_radius=2)
    sim = fs.FireSim.from_batch(batch, params, seed=14)
    sim.set_drop(mode or 0, 2)
    got = sim.step(T, actions=None if act is None else torch.from_numpy(act), counts=True)
    assert np.array_equal(got.cpu().numpy(), want)
    assert np.array_equal(sim.states.cpu().numpy(), ref.states)
