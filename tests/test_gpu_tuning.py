"""The autotuner over plans that run on the same kernel, and its cache."""
import numpy as np
import pytest

import firegen

pytestmark = pytest.mark.gpu

fs = pytest.importorskip("paper_2512_06102_amd")


def _sim(sizes, seed=107):
    params = firegen.Params(veg=tuple(float(v) for v in firegen.veg_table(np.random.default_rng(seed))))
    return fs.FireSim.from_batch(firegen.landscape_batch(seed, sizes), params, seed=0)


@pytest.mark.parametrize("sizes", [[(128, 128)] * 4, [(700, 640)]])
def test_plans_of_one_kernel_are_timed_once(sizes):
    """The tile shape of such plans does not matter: not chosen by noise."""
    sim = _sim(sizes)
    res = sim.autotune(T_probe=30, allow_skip=True, allow_sparse=True)
    same = [(p, ms) for p, ms in res if p["skip_static"] and p["sparse"] and not p["resident"]]
    assert len(same) == 8 and len({ms for _, ms in same}) == 1
    assert (same[0][0]["tile_rows"], same[0][0]["tile_width"]) == (4, 64)
    plan = sim.plan()
    if plan["sparse"] and plan["skip_static"] and not plan["resident"]:
        assert (plan["tile_rows"], plan["tile_width"]) == (4, 64)


def test_cache_lines_of_other_kernels_do_not_count(tmp_path):
    """Times in the cache hold for the kernels, and the table of rates, that
    they were taken with."""
    sizes = [(128, 128)] * 3
    cache = tmp_path / "plans.txt"
    tune = dict(T_probe=6, allow_skip=True, allow_sparse=True, cache_path=str(cache))
    assert not _sim(sizes).autotune_classes(**tune)[0]["from_cache"]
    assert _sim(sizes).autotune_classes(**tune)[0]["from_cache"]
    key, value = cache.read_text().splitlines()[0].split(" : ")
    older = " ".join(w for w in key.split() if not w.startswith(("kernels=", "table=")))
    assert older.endswith("allow_sparse=1") and older != key
    cache.write_text(older + " : 1 256 8 1 0 0 0.001\n")
    got = _sim(sizes).autotune_classes(**tune)[0]
    assert not got["from_cache"] and got["ms_per_step"] != pytest.approx(0.001)
    sim = _sim(sizes)
    sim.set_rate_table(False)
    assert not sim.autotune_classes(**tune)[0]["from_cache"]
