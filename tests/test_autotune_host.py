"""Keys of the launch-shape cache (no device)."""
import numpy as np

from paper_1806_10251_amd import autotune, lbm

CAVITY = (lbm.WALL, lbm.WALL, lbm.WALL, lbm.LID)
CHANNEL = (lbm.INLET, lbm.OUTLET, lbm.WALL, lbm.WALL)
DUCT = (lbm.PERIODIC, lbm.PERIODIC, lbm.WALL, lbm.WALL)
MILL = (lbm.PERIODIC,) * 4


def test_configurations_that_run_other_kernels_have_other_keys():
    few = np.zeros((100, 200), np.uint8)
    few[40:60, 50:70] = 1
    many = (np.arange(20000).reshape(100, 200) % 3 == 0).astype(np.uint8)
    key = autotune.lattice_key
    keys = [key(200, 100, s, m, st, **v)
            for s in (CAVITY, CHANNEL, DUCT, MILL) for m in (None, few, many)
            for st in ("f16", "f32", "f64")
            for v in ({}, {"mrt": 1}, {"strain_fd": 1}, {"mrt": 1, "strain_fd": 1})]
    keys += [key(201, 100, CAVITY, None, "f32"), key(200, 101, CAVITY, None, "f32")]
    assert len(set(keys)) == len(keys)
    # a mask without solid nodes is no mask
    assert key(200, 100, CAVITY, 0 * few, "f32") == key(200, 100, CAVITY, None, "f32")


def test_choices_made_for_other_kernels_are_not_taken(monkeypatch, tmp_path):
    now = autotune.lattice_key(1024, 1024, CAVITY, None, "f32")
    assert now != "1024x1024:f32:obst0:outlet0"       # without a revision
    assert autotune.kernel_revision() in now
    monkeypatch.setattr(autotune, "kernel_revision", lambda: "other")
    assert autotune.lattice_key(1024, 1024, CAVITY, None, "f32") != now


def test_cached_choice_is_found_again(monkeypatch, tmp_path):
    monkeypatch.setenv("LBM_TUNE_CACHE", str(tmp_path / "t.json"))
    key = autotune.lattice_key(64, 48, DUCT, None, "f32", 1, 0)
    autotune._save_cache({key: {"shape": [8, 2], "table": {"[8, 2]": 1.5}}})
    assert autotune.tune_lattice(64, 48, DUCT, storage="f32", mrt=1) == ((8, 2), {(8, 2): 1.5})
