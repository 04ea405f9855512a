"""Launch shapes chosen by size or by the tuner: which one runs, and that it leaves every bit alone."""
import json

import pytest
import torch

from stag_inputs import (fat_field, fat_field_device, gaussian_source, gaussian_source_device, random_su3_field,
                         random_su3_field_device)

pytestmark = pytest.mark.gpu
NAIK = -1.0 / 24.0


def setup(dims, seed, precs=("f64", "f32", "f16"), long_su3=False):
    from paper_1010_4782_amd.stagcg import Lattice

    lat = Lattice(dims)
    lat.load_links(fat_field_device(dims, seed), random_su3_field_device(dims, seed + 1), NAIK, precs=precs,
                   long_su3=long_su3)
    return lat


def saved_shape(tmp_path, key):
    from paper_1010_4782_amd.stagcg import tune_cache_save

    tune_cache_save(str(tmp_path / "table.json"))
    return json.loads((tmp_path / "table.json").read_text()).get(key)


def test_tuner_keeps_the_default_where_it_is_the_fastest(gpu_lib, tmp_path):
    """28 z planes rule out z blocks and 12 right-hand sides divide by 4: the default sweeps t per XCD (1108 us at
    28^3 x 96), which no settable shape does (1322 us)."""
    dims, nrhs = (28, 28, 28, 96), 12
    print(f"tuner {dims} x {nrhs}", flush=True)
    lat = setup(dims, 31, precs=("f64",))
    x = gaussian_source_device(dims, 33, nrhs)
    ref = lat.dslash(x, 1)
    best, timed = lat.tune_dslash("f64", nrhs)
    kept = saved_shape(tmp_path, "p0:28x28x28x96/12")
    assert kept == [64, 4, 0, 0, 1, 1], kept
    assert best[5] == min(t[5] for t in timed) and nrhs % best[1] == 0
    assert torch.equal(lat.dslash(x, 1), ref)
    lat.set_dslash_shape("f64", nrhs, 0)
    assert saved_shape(tmp_path, "p0:28x28x28x96/12") is None
