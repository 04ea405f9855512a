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


def test_time_streaming_call_fills_its_table_once(gpu_lib):
    """The nodes a stream capture records of a call with a pinned time-streaming shape (the graph is never
    launched): the input's conversion, one copy of the table, the operator, the output's conversion."""
    import ctypes as C

    dims, nrhs = (4, 4, 8, 4), 8
    print(f"time-streaming table {dims} x {nrhs}", flush=True)
    lat = setup(dims, 35, precs=("f64", "f16"))
    x = gaussian_source_device(dims, 36, nrhs)
    ref = lat.dslash(x, 1, prec="f16")
    lat.set_dslash_shape("f16", nrhs, 64, 8, 0, 2, 1)
    out = lat.dslash(x, 1, prec="f16")  # its workspace and the ring exist from here on
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    hip = gpu_lib  # the HIP runtime that the library is linked with
    hip.hipGetLastError.argtypes = []
    hip.hipStreamBeginCapture.argtypes = [C.c_void_p, C.c_int]
    hip.hipStreamEndCapture.argtypes = [C.c_void_p, C.POINTER(C.c_void_p)]
    hip.hipGraphGetNodes.argtypes = [C.c_void_p, C.c_void_p, C.POINTER(C.c_size_t)]
    hip.hipGraphDestroy.argtypes = [C.c_void_p]
    side = torch.cuda.Stream()
    graph, n = C.c_void_p(), C.c_size_t(0)
    assert hip.hipStreamBeginCapture(side.cuda_stream, 2) == 0  # relaxed mode
    lat.dslash(x, 1, prec="f16", out=out, stream=side)
    assert hip.hipStreamEndCapture(side.cuda_stream, C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    lat.set_dslash_shape("f16", nrhs, 0)
    lat.close()
    hip.hipGetLastError()  # waiting for an event whose record was captured is an error that nothing else should see
    assert n.value == 4, n.value


# z blocks below 2 MiB of colour vectors per slice: one or two per lane from 3 x 2^18 sites on; not where the sites
# are a power of two, not with four, nor z extents that 8 does not divide
@pytest.mark.parametrize("dims,nrhs,su3,order", [((32, 32, 32, 48), 1, True, 1), ((32, 32, 32, 46), 1, True, 0),
                                                 ((32, 32, 24, 64), 2, False, 1), ((32, 32, 24, 62), 2, False, 0),
                                                 ((32, 32, 32, 64), 1, False, 0), ((32, 32, 32, 64), 2, True, 0),
                                                 ((32, 32, 24, 64), 4, False, 0), ((16, 16, 16, 384), 1, False, 1),
                                                 ((32, 32, 28, 56), 2, True, 0)])
def test_f16_tile_order_by_size(gpu_lib, dims, nrhs, su3, order):
    print(f"FP16 tile order {dims} x {nrhs} su3 {su3}", flush=True)
    lat = setup(dims, 37, precs=("f64", "f16"), long_su3=su3)
    x = gaussian_source_device(dims, 39, nrhs)
    _, info = lat.cg_solve(x, 0.5, prec="f16", max_iter=1, max_restarts=0, raise_on_fail=False)
    assert info[0]["dslash_order"] == order
    out = lat.dslash(x, 1, prec="f16")
    lat.set_dslash_shape("f16", nrhs, 64, 1)
    assert torch.equal(lat.dslash(x, 1, prec="f16"), out)
    lat.set_dslash_shape("f16", nrhs, 0)


# an FP64 launch of at most 1024 waves is not split beyond that; waves at 4, 2 and 1 per lane: 324, 648, 1296; 972,
# 1944; 4, 8, 16; 1536, 3072; -, 1024, 2048
@pytest.mark.parametrize("dims,nrhs,per_lane", [((12, 12, 12, 12), 8, 2), ((12, 12, 12, 12), 24, 4), ((4, 4, 4, 2), 8, 1),
                                                ((16, 16, 16, 48), 4, 2), ((16, 16, 16, 32), 2, 2)])
def test_f64_right_hand_sides_per_lane(gpu_lib, dims, nrhs, per_lane):
    print(f"FP64 per lane {dims} x {nrhs}", flush=True)
    lat = setup(dims, 41, precs=("f64",))
    x = gaussian_source_device(dims, 43, nrhs)
    _, info = lat.cg_solve(x, 0.5, max_iter=1, max_restarts=0, raise_on_fail=False)
    assert info[0]["dslash_rhs"] == per_lane
    out = lat.dslash(x, 1)
    for r in (0, nrhs - 1):
        assert torch.equal(lat.dslash(x[r:r + 1].contiguous(), 1)[0], out[r])
