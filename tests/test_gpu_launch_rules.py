"""Launch shapes chosen by size or by the tuner: which one runs, and that it leaves every bit alone."""
import json

import numpy as np
import pytest
import torch

from stag_inputs import fat_field_device, gaussian_source_device, random_su3_field_device

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


# more than 256 tiles of 1024 sites in all, so that every workgroup of the wide CG kernels walks several: 151 ragged
# ones for each of 3 right-hand sides, and 69 for each of 5 beside a single one
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_wide_cg_walks_are_the_general_iterations(gpu_lib, prec):
    from paper_1010_4782_amd.stagcg import cg_solve_batch

    dims, nrhs = (22, 18, 26, 30), 3
    print(f"wide CG walk {dims} x {nrhs} {prec}", flush=True)
    lat = setup(dims, 45, long_su3=True)
    b = gaussian_source_device(dims, 47, nrhs)
    mass = [0.2 + 0.2 * r for r in range(nrhs)]  # slots stop at different iterations
    out = []
    for profile in (0, 1000):
        hist = np.zeros((nrhs, 40, 2))
        x, info = lat.cg_solve(b, mass, prec=prec, profile=profile, history_len=40, history=hist)
        out.append((x, hist, [(i["iters"], i["n_reliable"], i["true_resid"]) for i in info]))
    assert torch.equal(out[0][0], out[1][0]) and out[0][2] == out[1][2]
    np.testing.assert_array_equal(out[0][1], out[1][1])
    shapes = [((14, 18, 26, 22), 5), ((2, 4, 4, 2), 2)]
    lats = [setup(d, 49 + i, long_su3=True) for i, (d, _) in enumerate(shapes)]
    bs = [gaussian_source_device(d, 51 + i, n) for i, (d, n) in enumerate(shapes)]
    out = []
    for profile in (0, 1000):
        xs, info = cg_solve_batch([(l, v, 0.3, None) for l, v in zip(lats, bs)], prec=prec, profile=profile)
        out.append((xs, [(i["iters"], i["n_reliable"], i["true_resid"]) for i in info]))
    assert all(torch.equal(u, v) for u, v in zip(out[0][0], out[1][0])) and out[0][1] == out[1][1]


def test_sweep_over_several_lattices_is_the_lattice_order(gpu_lib):
    """A batch whose largest slice passes 2 MiB sweeps t per XCD over all its lattices, slices that eight does not
    divide and a lattice smaller than the XCDs' shares among them; each solve has the bits of its solve alone in
    lattice order."""
    from paper_1010_4782_amd.stagcg import cg_solve_batch

    shapes = [((22, 18, 14, 6), 16), ((6, 10, 6, 10), 3), ((2, 2, 2, 2), 1)]
    print(f"sweep over {shapes}", flush=True)
    lats = [setup(d, 53 + i) for i, (d, _) in enumerate(shapes)]
    bs = [gaussian_source_device(d, 57 + i, n) for i, (d, n) in enumerate(shapes)]
    xs, info = cg_solve_batch([(l, b, 0.4, None) for l, b in zip(lats, bs)])
    k = 0
    for lat, b, x, (dims, n) in zip(lats, bs, xs, shapes):
        lat.set_dslash_shape("f64", n, 64, 1)
        y, one = lat.cg_solve(b, 0.4)
        lat.set_dslash_shape("f64", n, 0)
        assert torch.equal(x, y) and [i["iters"] for i in one] == [i["iters"] for i in info[k:k + n]], dims
        k += n


@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
@pytest.mark.parametrize("su3", [False, True])
def test_sweep_on_a_slab_is_the_whole_lattice(gpu_lib, prec, su3):
    """Slabs whose slices pass 2 MiB of colour vectors and whose z extent rules out z blocks: the XCD sweep, the
    single right-hand side in lattice order."""
    dims, nrhs = (28, 26, 22, 8), 18
    print(f"slab sweep {dims} x {nrhs} {prec} su3 {su3}", flush=True)
    lat = setup(dims, 61, precs=("f64", prec), long_su3=su3)
    S, Lt = dims[0] * dims[1] * dims[2] // 2, dims[3]
    assert S * nrhs * {"f64": 48, "f32": 24, "f16": 16}[prec] >= 2 << 20
    b = gaussian_source_device(dims, 63, nrhs)
    for par in (0, 1):
        ref = torch.cat([lat.dslash(b[r:r + 1].contiguous(), par, prec=prec) for r in range(nrhs)])
        for t0, lt in ((0, 2), (2, 6), (4, 4)):
            rows = torch.cat([torch.arange(((t0 + k) % Lt) * S, ((t0 + k) % Lt + 1) * S) for k in range(-3, lt + 3)])
            out = lat.dslash_slab(b[:, rows.cuda(), :].contiguous(), par, t0, lt, prec=prec)
            assert torch.equal(out, ref[:, t0 * S:(t0 + lt) * S, :]), (par, t0, lt)
