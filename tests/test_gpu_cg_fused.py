"""CG iterations with the scalar steps inside the vector kernels (small problems) against the general
launches, which a sampled profile keeps: the same bits, counts and recorded coefficients."""
import numpy as np
import pytest
import torch

from stag_inputs import fat_field, gaussian_source, random_su3_field

pytestmark = pytest.mark.gpu
NAIK = -1.0 / 24.0


def setup(dims, seed):
    from paper_1010_4782_amd.stagcg import Lattice

    lat = Lattice(dims)
    lat.load_links(torch.from_numpy(fat_field(dims, seed)).cuda(), torch.from_numpy(random_su3_field(dims, seed + 1)).cuda(),
                   NAIK, precs=("f64", "f32", "f16"))
    return lat


@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
# 8 sites; one and two r tiles with a ragged last one; 1024 <d, Ad> partials, the most the fused path takes
@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 1), ((4, 4, 4, 8), 3), ((6, 6, 4, 10), 4), ((16, 16, 16, 32), 1)])
def test_fused_iterations_are_the_general_ones(gpu_lib, dims, nrhs, prec):
    print(f"fused CG {dims} x {nrhs} {prec}", flush=True)
    lat = setup(dims, 91)
    b = gaussian_source(dims, 92, nrhs)
    if nrhs > 2:
        b[1] = 0.0  # a slot that never runs
    bt = torch.from_numpy(b).cuda()
    mass = [0.08 + 0.15 * r for r in range(nrhs)]  # slots stop at different iterations
    out = []
    for profile in (0, 1000):
        hist = np.zeros((nrhs, 40, 2))
        x, info = lat.cg_solve(bt, mass, prec=prec, profile=profile, history_len=40, history=hist)
        out.append((x, hist, [(i["iters"], i["restarts"], i["n_reliable"], i["status"], i["true_resid"]) for i in info]))
    assert torch.equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1], out[1][1])
    assert out[0][2] == out[1][2]
    assert all(i[4] <= 1e-10 for i in out[0][2])


def test_fused_iteration_cap(gpu_lib):
    """max_iter reached inside a batch of iterations: the last x update is applied, the solve reports it."""
    print("fused CG iteration cap", flush=True)
    dims = (4, 4, 4, 8)
    lat = setup(dims, 93)
    bt = torch.from_numpy(gaussian_source(dims, 94, 2)).cuda()
    out = []
    for profile in (0, 1000):
        x, info = lat.cg_solve(bt, [0.01, 0.5], max_iter=7, max_restarts=0, raise_on_fail=False, profile=profile)
        out.append((x, [(i["iters"], i["status"], i["true_resid"]) for i in info]))
    assert torch.equal(out[0][0], out[1][0])
    assert out[0][1] == out[1][1]
    assert out[0][1][0][0] == 7 and out[0][1][0][1] == 5


def test_fused_batch_of_lattices(gpu_lib):
    from paper_1010_4782_amd.stagcg import cg_solve_batch

    print("fused CG batch", flush=True)
    shapes = [((4, 4, 4, 8), 2), ((6, 4, 4, 6), 1), ((8, 8, 8, 8), 3)]
    lats = [setup(d, 95 + i) for i, (d, _) in enumerate(shapes)]
    bs = [torch.from_numpy(gaussian_source(d, 100 + i, n)).cuda() for i, (d, n) in enumerate(shapes)]
    out = []
    for profile in (0, 1000):
        xs, info = cg_solve_batch([(l, b, 0.1, None) for l, b in zip(lats, bs)], prec="f16", profile=profile)
        out.append((xs, [(i["iters"], i["n_reliable"], i["true_resid"]) for i in info]))
    assert all(torch.equal(a, b) for a, b in zip(out[0][0], out[1][0]))
    assert out[0][1] == out[1][1]


# 2048 and 1064 partials of <d, Ad>, more than the one-tile kernels take: even, and ragged tiles with a slot that
# never runs; slots stop at different iterations
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
@pytest.mark.parametrize("dims,nrhs", [((16, 16, 16, 64), 1), ((18, 10, 14, 54), 3)])
def test_wide_iterations_are_the_general_ones(gpu_lib, dims, nrhs, prec):
    test_fused_iterations_are_the_general_ones(gpu_lib, dims, nrhs, prec)


def test_wide_batch_of_lattices(gpu_lib):
    from paper_1010_4782_amd.stagcg import cg_solve_batch

    print("wide CG batch", flush=True)
    shapes = [((2, 4, 4, 2), 2), ((16, 16, 16, 40), 2), ((6, 10, 4, 6), 3)]  # one of them a single tile
    lats = [setup(d, 105 + i) for i, (d, _) in enumerate(shapes)]
    bs = [torch.from_numpy(gaussian_source(d, 110 + i, n)).cuda() for i, (d, n) in enumerate(shapes)]
    out = []
    for profile in (0, 1000):
        xs, info = cg_solve_batch([(l, b, 0.2, None) for l, b in zip(lats, bs)], prec="f16", profile=profile)
        out.append((xs, [(i["iters"], i["n_reliable"], i["true_resid"]) for i in info]))
    assert all(torch.equal(a, b) for a, b in zip(out[0][0], out[1][0]))
    assert out[0][1] == out[1][1]
