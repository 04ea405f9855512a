"""GPU parity of the network preconditioner and of flexible CG against the oracle."""
import os

import numpy as np
import pytest
import torch

from oracle import quant
from oracle.cg import true_residual
from oracle.dslash import apply_m
from oracle.net import folded_fat, init_weights, loss_and_grads, net_forward
from stag_inputs import fat_field, gaussian_source, random_su3_field

pytestmark = pytest.mark.gpu
NAIK = -1.0 / 24.0


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def fp32_bound(Ft32, W32, r32, dims):
    """Elementwise bound on |GPU - oracle| (real and imaginary part each) for the FP32 network on the same
    FP32 links, weights and input.  Every real output of a layer is a sum of at most
    n = 9 directions x C_in channels x 3 colours x 4 real products (w U v), accumulated in binary32:
    its error is at most gamma_n = n u / (1 - n u), u = 2^-24, times the sum of the terms' magnitudes.
    That sum is bounded by the same network run on the magnitudes |Re| + |Im| of links, weights and
    input, in FP64; the layers add their errors, so the output bound is layers x gamma_n x that run."""
    mag = lambda a: (np.abs(a.real) + np.abs(a.imag)).astype(np.complex128)
    cin = max(w.shape[2] for w in W32)
    n = 9 * cin * 3 * 4
    gamma = n * 2.0**-24 / (1 - n * 2.0**-24)
    m = net_forward(mag(Ft32), [mag(w) for w in W32], mag(r32), dims).real
    return len(W32) * gamma * m


def assert_within(out, ref, bound):
    assert np.all(np.abs(out.real - ref.real) <= bound) and np.all(np.abs(out.imag - ref.imag) <= bound), \
        f"max excess {np.max(np.maximum(np.abs(out.real - ref.real), np.abs(out.imag - ref.imag)) / bound):.3g} of the bound"


def setup(dims, seed):
    from paper_1010_4782_amd.stagcg import Lattice

    fat, lng = fat_field(dims, seed), random_su3_field(dims, seed + 1)
    lat = Lattice(dims)
    lat.load_links(torch.from_numpy(fat).cuda(), torch.from_numpy(lng).cuda(), NAIK, precs=("f64", "f32"))
    return lat, fat, lng


@pytest.mark.parametrize("dims,channels", [((4, 4, 4, 8), [1, 4, 4, 1]), ((6, 4, 4, 6), [1, 8, 8, 8, 1]),
                                           ((4, 2, 6, 4), [1, 2, 1]), ((4, 4, 4, 4), [1, 1])])
def test_net_forward_matches_oracle(gpu_lib, dims, channels):
    """FP32 network vs the FP64 oracle on FP32-rounded links and weights, every element within the
    rounding bound of fp32_bound."""
    from paper_1010_4782_amd.stagcg import Net

    print(f"net forward {dims} {channels}", flush=True)
    lat, fat, _ = setup(dims, 3)
    net = Net(lat, layers=len(channels) - 1, channels=max(channels[1:-1] or [1]))
    W = init_weights(channels, 4, scale=1.0)
    W32 = [quant.to_f32(w) for w in W]
    net.set_weights(W32)
    got = [g for g in net.get_weights()]
    for a, b in zip(got, W32):
        np.testing.assert_array_equal(a, b)
    r = gaussian_source(dims, 5, 2)
    out = net.apply(torch.from_numpy(r).cuda()).cpu().numpy()
    Ft = quant.to_f32(folded_fat(fat, dims))
    for k in range(2):
        r32 = quant.to_f32(r[k])
        ref = net_forward(Ft, W32, r32, dims)
        assert_within(out[k], ref, fp32_bound(Ft, W32, r32, dims))


@pytest.mark.parametrize("dims,width", [((4, 4, 2, 6), 4), ((6, 4, 2, 6), 8)])
def test_net_loss_and_gradients_match_oracle(gpu_lib, dims, width):
    """Loss and weight gradients; widths 4 and 8 run the matrix-core layer and gradient kernels
    (6x4x2x6: 144 sites per parity, a ragged last wave)."""
    from paper_1010_4782_amd.stagcg import Net

    print(f"net loss/grad {dims} width {width}", flush=True)
    lat, fat, _ = setup(dims, 7)
    channels = [1, width, width, 1]
    net = Net(lat, layers=3, channels=width)
    W32 = [quant.to_f32(w) for w in init_weights(channels, 8, scale=1.0)]
    net.set_weights(W32)
    b = gaussian_source(dims, 9, 3)
    x = gaussian_source(dims, 10, 3)
    loss, grads = net.loss_grad(torch.from_numpy(b).cuda(), torch.from_numpy(x).cuda())
    Ft = quant.to_f32(folded_fat(fat, dims))
    L, G = loss_and_grads(Ft, W32, [(quant.to_f32(b[i]), x[i]) for i in range(3)], dims)
    assert abs(loss - L) <= 1e-5 * abs(L)
    for g, gr in zip(grads, G):
        assert rel(g, gr) <= 1e-4


@pytest.mark.parametrize("dims,width", [((2, 6, 6, 4), 8), ((6, 2, 2, 10), 2), ((10, 14, 18, 26), 4), ((14, 18, 22, 26), 2)])
def test_net_uneven_ranges_match_oracle(gpu_lib, dims, width):
    """Time slices that the eight XCD ranges divide unevenly (36, 12 and 1260 sites per parity), a ragged last
    wave, and (10x14x18x26, 512 chunks of 64 sites) gradient waves with a second chunk: forward within
    fp32_bound, loss and gradients to the bounds of the test above."""
    from paper_1010_4782_amd.stagcg import Net

    print(f"net uneven ranges {dims} width {width}", flush=True)
    lat, fat, _ = setup(dims, 27)
    channels = [1, width, width, 1]
    net = Net(lat, layers=3, channels=width)
    W32 = [quant.to_f32(w) for w in init_weights(channels, 28, scale=1.0)]
    net.set_weights(W32)
    b, x = gaussian_source(dims, 29, 1), gaussian_source(dims, 30, 1)
    Ft = quant.to_f32(folded_fat(fat, dims))
    b32 = quant.to_f32(b[0])
    out = net.apply(torch.from_numpy(b).cuda()).cpu().numpy()
    assert_within(out[0], net_forward(Ft, W32, b32, dims), fp32_bound(Ft, W32, b32, dims))
    loss, grads = net.loss_grad(torch.from_numpy(b).cuda(), torch.from_numpy(x).cuda())
    L, G = loss_and_grads(Ft, W32, [(b32, x[0])], dims)
    assert abs(loss - L) <= 1e-5 * abs(L)
    for g, gr in zip(grads, G):
        assert rel(g, gr) <= 1e-4


def test_net_residual_loss_matches_oracle(gpu_lib):
    from paper_1010_4782_amd.stagcg import Net

    print("net residual loss/grad", flush=True)
    dims = (4, 4, 2, 6)
    lat, fat, lng = setup(dims, 17)
    channels = [1, 2, 2, 1]
    net = Net(lat, layers=3, channels=2)
    W32 = [quant.to_f32(w) for w in init_weights(channels, 18, scale=1.0)]
    net.set_weights(W32)
    b = gaussian_source(dims, 19, 2)
    m = 0.3
    loss, grads = net.loss_grad(torch.from_numpy(b).cuda(), torch.from_numpy(b).cuda(), loss="residual", mass=m)
    Ft = quant.to_f32(folded_fat(fat, dims))
    A = lambda v: apply_m(fat, lng, v, dims, m)
    # the network's FP32 output enters M in FP64 on both sides
    L, G = loss_and_grads(Ft, W32, [(quant.to_f32(b[i]), None) for i in range(2)], dims, apply_m=A)
    assert abs(loss - L) <= 1e-5 * abs(L)
    for g, gr in zip(grads, G):
        assert rel(g, gr) <= 1e-4


def test_fcg_identity_network_is_cg(gpu_lib):
    """A one-layer network with W_0 = 1 is the identity: FCG then follows plain CG."""
    from paper_1010_4782_amd.stagcg import Net

    print("fcg identity", flush=True)
    dims = (8, 8, 8, 8)
    lat, fat, lng = setup(dims, 11)
    net = Net(lat, layers=1, channels=1)
    W = np.zeros((9, 1, 1), complex)
    W[0, 0, 0] = 1.0
    net.set_weights([W])
    m = 0.05
    b = gaussian_source(dims, 12)
    bt = torch.from_numpy(b).cuda()
    x0, i0 = lat.cg_solve(bt, m)
    x1, i1 = lat.cg_solve(bt, m, net=net, stall_window=10)
    assert i1[0]["converged"] == 1 and i1[0]["fell_back"] == 0
    assert abs(i1[0]["iters"] - i0[0]["iters"]) <= max(5, 0.02 * i0[0]["iters"])
    A = lambda v: apply_m(fat, lng, v, dims, m)
    assert true_residual(A, b[0], x1.cpu().numpy()[0]) <= 1.05e-10
    # the same with the operator in FP32 and FP16 storage: reliable updates bring the true residual down
    for prec in ("f32", "f16"):
        lat.load_links(torch.from_numpy(fat).cuda(), torch.from_numpy(lng).cuda(), NAIK, precs=("f64", "f32", prec))
        xm, im = lat.cg_solve(bt, m, prec=prec)
        xf, jf = lat.cg_solve(bt, m, prec=prec, net=net, stall_window=10)
        assert jf[0]["converged"] == 1 and jf[0]["fell_back"] == 0, (prec, jf[0])
        assert jf[0]["n_reliable"] >= 1
        assert jf[0]["iters"] <= 1.5 * im[0]["iters"] + 10, (prec, jf[0]["iters"], im[0]["iters"])
        assert true_residual(A, b[0], xf.cpu().numpy()[0]) <= 1.05e-10


def test_fcg_trained_network_and_forced_fallback(gpu_lib):
    """Train on solver-made pairs; FCG with the network reaches the true residual; a stall threshold
    that no progress can meet forces the plain-CG fallback, which still converges."""
    from paper_1010_4782_amd.stagcg import Net

    print("fcg trained + fallback", flush=True)
    dims = (8, 8, 8, 8)
    lat, fat, lng = setup(dims, 13)
    m = 0.05
    bs = torch.from_numpy(gaussian_source(dims, 14, 16)).cuda()
    xs, _ = lat.cg_solve(bs, m)
    net = Net(lat, layers=4, channels=4, seed=3, hermitian=True)
    info = net.train(bs, xs, epochs=6, batch=4, lr=3e-3, loss="residual", mass=m)
    w = net.get_weights()
    from oracle.net import hermitian_weights
    for a, c in zip(w, hermitian_weights(w[:2])):
        np.testing.assert_array_equal(a, c)
    assert info["loss_last"] < info["loss_first"]
    b = gaussian_source(dims, 15)
    bt = torch.from_numpy(b).cuda()
    A = lambda v: apply_m(fat, lng, v, dims, m)
    x1, i1 = lat.cg_solve(bt, m, net=net, stall_window=10)
    assert i1[0]["converged"] == 1
    assert true_residual(A, b[0], x1.cpu().numpy()[0]) <= 1.05e-10
    x2, i2 = lat.cg_solve(bt, m, net=net, stall_window=5, stall_ratio=1e-30)
    assert i2[0]["fell_back"] == 1 and i2[0]["converged"] == 1
    assert true_residual(A, b[0], x2.cpu().numpy()[0]) <= 1.05e-10
    # one-iteration windows (the benchmark's setting): handed over after the first iteration when the
    # ratio cannot be met; with the FP16 operator and a ratio any progress meets, the flexible phase runs
    # while each iteration lowers the residual (reliable updates at the window ends) and the solve still
    # reaches the true residual
    x3, i3 = lat.cg_solve(bt, m, net=net, stall_window=1, stall_ratio=1e-30)
    assert i3[0]["fell_back"] == 1 and i3[0]["converged"] == 1
    assert true_residual(A, b[0], x3.cpu().numpy()[0]) <= 1.05e-10
    lat.load_links(torch.from_numpy(fat).cuda(), torch.from_numpy(lng).cuda(), NAIK, precs=("f64", "f32", "f16"))
    x4, i4 = lat.cg_solve(bt, m, prec="f16", net=net, stall_window=1, stall_ratio=0.9999)
    assert i4[0]["converged"] == 1 and i4[0]["n_reliable"] >= 1, i4[0]
    assert true_residual(A, b[0], x4.cpu().numpy()[0]) <= 1.05e-10


def test_hermitian_network_on_gpu(gpu_lib):
    """With tied weights the GPU network is Hermitian and positive to FP32 accuracy."""
    from paper_1010_4782_amd.stagcg import Net

    print("hermitian net", flush=True)
    dims = (6, 4, 4, 6)
    lat, fat, _ = setup(dims, 21)
    net = Net(lat, layers=4, channels=8, seed=5, hermitian=True)
    u = torch.from_numpy(gaussian_source(dims, 22)).cuda()
    v = torch.from_numpy(gaussian_source(dims, 23)).cuda()
    a = torch.vdot(u.flatten(), net.apply(v).flatten()).item()
    b = torch.vdot(v.flatten(), net.apply(u).flatten()).item().conjugate()
    assert abs(a - b) <= 1e-5 * abs(a)
    q = torch.vdot(v.flatten(), net.apply(v).flatten()).item()
    assert q.real > 0 and abs(q.imag) <= 1e-5 * q.real


def test_net_refuses_when_fp32_links_were_dropped(gpu_lib):
    """The transports read the lattice's FP32 links at every launch: after a reload without them,
    every network call returns STAG_ERR_STATE before launching anything."""
    from paper_1010_4782_amd.stagcg import Net, StagError

    print("net after link reload", flush=True)
    dims = (4, 4, 4, 4)
    lat, fat, lng = setup(dims, 31)
    net = Net(lat, layers=2, channels=2)
    b = torch.from_numpy(gaussian_source(dims, 32, 1)).cuda()
    net.apply(b)
    lat.load_links(torch.from_numpy(fat).cuda(), torch.from_numpy(lng).cuda(), NAIK, precs=("f64",))
    with pytest.raises(StagError) as ei:
        net.apply(b)
    assert ei.value.status == 4  # STAG_ERR_STATE
    with pytest.raises(StagError):
        lat.cg_solve(b, 0.1, tol=1e-10, net=net)
    lat.load_links(torch.from_numpy(fat).cuda(), torch.from_numpy(lng).cuda(), NAIK, precs=("f64", "f32"))
    net.apply(b)  # usable again once the FP32 links are back


def test_net_forward_full_size_24cubed_48(gpu_lib):
    """The learned-preconditioner workload's lattice and network (24^3 x 48, 4 layers of 8 channels,
    the 8 -> 8 layers on the matrix cores) against the FP64 oracle on FP32-rounded links and weights."""
    from paper_1010_4782_amd.stagcg import Lattice, Net
    from stag_inputs import WORKLOADS, workload_links

    w = WORKLOADS[4]
    dims = w["lattices"][0][0]
    print(f"net forward full size {dims} (about half a minute of oracle time)", flush=True)
    fat, lng = workload_links(4)
    lat = Lattice(dims)
    lat.load_links(torch.from_numpy(fat).cuda(), torch.from_numpy(lng).cuda(), NAIK, precs=("f64", "f32"),
                   long_su3=True)
    channels = [1] + [w["channels"]] * (w["layers"] - 1) + [1]
    net = Net(lat, layers=w["layers"], channels=w["channels"])
    W32 = [quant.to_f32(x) for x in init_weights(channels, 41, scale=1.0)]
    net.set_weights(W32)
    r = gaussian_source(dims, 42, 1)
    out = net.apply(torch.from_numpy(r).cuda()).cpu().numpy()
    Ft = quant.to_f32(folded_fat(fat, dims))
    r32 = quant.to_f32(r[0])
    ref = net_forward(Ft, W32, r32, dims)
    assert_within(out[0], ref, fp32_bound(Ft, W32, r32, dims))


def test_fcg_trained_network_24cubed_48(gpu_lib):
    """The learned-preconditioner workload: 24^3 x 48, m = 0.01, 4 layers of 8 channels trained on
    solver-made pairs (a small set: the test checks the path, not the network's quality), then FCG with
    the FP64 operator and with the FP16 operator plus reliable updates; the oracle recomputes each
    true residual."""
    from paper_1010_4782_amd.stagcg import Lattice, Net
    from oracle.dslash import apply_m_chunked
    from stag_inputs import WORKLOADS, workload_links

    w = WORKLOADS[4]
    dims, m = w["lattices"][0][0], w["masses"][0]
    print(f"fcg trained network at {dims} m={m}", flush=True)
    fat, lng = workload_links(4)
    lat = Lattice(dims)
    lat.load_links(torch.from_numpy(fat).cuda(), torch.from_numpy(lng).cuda(), NAIK, precs=("f64", "f32", "f16"),
                   long_su3=True)
    bs = torch.from_numpy(gaussian_source(dims, 43, 8)).cuda()
    xs, _ = lat.cg_solve(bs, m)
    net = Net(lat, layers=w["layers"], channels=w["channels"], seed=7)
    info = net.train(bs, xs, epochs=2, batch=4, lr=2e-3, loss="solution")
    assert info["loss_last"] < info["loss_first"]
    b = gaussian_source(dims, 44, 1)
    bt = torch.from_numpy(b).cuda()
    workers = min(16, os.cpu_count() or 1)
    for prec in ("f64", "f16"):
        x, inf = lat.cg_solve(bt, m, prec=prec, net=net, stall_window=10)
        assert inf[0]["converged"] == 1, (prec, inf[0])
        xh = x.cpu().numpy()
        r = b - apply_m_chunked(fat, lng, xh, dims, m, workers=workers)
        res = float(np.linalg.norm(r) / np.linalg.norm(b))
        print(f"  {prec}: iters {inf[0]['iters']} fell_back {inf[0]['fell_back']} reliable {inf[0]['n_reliable']} "
              f"oracle true residual {res:.3e}", flush=True)
        assert res <= 1.05e-10
