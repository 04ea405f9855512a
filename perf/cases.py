"""Performance cases: the calls that users of the library make, over the sizes they make them at.

Each case names an entry point of paper_1010_4782_amd.stagcg, the lattice (Lx x Ly x Lz x Lt), and the
options of the call.  `listed()` gives the fixed cases, `draw(rng)` another case of the same ranges,
`prepare` makes what a program holds before the call (links loaded, sources on the GPU), `run` makes the
call, `work` counts the bytes and operations the call cannot do without, and `exact` computes the same
outputs with plain torch in complex128.

Links: three-hop links are random SU(3) matrices near the identity, fat links 0.6 SU(3) plus complex
Gaussian noise (the recipe of the test inputs, here by Gram-Schmidt so that the largest lattice is drawn
in a moment); sources are Gaussian.  Everything is drawn on the GPU from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1010_4782_amd.stagcg import Lattice, Net, cg_solve_batch

NAIK = -1.0 / 24.0
DEVICE = "cuda"


def listed():
    return [
        # the smallest call: one operator application on a test-sized lattice, bound by latency
        dict(name="dslash_f64_8x8x8x8", op="dslash", dims="8x8x8x8", nrhs=1, prec="f64", long_su3=False),
        # the operator of the production lattice, eight right-hand sides in the storage the solver uses
        dict(name="dslash_f16_48x48x48x144_8rhs", op="dslash", dims="48x48x48x144", nrhs=8, prec="f16",
             long_su3=False),
        # the normal operator on the paper's lattice (residual checks, user-side Krylov methods)
        dict(name="apply_m_28x28x28x96", op="apply_m", dims="28x28x28x96", nrhs=1, mass=0.0062, long_su3=True),
        # a whole plain FP64 solve on a small lattice: many dependent short launches
        dict(name="solve_f64_8x8x8x8", op="solve", dims="8x8x8x8", nrhs=1, mass=0.05, prec="f64", long_su3=False),
        # the mixed-precision solve of the paper's lattice at its light mass
        dict(name="solve_f16_28x28x28x96", op="solve", dims="28x28x28x96", nrhs=1, mass=0.0062, prec="f16",
             long_su3=True),
        # an FP32 solve with ragged extents and an odd number of right-hand sides
        dict(name="solve_f32_10x14x18x22_3rhs", op="solve", dims="10x14x18x22", nrhs=3, mass=0.05, prec="f32",
             long_su3=True),
        # three ensembles of different shapes solved as one batch
        dict(name="batch_f16_three_lattices", op="batch", dims="16x16x16x16/4,24x24x24x48/12,32x32x32x64/8",
             mass=0.05, prec="f16", long_su3=True),
        # a new gauge configuration arrives: its links are packed, then applied once in both precisions
        dict(name="load_links_28x28x28x96", op="load", dims="28x28x28x96", prec="f16", long_su3=True),
        # smearing of a thin gauge field into the improved action's two link fields
        dict(name="fatten_24x24x24x48", op="fatten", dims="24x24x24x48", u0=1.0),
        # one application of the learned preconditioner (the size it is trained and used at)
        dict(name="net_apply_24x24x24x48", op="net", dims="24x24x24x48", nrhs=1, layers=4, channels=8),
        # one optimiser step's forward and backward pass of that network
        dict(name="net_grad_24x24x24x48", op="grad", dims="24x24x24x48", nrhs=2, layers=4, channels=8, mass=0.01,
             loss="residual"),
        # the correlator of four point-source propagators, after their solve
        dict(name="pion_28x28x28x96_4src", op="pion", dims="28x28x28x96", nrhs=12, mass=0.0062),
    ]


def _draw_dims(rng, lo, hi):
    """Even extents with a volume spread over the logarithm of [lo, hi]; rarely equal, time often the longest."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    side = (v / rng.choice([1.0, 2.0, 3.0])) ** 0.25
    sp = [min(48, max(4, 2 * round(side * rng.uniform(0.8, 1.25) / 2))) for _ in range(3)]
    lt = min(144, max(4, 2 * int(v / (sp[0] * sp[1] * sp[2]) / 2)))
    return sp + [lt]


def _text(dims):
    return "x".join(str(d) for d in dims)


def draw(rng):
    op = rng.choice(["dslash", "dslash", "apply_m", "solve", "solve", "batch", "load", "fatten", "net", "grad", "pion"])
    su3 = rng.random() < 0.5
    if op == "dslash":
        return dict(op=op, dims=_text(_draw_dims(rng, 4e3, 8e6)), nrhs=rng.choice([1, 1, 2, 3, 4, 6, 8]),
                    prec=rng.choice(["f64", "f32", "f16"]), long_su3=su3)
    if op == "apply_m":
        return dict(op=op, dims=_text(_draw_dims(rng, 4e3, 2e6)), nrhs=rng.choice([1, 1, 2, 3, 4, 8]),
                    mass=round(rng.uniform(0.005, 0.1), 4), long_su3=su3)
    if op == "solve":
        dims = _draw_dims(rng, 4e3, 1.5e6)
        vol = math.prod(dims)
        nrhs = rng.choice([n for n in (1, 2, 3, 4, 8) if n == 1 or n * vol <= 2e6])
        return dict(op=op, dims=_text(dims), nrhs=nrhs, mass=round(rng.uniform(0.01, 0.1), 4),
                    prec=rng.choice(["f64", "f32", "f16"]), long_su3=su3)
    if op == "batch":
        parts = [(_draw_dims(rng, 2e4, 7e5), rng.choice([1, 2, 3, 4, 8])) for _ in range(rng.choice([2, 3]))]
        return dict(op=op, dims=",".join("%s/%d" % (_text(d), n) for d, n in parts),
                    mass=round(rng.uniform(0.02, 0.1), 4), prec=rng.choice(["f64", "f32", "f16"]), long_su3=su3)
    if op == "load":
        return dict(op=op, dims=_text(_draw_dims(rng, 4e3, 2e6)), prec=rng.choice(["f64", "f32", "f16"]), long_su3=su3)
    if op == "fatten":
        return dict(op=op, dims=_text(_draw_dims(rng, 4e3, 1e6)), u0=rng.choice([1.0, 0.87]))
    if op == "pion":
        return dict(op=op, dims=_text(_draw_dims(rng, 2e4, 2e6)), nrhs=3 * rng.choice([1, 2, 3, 4]),
                    mass=round(rng.uniform(0.005, 0.1), 4))
    c = dict(op=op, dims=_text(_draw_dims(rng, 4e3, 6e5)), nrhs=rng.choice([1, 2, 3]), layers=rng.choice([2, 3, 4]),
             channels=rng.choice([2, 4, 8]))
    if op == "grad":
        c.update(mass=round(rng.uniform(0.005, 0.1), 4), loss=rng.choice(["residual", "solution"]))
    return c


# ---- inputs ----------------------------------------------------------------------------------------

def _problems(case):
    """[(dims, nrhs)]: one lattice, or the lattices of a batch."""
    out = []
    for part in case["dims"].split(","):
        d, _, n = part.partition("/")
        out.append((tuple(int(v) for v in d.split("x")), int(n) if n else case.get("nrhs", 1)))
    return out


def _gen(seed, salt):
    g = torch.Generator(device=DEVICE)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFFFFFF)
    return g


def _gauss(shape, gen, scale=1.0):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=gen, dtype=torch.float64, device=DEVICE) * scale)


def _links(dims, seed, salt, fat):
    """SU(3) matrices near the identity, [4][Lt][Lz][Ly][Lx][3][3]; fat: 0.6 of them plus noise."""
    lx, ly, lz, lt = dims
    gen = _gen(seed, salt)
    out = torch.empty((4, lt, lz, ly, lx, 3, 3), dtype=torch.complex128, device=DEVICE)
    step = max(1, 4_000_000 // (lx * ly * lz))
    for mu in range(4):
        for t in range(0, lt, step):
            u = out[mu, t:t + step]
            rows = _gauss(u.shape[:-2] + (2, 3), gen, 0.2)
            rows[..., 0, 0] += 1.0
            rows[..., 1, 1] += 1.0
            a, b = rows[..., 0, :], rows[..., 1, :]
            a = a / torch.linalg.vector_norm(a, dim=-1, keepdim=True)
            b = b - (a.conj() * b).sum(-1, keepdim=True) * a
            b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
            u[..., 0, :] = a
            u[..., 1, :] = b
            for i, (j, k) in enumerate(((1, 2), (2, 0), (0, 1))):
                u[..., 2, i] = (a[..., j] * b[..., k] - a[..., k] * b[..., j]).conj()
            if fat:
                u *= 0.6
                u += _gauss(u.shape, gen, 0.05)
    return out


def _vectors(dims, nrhs, seed, salt):
    return _gauss((nrhs, math.prod(dims) // 2, 3), _gen(seed, salt))


def _weights(case, seed):
    rng = np.random.default_rng(int(seed) + 17)
    ch = [1] + [case["channels"]] * (case["layers"] - 1) + [1]
    out = []
    for ci, co in zip(ch[:-1], ch[1:]):
        w = rng.standard_normal((9, co, ci, 2)) * (0.5 / math.sqrt(9.0 * ci))
        w[0, :, :, 0] += 1.0 / ci
        out.append(np.ascontiguousarray(w).view(np.complex128)[..., 0])
    return out


def _precs(case):
    if case["op"] in ("net", "grad"):
        return ("f64", "f32")
    return tuple(dict.fromkeys(("f64", case.get("prec", "f64"))))


def prepare(case, seed):
    op = case["op"]
    s = dict(case=case, lats=[], x=[])
    for i, (dims, nrhs) in enumerate(_problems(case)):
        lat = Lattice(dims)
        s["lats"].append(lat)
        if op == "fatten":
            s["thin"] = _links(dims, seed, 100 * i + 1, False)
            continue
        fat, lng = _links(dims, seed, 100 * i + 1, True), _links(dims, seed, 100 * i + 2, False)
        if op == "load":
            s["fat"], s["lng"] = fat, lng
        else:
            lat.load_links(fat, lng, NAIK, precs=_precs(case), long_su3=bool(case.get("long_su3", False)))
        del fat, lng
        s["x"].append(_vectors(dims, nrhs, seed, 100 * i + 3))
        if op == "grad":
            s["sol"] = _vectors(dims, nrhs, seed, 100 * i + 4)
    if op in ("net", "grad"):
        s["net"] = Net(s["lats"][0], layers=case["layers"], channels=case["channels"], seed=int(seed))
        s["net"].set_weights(_weights(case, seed))
    return s


def run(s):
    case, op = s["case"], s["case"]["op"]
    lat = s["lats"][0]
    if op == "fatten":
        return lat.fatten_links(s["thin"], u0=case["u0"])
    x = s["x"][0]
    if op == "dslash":
        return lat.dslash(x, 1, prec=case["prec"])
    if op == "apply_m":
        return lat.apply_m(x, case["mass"])
    if op == "solve":
        return lat.cg_solve(x, case["mass"], tol=1e-10, prec=case["prec"])[0]
    if op == "batch":
        return cg_solve_batch([(l, b, case["mass"], None) for l, b in zip(s["lats"], s["x"])], tol=1e-10,
                              prec=case["prec"])[0]
    if op == "load":
        lat.load_links(s["fat"], s["lng"], NAIK, precs=_precs(case), long_su3=case["long_su3"])
        return [lat.dslash(x, 1, prec=p) for p in _precs(case)]
    if op == "net":
        return s["net"].apply(x)
    if op == "grad":
        return s["net"].loss_grad(x, s["sol"], loss=case["loss"], mass=case["mass"])
    if op == "pion":
        return lat.pion_correlator(x, case["mass"])
    raise ValueError(op)


# ---- what a pass cannot do without -----------------------------------------------------------------

_VEC = dict(f64=48, f32=24, f16=16)
_LINK = dict(f64=144, f32=72, f16=36)


def _link_bytes(prec, su3):
    """Packed links of one output site: eight one-hop and eight three-hop matrices (two rows each with su3)."""
    return 8 * _LINK[prec] + 8 * _LINK[prec] * (2 if su3 else 3) // 3 + (8 if prec == "f16" else 0)


def _iterations(dims, mass):
    """CG iterations to 1e-10 on these fields, fitted to counts between 8^4 and 28^3 x 96, m = 0.0062 to 0.1."""
    return 30.0 / math.sqrt(0.0005 + 4 * mass * mass) * min(1.0, (math.prod(dims) / 1e5) ** 0.15)


def work(case):
    op, su3 = case["op"], bool(case.get("long_su3", False))
    b = f = 0.0
    for dims, n in _problems(case):
        half = math.prod(dims) // 2
        if op == "dslash":
            b += half * (_link_bytes(case["prec"], su3) + 96 * n)
            f += half * n * 1146
        elif op == "apply_m":
            b += half * (2 * _link_bytes("f64", su3) + 96 * n)
            f += half * n * (2 * 1146 + 12)
        elif op == "pion":
            b += half * (_link_bytes("f64", su3) + 48 * n)
            f += half * n * (1146 + 24)
        elif op in ("solve", "batch"):
            # per iteration: both operator halves' links, the direction and its image, the residual, the
            # solution and the direction updated; each in its storage precision
            v, p = _VEC[case["prec"]], case["prec"]
            vx = 48 if p == "f64" else 24
            it = _iterations(dims, case["mass"])
            b += it * half * (2 * _link_bytes(p, su3) + n * (9 * v + 2 * vx))
            f += it * half * n * (2 * 1146 + 60)
        elif op == "load":
            b += 2 * half * 8 * 144 + 2 * half * sum(_link_bytes(p, su3) for p in _precs(case))
            b += half * sum(_link_bytes(p, su3) + 96 for p in _precs(case))
            f += half * len(_precs(case)) * 1146
        elif op == "fatten":
            b += 2 * half * 12 * 144
            f += 2 * half * 4 * (36 * 2 * 198 + 2 * 198)
        else:
            ch = [1] + [case["channels"]] * (case["layers"] - 1) + [1]
            act = sum(48 * c for c in ch[1:-1])  # both parities of the inner activations, complex64
            mix = sum(2 * (8 * 66 * ci + 9 * 24 * ci * co) for ci, co in zip(ch[:-1], ch[1:]))
            # forward: every layer reads the one-hop links and its input and writes its output
            fb, ff = 96 + 2 * act + len(ch[1:]) * 2 * 8 * 72, mix
            if op == "grad":
                fb += 48 * 2 + 3 * act + 2 * (len(ch[1:]) - 1) * 2 * 8 * 72
                ff += 2 * mix
                if case["loss"] == "residual":
                    fb += 4 * _link_bytes("f64", False)
                    ff += 4 * 1146
            b += half * n * fb
            f += half * n * ff
    return dict(bytes=float(b), flops=float(f))


# ---- the same outputs in 64 bits, by plain torch ---------------------------------------------------

def _parity(dims):
    lx, ly, lz, lt = dims
    r = lambda n, k: torch.arange(n, device=DEVICE).reshape([-1 if i == k else 1 for i in range(4)])  # noqa: E731
    return (r(lt, 0) + r(lz, 1) + r(ly, 2) + r(lx, 3)) % 2


def _embed(v, dims, parity):
    """[..., V/2, 3] on one parity -> [..., Lt, Lz, Ly, Lx, 3], zero on the other."""
    lx, ly, lz, lt = dims
    full = torch.zeros(v.shape[:-2] + (lx * ly * lz * lt, 3), dtype=v.dtype, device=v.device)
    full[..., (_parity(dims) == parity).reshape(-1), :] = v
    return full.reshape(v.shape[:-2] + (lt, lz, ly, lx, 3))


def _restrict(f, dims, parity):
    return f.reshape(f.shape[:-5] + (-1, 3))[..., (_parity(dims) == parity).reshape(-1), :]


def _signs(dims, mu, hop):
    """eta_mu(n), and the antiperiodic sign of a forward time hop that starts at n; [Lt, Lz, Ly, Lx, 1]."""
    lx, ly, lz, lt = dims
    r = lambda n, k: torch.arange(n, device=DEVICE).reshape([-1 if i == k else 1 for i in range(4)])  # noqa: E731
    s = torch.zeros((lt, lz, ly, lx), dtype=torch.int64, device=DEVICE)
    for k, n in list(enumerate((lx, ly, lz)))[:mu]:
        s = s + r(n, 3 - k)
    eta = 1.0 - 2.0 * (s % 2)
    start = 1.0 - 2.0 * (((r(lt, 0) + hop) // lt) % 2) if mu == 3 else torch.ones((1, 1, 1, 1), device=DEVICE)
    return eta.double()[..., None], start.double()[..., None]


def _mv(u, v):
    return u[..., 0] * v[..., 0, None] + u[..., 1] * v[..., 1, None] + u[..., 2] * v[..., 2, None]


def _hop(u, v, dims, mu, hop, fwd):
    """The signed hop term of D: eta s U psi(n + hop mu), or -eta s U^dag psi at n - hop mu."""
    eta, start = _signs(dims, mu, hop)
    axis = -2 - mu
    if fwd:
        return eta * start * _mv(u, torch.roll(v, -hop, axis))
    return -eta * torch.roll(start * _mv(u.conj().transpose(-1, -2), v), hop, axis)


def _d(fat, lng, v, dims, parity):
    """D restricted to output sites of `parity`, on [V/2, 3]."""
    f = _embed(v, dims, 1 - parity)
    out = torch.zeros_like(f)
    for mu in range(4):
        for fwd in (True, False):
            out += _hop(fat[mu], f, dims, mu, 1, fwd)
            out += NAIK * _hop(lng[mu], f, dims, mu, 3, fwd)
    return _restrict(out, dims, parity)


def _m(fat, lng, v, dims, mass):
    return 4 * mass * mass * v - _d(fat, lng, _d(fat, lng, v, dims, 1), dims, 0)


def _cg(fat, lng, b, dims, mass):
    x = torch.zeros_like(b)
    r, p = b.clone(), b.clone()
    rr = torch.vdot(r.reshape(-1), r.reshape(-1)).real
    stop = 1e-28 * rr
    for i in range(20000):
        ap = _m(fat, lng, p, dims, mass)
        a = rr / torch.vdot(p.reshape(-1), ap.reshape(-1)).real
        x = x + a * p
        r = r - a * ap
        new = torch.vdot(r.reshape(-1), r.reshape(-1)).real
        if i % 10 == 9 and bool(new < stop):
            break
        p, rr = r + (new / rr) * p, new
    return x


def _net(fat, ws, b, dims):
    """The network on one even-site vector; fat links with eta and the boundary sign folded in."""
    psi = _embed(b, dims, 0)[None]
    for w in ws:
        terms = [psi]
        for fwd in (True, False):
            for mu in range(4):
                t = _hop(fat[mu], psi, dims, mu, 1, fwd)
                terms.append(t if fwd else -t)
        flat = [t.reshape(t.shape[0], -1) for t in terms]
        psi = sum(w[d] @ flat[d] for d in range(9)).reshape((w.shape[1],) + psi.shape[1:])
    return _restrict(psi[0], dims, 0)


def _fatten(u, dims, u0):
    ax = lambda d: -3 - d  # noqa: E731  (lattice axis of direction d in [Lt, Lz, Ly, Lx, 3, 3])
    mul = lambda a, b: sum(a[..., :, k, None] * b[..., k, None, :] for k in range(3))  # noqa: E731
    dag = lambda a: a.conj().transpose(-1, -2)  # noqa: E731

    def wrap(f, mu, nu, sign):
        """The path that steps sign nu, follows f along mu, and steps back."""
        side = torch.roll(u[nu], -1, ax(mu))
        if sign > 0:
            return mul(mul(u[nu], torch.roll(f, -1, ax(nu))), dag(side))
        return torch.roll(mul(mul(dag(u[nu]), f), side), 1, ax(nu))

    def both(f, mu, nu):
        return wrap(f, mu, nu, 1) + wrap(f, mu, nu, -1)

    fat, lng = torch.empty_like(u), torch.empty_like(u)
    for mu in range(4):
        others = [d for d in range(4) if d != mu]
        v = 5.0 / 8.0 * u[mu]
        x = {}
        for nu in others:
            p, m = wrap(u[mu], mu, nu, 1), wrap(u[mu], mu, nu, -1)
            x[nu] = p + m
            v = v + x[nu] / (16.0 * u0 ** 2) - (wrap(p, mu, nu, 1) + wrap(m, mu, nu, -1)) / (16.0 * u0 ** 4)
        for rho in others:
            for si in others:
                if rho != si:
                    y = both(x[si], mu, rho)
                    third = sum(others) - rho - si
                    v = v + y / (64.0 * u0 ** 4) + both(y, mu, third) / (384.0 * u0 ** 6)
        fat[mu] = v
        lng[mu] = mul(mul(u[mu], torch.roll(u[mu], -1, ax(mu))), torch.roll(u[mu], -2, ax(mu)))
    return fat, lng


def exact(case, seed):
    op = case["op"]
    (dims, nrhs), *more = _problems(case)
    vol = math.prod(dims)
    if more or (op == "solve" and vol * nrhs > 200_000):
        return None  # a plain torch CG of this size takes longer than a check should
    if op == "fatten":
        return _fatten(_links(dims, seed, 1, False), dims, case["u0"])
    fat, lng = _links(dims, seed, 1, True), _links(dims, seed, 2, False)
    x = _vectors(dims, nrhs, seed, 3)
    if op == "dslash":
        return torch.stack([_d(fat, lng, v, dims, 1) for v in x])
    if op == "load":
        one = torch.stack([_d(fat, lng, v, dims, 1) for v in x])
        return [one for _ in _precs(case)]
    if op == "apply_m":
        return torch.stack([_m(fat, lng, v, dims, case["mass"]) for v in x])
    if op == "solve":
        return torch.stack([_cg(fat, lng, v, dims, case["mass"]) for v in x])
    if op == "pion":
        def slices(v):
            return v.abs().square().reshape(nrhs // 3, 3, dims[3], -1).sum(dim=(1, 3))
        odd = torch.stack([_d(fat, lng, v, dims, 1) for v in x])
        return 4 * case["mass"] ** 2 * slices(x) + slices(odd)
    ws = [torch.from_numpy(w).to(DEVICE) for w in _weights(case, seed)]
    if op == "net":
        return torch.stack([_net(fat, ws, v, dims) for v in x])
    # loss and its gradient with respect to conj(W): torch's gradient of a real function is twice that
    ws = [w.requires_grad_() for w in ws]
    total, sol = 0.0, _vectors(dims, nrhs, seed, 4)
    for b, y in zip(x, sol):
        out = _net(fat, ws, b, dims)
        if case["loss"] == "residual":
            loss = (_m(fat, lng, out, dims, case["mass"]) - b).abs().square().sum() / b.abs().square().sum()
        else:
            loss = (out - y).abs().square().sum() / y.abs().square().sum()
        loss.backward()
        total += float(loss.detach())
    return total, [(w.grad / 2).cpu().numpy() for w in ws]
