"""The workloads this library is timed on, each one call (or one step) of a user's program.

A case is a dict of plain values:
  kind    what is called: "synthesis", "adjoint" (spin 0, a batch of maps), "spin" (one step
          of a spin-weighted solver: synthesis then adjoint), "grad" (autograd forward and
          backward of a lensing-type loss, with respect to coefficients and positions),
          "solve" (a fixed number of CGLS iterations) or "learn" (the per-point weights:
          density, features, network forward and backward);
  lmax, mmax, nmaps, dtype ("f64" / "mixed"), eps, and per kind spin or iters;
  points  "uniform" (npts random points), "grid" (an equi-angular grid of `rings` rings of
          2 rings - 1 pixels, every point deflected by a few arcminutes: the CMB-lensing remap)
          or "holes" (npts random points with circular holes: a masked survey).
Inputs are drawn on the GPU from the seed alone.  The plan is what a program keeps between
calls, so it is made in prepare().
"""
import math

import torch

import paper_2406_14542_amd as P
from paper_2406_14542_amd import autograd, learned
from paper_2406_14542_amd import _binding as B

DEV = "cuda"
ARCMIN = math.pi / 10800.0


def _case(name, kind, lmax, points, size, nmaps=1, dtype="f64", eps=1e-12, mmax=None, **more):
    c = dict(name=name, kind=kind, lmax=lmax, mmax=lmax if mmax is None else mmax, points=points,
             nmaps=nmaps, dtype=dtype, eps=eps, **more)
    c["rings" if points == "grid" else "npts"] = size
    return c


def listed():
    return [
        # the smallest calls: an interactive or per-object transform, where latency counts
        _case("adjoint_l63_b2", "adjoint", 63, "uniform", 4096, nmaps=2),
        _case("synthesis_l127", "synthesis", 127, "uniform", 32768),
        # one map remapped / its adjoint on a deflected grid at a middle band limit, the inner
        # call of a lensing reconstruction
        _case("remap_l2047", "synthesis", 2047, "grid", 2048, eps=1e-10),
        _case("remap_adjoint_l2047", "adjoint", 2047, "grid", 2048, eps=1e-10),
        # band limits that are not 2^k - 1, mmax below lmax, batches that are not a multiple of
        # four: maps from a simulation at its own resolution, and a catalogue of positions
        _case("batch_l1500_b3", "synthesis", 1500, "uniform", 3000017, nmaps=3, eps=1e-10),
        _case("catalogue_adjoint_l1000_b5", "adjoint", 1000, "holes", 200003, nmaps=5, mmax=900),
        # the largest calls: the headline benchmark's batch, each direction
        _case("batch_l4095_b4", "synthesis", 4095, "uniform", 33550336, nmaps=4, dtype="mixed",
              eps=1e-5),
        _case("batch_adjoint_l4095_b4", "adjoint", 4095, "uniform", 33550336, nmaps=4,
              dtype="mixed", eps=1e-5),
        # polarisation: one spin-2 field, both directions
        _case("spin2_l2047", "spin", 2047, "grid", 2048, spin=2, eps=1e-10),
        # the gradient of a lensing-type loss over a batch of maps
        _case("grad_l1023_b8", "grad", 1023, "grid", 1024, nmaps=8),
        # iterations of the least-squares inverse on a masked, barely oversampled point set
        _case("solve_l1023", "solve", 1023, "holes", 1572864, iters=10),
        # weights of a point set of the learned inverse and their parameter gradient
        _case("weights_2m", "learn", 2047, "holes", 2000003, dtype="f32", eps=0.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["synthesis", "adjoint", "synthesis", "adjoint", "spin", "grad", "solve",
                       "learn"])
    if kind == "learn":
        return dict(kind=kind, lmax=2047, mmax=2047, points=rng.choice(["uniform", "holes"]),
                    npts=_log_int(rng, 3000, 2000000), nmaps=1, dtype="f32", eps=0.0)
    lmax = _log_int(rng, 40, 2200 if kind in ("synthesis", "adjoint") else 1100)
    c = dict(kind=kind, lmax=lmax, mmax=lmax if rng.random() < 0.7 else rng.randint(lmax // 2, lmax),
             points=rng.choice(["uniform", "grid", "holes"]))
    if kind == "grad" or rng.random() < 0.6:
        c["dtype"], c["eps"] = "f64", rng.choice([1e-8, 1e-10, 1e-12])
    else:
        c["dtype"], c["eps"] = "mixed", rng.choice([1e-4, 1e-5, 1e-6])
    if c["points"] == "grid":
        c["rings"] = lmax + rng.randint(1, lmax // 2)
    else:
        c["npts"] = _log_int(rng, max(1000, lmax * lmax // 8), 4 * lmax * lmax + 2000)
    c["nmaps"] = 1 if kind in ("spin", "solve") else rng.randint(1, 8 if lmax < 1100 else 4)
    if kind == "spin":
        c["spin"] = rng.choice([1, 2, 2, 3])
    if kind == "solve":
        c["iters"] = rng.randint(3, 10)
    return c


# ---- inputs -------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, dtype=torch.float64, device=DEV)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, dtype=torch.float64, device=DEV)


def _npts(case):
    return case["rings"] * (2 * case["rings"] - 1) if case["points"] == "grid" else case["npts"]


def _points(case, g):
    """theta, phi: float64 tensors of the case's point set."""
    if case["points"] == "grid":
        r = case["rings"]
        p = 2 * r - 1
        th = ((torch.arange(r, dtype=torch.float64, device=DEV) + 0.5) * (math.pi / r))
        ph = torch.arange(p, dtype=torch.float64, device=DEV) * (2.0 * math.pi / p)
        th, ph = th.repeat_interleave(p), ph.repeat(r)
        at, ap = (_randn(g, r * p) * (2.5 * ARCMIN) for _ in range(2))
        a = torch.hypot(at, ap)
        sinc, ca = torch.sin(a) / a.clamp_min(1e-300), torch.cos(a)
        ct, st = torch.cos(th), torch.sin(th)
        # the displaced direction in the frame of the point's meridian
        nx, ny, nz = ca * st + sinc * at * ct, sinc * ap, ca * ct - sinc * at * st
        return (torch.atan2(torch.hypot(nx, ny), nz).clamp(0.0, math.pi),
                torch.remainder(ph + torch.atan2(ny, nx), 2.0 * math.pi))
    n = case["npts"]
    if case["points"] == "uniform":
        return torch.acos(1.0 - 2.0 * _rand(g, n)), _rand(g, n) * (2.0 * math.pi)
    # 20 Gaussian holes of 5 degrees: rejection from uniform points (at most half are rejected)
    z = 1.0 - 2.0 * _rand(g, 20)
    p = _rand(g, 20) * (2.0 * math.pi)
    s = torch.sqrt(1.0 - z * z)
    hole = torch.stack([s * torch.cos(p), s * torch.sin(p), z])
    m = 2 * n + 4096
    th, ph = torch.acos(1.0 - 2.0 * _rand(g, m)), _rand(g, m) * (2.0 * math.pi)
    st = torch.sin(th)
    keep = torch.ones_like(th)
    for k in range(20):
        c = st * torch.cos(ph) * hole[0, k] + st * torch.sin(ph) * hole[1, k] + torch.cos(th) * hole[2, k]
        d = torch.acos(c.clamp(-1.0, 1.0)) * (180.0 / math.pi)
        keep *= 1.0 - torch.exp(-d * d / 50.0)
    sel = (_rand(g, m) < keep).nonzero().squeeze(1)[:n]
    return th[sel].contiguous(), ph[sel].contiguous()


def _degrees(case):
    """(l, m) of every stored coefficient."""
    lmax, mmax = case["lmax"], case["mmax"]
    m = torch.repeat_interleave(torch.arange(mmax + 1, device=DEV),
                                lmax + 1 - torch.arange(mmax + 1, device=DEV))
    start = m * (2 * lmax + 3 - m) // 2
    return torch.arange(m.numel(), device=DEV) - start + m, m


def _alm(case, g, rows):
    """rows coefficient sets with the falling spectrum C_l = 1 / (l + 10)^2."""
    l, m = _degrees(case)
    amp = (1.0 / (l + 10.0)) * torch.where(m == 0, 1.0, math.sqrt(0.5))
    x = _randn(g, rows, 2, l.numel())
    return torch.complex(x[:, 0] * amp, torch.where(m == 0, 0.0, 1.0) * x[:, 1] * amp)


def _inputs(case, seed):
    g = _generator(seed)
    d = dict(zip(("theta", "phi"), _points(case, g)))
    n, b = d["theta"].numel(), case["nmaps"]
    kind = case["kind"]
    if kind in ("synthesis", "grad"):
        d["alm"] = _alm(case, g, b)
    if kind == "grad":
        d["w"] = _rand(g, b, n)
    if kind == "adjoint":
        d["map"] = _randn(g, b, n)
    if kind == "spin":
        a = _alm(case, g, 2)
        a[:, _degrees(case)[0] < case["spin"]] = 0.0
        d["alm"], d["map"] = a[None], _randn(g, 1, 2, n)
    if kind == "solve":
        d["map"] = _randn(g, n)
    if kind == "learn":
        d["params"] = torch.from_numpy(learned.init_params(seed % 1000)).to(DEV)
        d["grad_w"] = _randn(g, n).float()
    return d


def prepare(case, seed):
    st = dict(_inputs(case, seed), case=case)
    if case["kind"] == "learn":
        st["net"] = learned.LearnedWeights(params=st.pop("params").cpu().numpy())
        return st
    st["plan"] = P.Plan(case["lmax"], case["mmax"], st["theta"], st["phi"], case["eps"],
                        dtype=case["dtype"])
    if case["kind"] != "grad":
        del st["theta"], st["phi"]
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "synthesis":
        return st["plan"].synthesis(st["alm"])
    if kind == "adjoint":
        return st["plan"].adjoint(st["map"])
    if kind == "spin":
        return (st["plan"].synthesis_spin(case["spin"], st["alm"]),
                st["plan"].adjoint_spin(case["spin"], st["map"]))
    if kind == "grad":
        leaf = [st[k].detach().requires_grad_(True) for k in ("alm", "theta", "phi")]
        f = autograd.synthesis(st["plan"], *leaf)
        f.backward(st["w"] * f.detach())  # d/df of sum w f^2 / 2
        return [f.detach()] + [x.grad for x in leaf]
    if kind == "solve":
        a, iters, relres, _ = st["plan"].solve(st["map"], tol=1e-13, maxiter=case["iters"],
                                               check=False)
        return a, iters, relres
    feat = st["net"].features(st["theta"], st["phi"])
    w = st["net"].weights(features=feat)
    grad = B.mlp_backward(st["net"].params, feat, st["grad_w"], st["net"].scale(feat.shape[0]))
    return feat, w, grad


# ---- what a pass cannot do without --------------------------------------------------------

def _nalm(case):
    lmax, mmax = case["lmax"], case["mmax"]
    return (mmax + 1) * (lmax + 1) - mmax * (mmax + 1) // 2


def work(case):
    """Bytes: coefficients, maps and points once each.  Flops: per (l, m) and ring pair one
    recurrence step and its products with every map, the taps' products of every point, and
    the FFTs of the fine grid (5 N log2 N over the half of its rows that points reach)."""
    n, b, kind = _npts(case), case["nmaps"], case["kind"]
    if kind == "learn":
        p = 2 * (12 * 128 + 2 * 128 * 128 + 128)
        return {"bytes": n * (16.0 + 2 * 48 + 4 + 4), "flops": float(n) * p * 4}
    nalm, half = _nalm(case), case["lmax"] / 2 + 1
    wid = math.ceil(math.log(1.0 / case["eps"]) / (math.pi * math.sqrt(0.5))) + 1
    rows = 2 if kind == "spin" else b
    grid = (4.0 * case["lmax"] + 2) * (4.0 * case["mmax"] + 2)
    fft = 2.5 * grid * math.log2(grid) / 2
    leg = nalm * half * ((14 + 16) if kind == "spin" else 3 + 4 * b)
    one = leg + rows * (fft + 2.0 * n * wid * wid)
    byt = 16.0 * n + rows * (8.0 * n + 16.0 * nalm)
    if kind == "spin":
        return {"bytes": 2 * byt, "flops": 2 * one}
    if kind == "grad":
        return {"bytes": 2 * byt + 8.0 * n * (2 + rows), "flops": 2 * one + rows * 4.0 * n * wid * wid}
    if kind == "solve":
        return {"bytes": 2 * case["iters"] * byt, "flops": 2 * case["iters"] * one}
    return {"bytes": byt, "flops": one}


# ---- direct sums in 64 bits ---------------------------------------------------------------
# lam_lm(theta) of all m <= min(l, mmax) at once, one degree after the other, over chunks of
# points.  No scaling of the exponent range: up to degree 1500 a start value that underflows
# belongs to a function that stays negligible.

def _lam_start(mmax, s):
    m = torch.arange(mmax + 1, dtype=torch.float64, device=DEV)
    k = torch.arange(1, mmax + 1, dtype=torch.float64, device=DEV)
    prod = torch.cat([torch.ones(1, dtype=torch.float64, device=DEV), torch.cumprod((2 * k - 1) / (2 * k), 0)])
    c = torch.sqrt((2 * m + 1) / (4 * math.pi) * prod) * torch.where(m % 2 == 1, -1.0, 1.0)
    return c[:, None] * torch.pow(s[None], m[:, None])


def _mirror(theta):
    """sin(theta), 1 - |cos(theta)| and the sign of cos(theta), accurate near both poles."""
    t = torch.minimum(theta, math.pi - theta)
    return torch.sin(theta), 2.0 * torch.sin(0.5 * t) ** 2, torch.where(theta <= 0.5 * math.pi, 1.0, -1.0)


def _lam_sweep(lmax, mmax, theta):
    """Yields (l, k, lam_l, lam_{l-1}): rows m = 0 .. k - 1 of the functions of degree l, l - 1."""
    s, y, sg = _mirror(theta)
    start = _lam_start(mmax, s)
    v, vp = torch.zeros_like(start), torch.zeros_like(start)
    m = torch.arange(mmax + 1, dtype=torch.float64, device=DEV)
    for l in range(lmax + 1):
        if l > 0:
            k = min(l, mmax + 1)
            a = torch.sqrt((4.0 * l * l - 1) / (l * l - m[:k] ** 2))[:, None]
            b = torch.sqrt(((l - 1.0) ** 2 - m[:k] ** 2).clamp_min(0.0) / (4.0 * (l - 1.0) ** 2 - 1))[:, None]
            new = a * (torch.addcmul(v[:k], v[:k], -y) * sg - b * vp[:k])
            vp[:k] = v[:k]
            v[:k] = new
        if l <= mmax:
            v[l] = start[l]
        k = min(l, mmax) + 1
        yield l, k, v[:k], vp[:k]


def _index(case, l, k):
    m = torch.arange(k, device=DEV)
    return m * (2 * case["lmax"] + 1 - m) // 2 + l


def _chunks(case, n, rows):
    size = max(256, int(2.5e8 / ((case["mmax"] + 1) * (2 * rows + 4))))
    return [slice(i, min(i + size, n)) for i in range(0, n, size)]


def _turn(case, phi):
    m = torch.arange(case["mmax"] + 1, dtype=torch.float64, device=DEV)
    a = m[:, None] * phi[None]
    return torch.cos(a), torch.sin(a)


def _weight(case):
    m = torch.full((case["mmax"] + 1, 1), 2.0, dtype=torch.float64, device=DEV)
    m[0] = 1.0
    return m


def _direct_synthesis(case, theta, phi, alm, deriv=False):
    """maps [b][n], and with deriv their theta and phi derivatives."""
    b, n, m1 = alm.shape[0], theta.numel(), case["mmax"] + 1
    ri = torch.view_as_real(alm).permute(1, 0, 2).reshape(-1, 2 * b).clone()  # [nalm][2 b]
    ri[: case["lmax"] + 1, 1::2] = 0.0
    f, ft, fp = (torch.zeros(b, n, dtype=torch.float64, device=DEV) for _ in range(3))
    mm = torch.arange(m1, dtype=torch.float64, device=DEV)[:, None]
    for c in _chunks(case, n, b * (2 if deriv else 1)):
        th = theta[c]
        s = torch.sin(th)
        cot = torch.cos(th) / s
        F = torch.zeros(m1, 2 * b, th.numel(), dtype=torch.float64, device=DEV)
        D = torch.zeros_like(F) if deriv else None
        for l, k, v, vp in _lam_sweep(case["lmax"], case["mmax"], th):
            A = ri[_index(case, l, k)][:, :, None]
            F[:k].addcmul_(A, v[:, None])
            if deriv and l > 0:
                q = torch.sqrt((2.0 * l + 1) / (2.0 * l - 1) * (l * l - mm[:k] ** 2))
                D[:k].addcmul_(A, (l * cot * v - q * vp / s)[:, None])
        co, si = _turn(case, phi[c])
        w = _weight(case)
        for i in range(b):
            f[i, c] = (w * (F[:, 2 * i] * co - F[:, 2 * i + 1] * si)).sum(0)
            if deriv:
                ft[i, c] = (w * (D[:, 2 * i] * co - D[:, 2 * i + 1] * si)).sum(0)
                fp[i, c] = (-w * mm * (F[:, 2 * i] * si + F[:, 2 * i + 1] * co)).sum(0)
    return (f, ft, fp) if deriv else f


def _direct_adjoint(case, theta, phi, maps):
    b, n = maps.shape
    out = torch.zeros(_nalm(case), 2 * b, dtype=torch.float64, device=DEV)
    for c in _chunks(case, n, b):
        co, si = _turn(case, phi[c])
        G = torch.stack([x for i in range(b) for x in (maps[i, c] * co, -maps[i, c] * si)], 1)
        for l, k, v, _ in _lam_sweep(case["lmax"], case["mmax"], theta[c]):
            out[_index(case, l, k)] += torch.matmul(G[:k], v[:, :, None])[:, :, 0]
    out[: case["lmax"] + 1, 1::2] = 0.0
    return torch.view_as_complex(out.reshape(-1, b, 2).permute(1, 0, 2).contiguous())


def _spin_sweep(case, theta):
    """Yields (l, p, q), rows m = 0 .. mmax: the functions of spin s and -s of degree l (zero for
    l < max(m, s)), from the three-term recurrence of Wigner's d started at l = max(m, s)."""
    s, m1 = case["spin"], case["mmax"] + 1
    m = torch.arange(m1, dtype=torch.float64, device=DEV)
    l0, lo = m.clamp_min(s), m.clamp_max(s)
    ln = 0.5 * (torch.log((2 * l0 + 1) / (4 * math.pi)) + torch.lgamma(2 * l0 + 1)
                - torch.lgamma(l0 + lo + 1) - torch.lgamma(l0 - lo + 1))
    sh, ch = torch.sin(0.5 * theta), torch.sin(0.5 * (math.pi - theta))
    ls, lc = torch.log(sh)[None], torch.log(ch)[None]
    d, t = (m - s).abs()[:, None], (m + s)[:, None]
    odd = torch.where(m % 2 == 1, -1.0, 1.0)
    p0 = odd[:, None] * torch.exp(ln[:, None] + d * lc + t * ls)
    q0 = torch.where(m >= s, odd, (-1.0) ** s)[:, None] * torch.exp(ln[:, None] + t * lc + d * ls)
    x = torch.where(theta <= 0.5 * math.pi, 1.0 - 2.0 * sh * sh, 2.0 * ch * ch - 1.0)
    p, q, pp, qp = (torch.zeros_like(p0) for _ in range(4))
    for l in range(case["lmax"] + 1):
        c, live = l - 1.0, (l0 < l)[:, None]
        if l > s:
            dc = torch.sqrt(((c * c - m * m) * (c * c - s * s)).clamp_min(0.0))
            d1 = torch.sqrt(((l * l - m * m) * (l * l - s * s)).clamp_min(1e-300))
            r = math.sqrt((2 * c + 3) * (2 * c + 1))
            al = (r * l / d1)[:, None]
            be = (r * m * s / (max(c, 1.0) * d1))[:, None]
            ga = (math.sqrt((2 * c + 3) / (2 * c - 1)) * l * dc / (max(c, 1.0) * d1))[:, None] if c > 0.5 else 0.0 * al
            pn, qn = (al * x + be) * p - ga * pp, (al * x - be) * q - ga * qp
            pp, qp = p, q
            p, q = torch.where(live, pn, 0.0), torch.where(live, qn, 0.0)
        here = (l0 == l)[:, None]
        p, q = torch.where(here, p0, p), torch.where(here, q0, q)
        yield l, p, q


def _direct_spin(case, theta, phi, alm, maps):
    """Q + iU = sum s_a sY with s_a = -(G + iC) and its transpose."""
    n, sg = theta.numel(), (-1.0) ** case["spin"]
    qu = torch.zeros(2, n, dtype=torch.float64, device=DEV)
    gc = torch.zeros(2, _nalm(case), dtype=torch.complex128, device=DEV)
    al = alm[0].clone()
    al[:, : case["lmax"] + 1] = al[:, : case["lmax"] + 1].real.to(torch.complex128)
    w = _weight(case)
    for c in _chunks(case, n, 6):
        co, si = _turn(case, phi[c])
        e = torch.complex(co, si)
        Q, U = torch.zeros_like(e), torch.zeros_like(e)
        mq, mu = maps[0, 0, c] * e.conj(), maps[0, 1, c] * e.conj()
        for l, p, q in _spin_sweep(case, theta[c]):
            k = min(l, case["mmax"]) + 1
            ix = _index(case, l, k)
            wp, wm = 0.5 * (p + sg * q)[:k], 0.5 * (p - sg * q)[:k]
            G, C = al[0][ix][:, None], al[1][ix][:, None]
            Q[:k] -= G * wp + 1j * C * wm
            U[:k] -= C * wp - 1j * G * wm
            gc[0][ix] -= (mq[:k] * wp + 1j * mu[:k] * wm).sum(1)
            gc[1][ix] -= (mu[:k] * wp - 1j * mq[:k] * wm).sum(1)
        qu[0, c], qu[1, c] = (w * (Q * e).real).sum(0), (w * (U * e).real).sum(0)
    gc[:, : case["lmax"] + 1] = gc[:, : case["lmax"] + 1].real.to(torch.complex128)
    l, _ = _degrees(case)
    gc[:, l < case["spin"]] = 0.0
    return qu[None], gc[None]


def _direct_solve(case, theta, phi, d):
    """CGLS on min ||S a - d|| in <a, b>_m, from zero."""
    wt = torch.full((_nalm(case),), 2.0, dtype=torch.float64, device=DEV)
    wt[: case["lmax"] + 1] = 1.0

    def dot(a):
        return (wt * (a.real ** 2 + a.imag ** 2)).sum()

    x = torch.zeros(_nalm(case), dtype=torch.complex128, device=DEV)
    u = d.clone()
    s = _direct_adjoint(case, theta, phi, u[None])[0]
    p, gam = s.clone(), dot(s)
    for _ in range(case["iters"]):
        q = _direct_synthesis(case, theta, phi, p[None])[0]
        al = gam / (q * q).sum()
        x, u = x + al * p, u - al * q
        s = _direct_adjoint(case, theta, phi, u[None])[0]
        new = dot(s)
        p, gam = s + (new / gam) * p, new
    return x, None, float(u.norm() / d.norm())


def _direct_learn(case, d):
    """Density, features and the network with its parameter gradient, in 64 bits."""
    nt, npj, n = 64, 128, d["theta"].numel()
    th, pw = d["theta"], torch.remainder(d["phi"], 2 * math.pi)
    a, b = (th * (nt / math.pi)).long().clamp(0, nt - 1), (pw * (npj / (2 * math.pi))).long().clamp(0, npj - 1)
    cnt = torch.bincount(a * npj + b, minlength=nt * npj).reshape(nt, npj).double()
    e = torch.arange(nt + 1, dtype=torch.float64, device=DEV) * (math.pi / nt)
    area = (torch.cos(e[:-1]) - torch.cos(e[1:])) * (2 * math.pi / npj)
    lr = torch.log((cnt / (n * area[:, None] / (4 * math.pi))).clamp_min(1e-3))

    def at(i, j):
        return lr[i.clamp(0, nt - 1), torch.remainder(j, npj)]

    u, v = th * (nt / math.pi) - 0.5, pw * (npj / (2 * math.pi)) - 0.5
    i, j = torch.floor(u).long(), torch.floor(v).long()
    fu, fv = u - i, v - j
    cols = [(1 - fu) * ((1 - fv) * at(i, j) + fv * at(i, j + 1)) + fu * ((1 - fv) * at(i + 1, j) + fv * at(i + 1, j + 1))]
    cols += [at(a + x, b + y) for x in (-1, 0, 1) for y in (-1, 0, 1)] + [torch.cos(th), torch.sin(th)]
    feat = torch.stack(cols, 1)
    prm = d["params"].double()
    sizes, o, lay = learned.SIZES, 0, []
    for k in range(len(sizes) - 1):
        w = prm[o:o + sizes[k] * sizes[k + 1]].reshape(sizes[k], sizes[k + 1])
        o += w.numel()
        lay.append((w, prm[o:o + sizes[k + 1]]))
        o += sizes[k + 1]
    acts, h = [], feat
    for w, bias in lay[:-1]:
        acts.append(h)
        h = torch.tanh(h @ w + bias)
    acts.append(h)
    z = (h @ lay[-1][0] + lay[-1][1])[:, 0]
    scale = 4 * math.pi / n
    delta, out = (d["grad_w"].double() * scale * torch.sigmoid(z))[:, None], []
    for k in range(len(lay) - 1, -1, -1):
        out = [(acts[k].T.contiguous() @ delta).reshape(-1), delta.sum(0)] + out
        if k:
            delta = (delta @ lay[k][0].T.contiguous()) * (1 - acts[k] ** 2)
    return feat, torch.nn.functional.softplus(z) * scale, torch.cat(out)


def exact(case, seed):
    kind, n, b = case["kind"], _npts(case), case["nmaps"]
    cost = float(_nalm(case)) * n * {"grad": 3 + 3 * b, "solve": 5.0 * case.get("iters", 0), "spin": 30.0,
                                     "learn": 0.0}.get(kind, 2 + b)
    if cost > 1e12 or case["lmax"] > (900 if kind == "spin" else 1500) and kind != "learn":
        return None
    d = _inputs(case, seed)
    if kind == "learn":
        return _direct_learn(case, d)
    th, ph = d["theta"], d["phi"]
    if kind == "synthesis":
        return _direct_synthesis(case, th, ph, d["alm"])
    if kind == "adjoint":
        return _direct_adjoint(case, th, ph, d["map"])
    if kind == "spin":
        return _direct_spin(case, th, ph, d["alm"], d["map"])
    if kind == "solve":
        return _direct_solve(case, th, ph, d["map"])
    f, ft, fp = _direct_synthesis(case, th, ph, d["alm"], deriv=True)
    g = d["w"] * f
    ga = _direct_adjoint(case, th, ph, g)
    ga[:, case["lmax"] + 1:] *= 2.0
    return [f, ga, (g * ft).sum(0), (g * fp).sum(0)]
