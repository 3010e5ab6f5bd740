"""The work a user of the library has it do, as cases that can be timed and compared.

A case is a dict: the operation (`op`), the lattice (`lx ly lz lt`), the number of
right-hand sides and the options of the entry point.  `prepare` makes what a
program holds before the call (links, sources, the gauge handle), `run` is one call
of a public entry point, `exact` the same result in plain complex128 torch.
The workloads are the repository's own (bench.py, tests/): smooth random links
exp(i eps H) with eps = 0.3 (0.2 for the sign function), Haar links on the smallest
lattice, Gaussian or point sources, kappa 0.12 - 0.1248.
"""
import math

import torch

from paper_2001_05706_amd import wilson as wl

DEV = "cuda"
LINK_BYTES = {("f64", 18): 144, ("f64", 12): 96, ("f32", 18): 72, ("f32", 12): 48, ("f16", 12): 24, ("bf16", 12): 24}
SITE_BYTES = {"f64": 192, "f32": 96, "f16": 52, "bf16": 52}
RHO, LO, HI, SCALE = 1.5, 0.003, 1.0, 42.25  # sign function: valid for any SU(3) links


def _case(op, L, **kw):
    c = {"op": op, "lx": L[0], "ly": L[1], "lz": L[2], "lt": L[3], "nrhs": 1, "prec": "f32", "recon": 12, "eps": 0.3}
    c.update(kw)
    return c


def listed():
    return [
        # one hop on a small lattice: a call's latency, as in a test or a smoothing loop
        _case("dslash", (8, 8, 8, 16), name="hop_f32_8c16", parity=0, dagger=0, kappa=0.12),
        # the whole-lattice operator in FP64 on extents that fit no power of two
        _case("dslash", (12, 14, 10, 18), name="wilson_f64_ragged", parity=-1, dagger=1, kappa=0.1245, prec="f64", recon=18),
        # the D-slash of a propagator: the 12 spin-colour sources of one site
        _case("dslash", (24, 24, 24, 48), name="hop_f32_24c48_12rhs", parity=0, dagger=0, kappa=0.1245, nrhs=12),
        # the D-slash in half-precision storage on the largest lattice
        _case("dslash", (32, 32, 32, 64), name="hop_f16_32c64", parity=1, dagger=1, kappa=0.1248, prec="f16"),
        # the clover operator on an ordinary lattice
        _case("clover", (16, 16, 16, 32), name="clover_f32_16c32", dagger=0, kappa=0.1245, csw=1.0),
        # the smallest exact solve: FP64 on Haar links
        _case("cg", (4, 4, 4, 4), name="cg_f64_4c4", kappa=0.12, tol=1e-12, prec="f64", recon=18, eps=0.0),
        # a mixed-precision solve on an ordinary lattice
        _case("cg", (16, 16, 16, 32), name="cg_f32_16c32", kappa=0.1245, tol=1e-10),
        # the headline of bench.py: FP16 storage on the largest lattice
        _case("cg", (32, 32, 32, 64), name="cg_f16_32c64", kappa=0.1248, tol=1e-10, prec="f16"),
        # a point-to-all propagator: 12 point sources in one batched solve
        _case("cg", (24, 24, 24, 48), name="cg_f32_24c48_12pt", kappa=0.1245, tol=1e-10, nrhs=12, point=True),
        # BiCGStab with half-precision storage
        _case("bicgstab", (24, 24, 24, 48), name="bicgstab_f16_24c48", kappa=0.1245, tol=1e-10, prec="f16"),
        # lattices of uneven size solved together: four of each of 8^4, 12^4, 16^3x32, 24^3x48
        _case("multi", (24, 24, 24, 48), name="multi_f32_uneven", kappa=0.1245, tol=1e-10, copies=4),
        # the kernel of the overlap operator: degree-200 sign function on 12 vectors
        _case("sign", (16, 16, 16, 32), name="sign_f32_16c32_12rhs", nrhs=12, degree=200, eps=0.2),
    ]


def _extents(rng, vmin, vmax):
    """Even extents between 4 and 64 whose volume is about log-uniform in [vmin, vmax], the time extent the longest."""
    for _ in range(1000):
        v = math.exp(rng.uniform(math.log(vmin), math.log(vmax)))
        side = (v / 2) ** 0.25
        L = [max(4, min(32, 2 * round(side * rng.uniform(0.75, 1.3) / 2))) for _ in range(3)]
        t = 2 * round(v / (2 * L[0] * L[1] * L[2]))
        if 4 <= t <= 64 and vmin <= L[0] * L[1] * L[2] * t <= vmax:
            return L[0], L[1], L[2], t
    return 8, 8, 8, 16


def draw(rng):
    op = rng.choice(["dslash", "dslash", "clover", "cg", "cg", "bicgstab", "multi", "sign"])
    prec, recon = rng.choice([("f64", 18), ("f64", 12), ("f32", 12), ("f32", 12), ("f32", 18), ("f16", 12), ("bf16", 12)])
    kappa = rng.choice([0.12, 0.122, 0.1245])
    if op in ("dslash", "clover"):
        nrhs = rng.choice([1, 1, 1, 2, 3, 5, 12])
        L = _extents(rng, 256, 32 ** 3 * 64 if nrhs == 1 else 24 ** 3 * 48 // nrhs * 2)
        kw = {"parity": rng.choice([-1, 0, 1])} if op == "dslash" else {"csw": rng.choice([1.0, 1.7])}
        return _case(op, L, nrhs=nrhs, prec=prec, recon=recon, kappa=kappa, dagger=rng.randrange(2), **kw)
    if op == "multi":
        copies = rng.choice([1, 2, 3])
        return _case(op, _extents(rng, 4096, 24 ** 3 * 48 // copies), kappa=kappa, tol=1e-10, copies=copies, prec=prec, recon=recon)
    if op == "sign":
        nrhs = rng.choice([1, 2, 4, 12])
        return _case(op, _extents(rng, 256, 16 ** 3 * 32 * 2 // nrhs), nrhs=nrhs, degree=rng.choice([20, 60, 100]),
                     eps=0.2, prec=rng.choice(["f32", "f32", "f64"]))
    nrhs = rng.choice([1, 1, 1, 2, 4, 12])
    L = _extents(rng, 256, 24 ** 3 * 48 // nrhs)
    kw = {"csw": 1.0} if rng.random() < 0.25 else {}
    return _case(op, L, nrhs=nrhs, prec=prec, recon=recon, kappa=kappa, tol=1e-10, point=nrhs == 12, **kw)


# ------------------------------------------------------------------ inputs


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) % (1 << 62))


def _gauss(shape, g):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=g, device=DEV, dtype=torch.float64)) * math.sqrt(0.5)


def _mul(a, b):
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _su3(m):
    """Rows 0 and 1 orthonormalised, row 2 = conj(row0 x row1)."""
    r0 = m[..., 0, :] / m[..., 0, :].abs().square().sum(-1, keepdim=True).sqrt()
    r1 = m[..., 1, :] - (r0.conj() * m[..., 1, :]).sum(-1, keepdim=True) * r0
    r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
    return torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj()], dim=-2)


def _links(L, eps, g):
    """(V, 4, 3, 3): exp(i eps H) of traceless GUE matrices H, or Haar links for eps = 0."""
    V = L[0] * L[1] * L[2] * L[3]
    a = _gauss((V, 4, 3, 3), g)
    if eps == 0:
        return _su3(a).contiguous()
    h = (a + a.conj().transpose(-1, -2)) / math.sqrt(2.0)
    h = h - torch.eye(3, device=DEV) * (torch.diagonal(h, dim1=-2, dim2=-1).sum(-1) / 3)[..., None, None]
    ih, u = 1j * eps * h, torch.eye(3, device=DEV, dtype=torch.complex128).expand_as(h)
    for k in range(16, 0, -1):  # Horner form of the exponential series
        u = torch.eye(3, device=DEV) + _mul(ih, u) / k
    return _su3(u).contiguous()


def _systems(c):
    """(extents, right-hand sides) of each system of the case."""
    L = (c["lx"], c["ly"], c["lz"], c["lt"])
    if c["op"] != "multi":
        return [(L, c["nrhs"])]
    vol = L[0] * L[1] * L[2] * L[3]
    sizes = [s for s in ((8, 8, 8, 8), (12, 12, 12, 12), (16, 16, 16, 32)) if s[0] * s[1] * s[2] * s[3] < vol] + [L]
    return [(s, 1) for s in sizes for _ in range(c["copies"])]


def _inputs(c, seed):
    """Links and source of each system, complex128 on the GPU."""
    g = _gen(seed)
    out = []
    for L, n in _systems(c):
        V = L[0] * L[1] * L[2] * L[3]
        U = _links(L, c["eps"], g)
        if c.get("point"):
            eta = torch.zeros((n, V, 4, 3), dtype=torch.complex128, device=DEV)
            site = int(torch.randint(V, (1,), generator=g, device=DEV))
            for r in range(n):
                eta[r, site, r // 3, r % 3] = 1.0
        else:
            eta = _gauss((n, V, 4, 3), g)
        out.append((L, U, eta))
    return out


def prepare(case, seed):
    systems = _inputs(case, seed)
    st = {"case": case, "gauge": [wl.Gauge(L, torch.view_as_real(U)) for L, U, _ in systems],
          "in": [torch.view_as_real(eta) for _, _, eta in systems]}
    st["out"] = [torch.zeros_like(v) for v in st["in"]]
    return st


def run(st):
    c, g, src, out = st["case"], st["gauge"], st["in"], st["out"]
    op, n, prec, recon = c["op"], c["nrhs"], c["prec"], c["recon"]
    if op == "dslash":
        wl.wilson_dslash(g[0], src[0], out[0], n, c["kappa"], c["parity"], c["dagger"], prec, recon)
    elif op == "clover":
        wl.wilson_clover_dslash(g[0], src[0], out[0], n, c["kappa"], c["csw"], c["dagger"], prec, recon)
    elif op == "sign":
        wl.overlap_sign_cheb(g[0], src[0], out[0], n, RHO, c["degree"], LO, HI, SCALE, prec, recon)
    else:
        for x in out:
            x.zero_()  # no initial guess
        if op == "multi":
            m = len(g)
            wl.wilson_cg_multi(g, src, out, [1] * m, [c["kappa"]] * m, c["tol"], 1000, prec, recon)
        elif c.get("csw"):
            solve = wl.wilson_clover_cg if op == "cg" else wl.wilson_clover_bicgstab
            solve(g[0], src[0], out[0], n, c["kappa"], c["csw"], c["tol"], 1000, prec, recon)
        else:
            solve = wl.wilson_cg if op == "cg" else wl.wilson_bicgstab
            solve(g[0], src[0], out[0], n, c["kappa"], c["tol"], 1000, prec, recon)
    return out


# ------------------------------------------------------------------ what a pass cannot do without


def work(c):
    """Canonical FP64 fields read and written once, packed links once per pass over them.

    Solves are counted as 60 CGNR (30 BiCGStab) iterations of 4 hops on the packed
    fields (about what these systems take to 1e-10); the sign function as its
    2 (degree + 1) + 1 applications of H_W."""
    nb = nf = 0.0
    lb, sb = LINK_BYTES[c["prec"], c["recon"]], SITE_BYTES[c["prec"]]
    for L, n in _systems(c):
        V = float(L[0] * L[1] * L[2] * L[3])
        vh = V / 2
        links, canon = 8 * vh * lb, 192 * V * n
        hop, flop = links + 2 * sb * vh * n, 1320 * vh * n
        clov = 288 * vh if c.get("csw") else 0.0
        if c["op"] in ("dslash", "clover"):
            single = c.get("parity", -1) >= 0
            nb += links + canon * (1.5 if single else 2) + 2 * clov
            nf += flop if single else 2 * flop
        elif c["op"] == "sign":
            k = 2 * (c["degree"] + 1) + 1
            nb += 2 * canon + k * (2 * hop + 2 * sb * vh * n)
            nf += 2 * k * flop
        else:
            k = 30 if c["op"] == "bicgstab" else 60
            fields = 17 if c["op"] == "bicgstab" else 10
            nb += 2 * canon + k * (4 * hop + fields * sb * vh * n + 4 * clov)
            nf += k * (4 * flop + 200 * vh * n)
    return {"bytes": nb, "flops": nf}


# ------------------------------------------------------------------ the same in plain torch, complex128

# gamma matrices (DeGrand-Rossi) as {(row, column): entry}
GAMMA = [{(0, 3): 1j, (1, 2): 1j, (2, 1): -1j, (3, 0): -1j}, {(0, 3): -1, (1, 2): 1, (2, 1): 1, (3, 0): -1},
         {(0, 2): 1j, (1, 3): -1j, (2, 0): -1j, (3, 1): 1j}, {(0, 2): 1, (1, 3): 1, (2, 0): 1, (3, 1): 1}]


def _grid(f, L, lead):
    """Site axis -> (t, z, y, x)."""
    return f.reshape(f.shape[:lead] + (L[3], L[2], L[1], L[0]) + f.shape[lead + 1:])


def _col(u, h):
    return sum(u[..., None, :, b] * h[..., b, None] for b in range(3))


def _hop(U, psi, dagger=False):
    """H psi on one field (t, z, y, x, spin, colour), antiperiodic in t."""
    out = torch.zeros_like(psi)
    for mu in range(4):
        ax = 3 - mu
        u = U[..., mu, :, :]
        g = torch.zeros((4, 4), dtype=torch.complex128, device=DEV)
        for (i, j), v in GAMMA[mu].items():
            g[i, j] = v
        for fwd in (True, False):
            sg = (1.0 if dagger else -1.0) * (1.0 if fwd else -1.0)
            # the upper two spin components of (1 + sg gamma) psi fix the lower two
            low = [[j for j in range(4) if (i, j) in GAMMA[mu]][0] for i in range(2)]
            h = torch.stack([psi[..., i, :] + sg * g[i, low[i]] * psi[..., low[i], :] for i in range(2)], dim=-2)
            if fwd:
                h = h.roll(-1, dims=ax)
                if mu == 3:
                    h[-1] *= -1
                h = _col(u, h)
            else:
                h = _col(u.conj().transpose(-1, -2), h).roll(1, dims=ax)
                if mu == 3:
                    h[0] *= -1
            out[..., :2, :] += h
            for i in range(2):
                out[..., low[i], :] += sg * g[low[i], i] * h[..., i, :]
    return out


def _clover(U, kc):
    """A - 1 as (t, z, y, x, 12, 12)."""
    def sh(f, *steps):  # the field at x + steps
        for mu, s in steps:
            f = f.roll(-s, dims=3 - mu)
        return f

    dag = lambda m: m.conj().transpose(-1, -2)  # noqa: E731
    g = torch.zeros((4, 4, 4), dtype=torch.complex128, device=DEV)
    for mu in range(4):
        for (i, j), v in GAMMA[mu].items():
            g[mu, i, j] = v
    A = 0
    for m in range(4):
        for n in range(m + 1, 4):
            um, un = U[..., m, :, :], U[..., n, :, :]
            P = _mul(_mul(um, sh(un, (m, 1))), _mul(dag(sh(um, (n, 1))), dag(un)))
            Q = P
            Q = Q + _mul(_mul(un, dag(sh(um, (n, 1), (m, -1)))), _mul(dag(sh(un, (m, -1))), sh(um, (m, -1))))
            Q = Q + _mul(_mul(dag(sh(um, (m, -1))), dag(sh(un, (m, -1), (n, -1)))),
                         _mul(sh(um, (m, -1), (n, -1)), sh(un, (n, -1))))
            Q = Q + _mul(_mul(dag(sh(un, (n, -1))), sh(um, (n, -1))), _mul(sh(un, (n, -1), (m, 1)), dag(um)))
            F = (Q - dag(Q)) / 8
            s = 0.5j * (g[m] @ g[n] - g[n] @ g[m])
            A = A + 1j * kc * s[:, None, :, None] * F[..., None, :, None, :]
    return A.reshape(A.shape[:4] + (12, 12))


def _apply_clover(A, psi):
    v = psi.reshape(psi.shape[:4] + (12,))
    return psi + sum(A[..., :, j] * v[..., j, None] for j in range(12)).reshape(psi.shape)


def _solve(D, eta, tol):
    """CG on the normal equations, restarted from the true residual until |eta - D x| <= tol |eta|."""
    norm2 = lambda f: f.abs().square().sum()  # noqa: E731
    x, goal = torch.zeros_like(eta), tol * eta.norm()
    for _ in range(4):
        r = eta - D(x)
        if r.norm() <= goal:
            break
        p = s = D(r, True)
        gam = norm2(s)
        for _ in range(400):
            q = D(p)
            al = gam / norm2(q)
            x, r = x + al * p, r - al * q
            if r.norm() <= 0.5 * goal:
                break
            s = D(r, True)
            gam, old = norm2(s), gam
            p = s + (gam / old) * p
    return x


def _inv_sqrt_coeffs(degree):
    n = degree + 1
    th = [math.pi * (k + 0.5) / n for k in range(n)]
    f = [1 / math.sqrt(0.5 * (HI - LO) * math.cos(t) + 0.5 * (HI + LO)) for t in th]
    return [2.0 / n * sum(f[k] * math.cos(j * th[k]) for k in range(n)) for j in range(n)]


def _sign(U, v, degree):
    g5 = torch.tensor([1.0, 1.0, -1.0, -1.0], device=DEV, dtype=torch.float64)[:, None]
    hw = lambda f: g5 * ((4 - RHO) * f - 0.5 * _hop(U, f))  # noqa: E731
    a, b = 2 / ((HI - LO) * SCALE), -(HI + LO) / (HI - LO)
    y = lambda f: a * hw(hw(f)) + b * f  # noqa: E731
    c = _inv_sqrt_coeffs(degree)
    b1, b2 = torch.zeros_like(v), torch.zeros_like(v)
    for j in range(degree, 0, -1):
        b1, b2 = c[j] * v + 2 * y(b1) - b2, b1
    return hw(0.5 * c[0] * v + y(b1) - b2) / math.sqrt(SCALE)


def exact(case, seed):
    c, op, outs = case, case["op"], []
    systems = _inputs(c, seed)
    if op in ("cg", "bicgstab", "multi") and sum(n * L[0] * L[1] * L[2] * L[3] for L, n in _systems(c)) > 3e6:
        return None  # the batched solves: too long in plain torch
    for L, U, eta in systems:
        U, eta = _grid(U, L, 0), _grid(eta, L, 1)
        A = _clover(U, c["kappa"] * c["csw"]) if c.get("csw") else None
        site = (lambda f: f) if A is None else (lambda f: _apply_clover(A, f))
        D = lambda f, dg=False: site(f) - c["kappa"] * _hop(U, f, dg)  # noqa: E731
        res = torch.empty_like(eta)
        for r in range(eta.shape[0]):
            if op == "dslash" and c["parity"] >= 0:
                t, z, y, x = torch.meshgrid(*[torch.arange(n, device=DEV) for n in (L[3], L[2], L[1], L[0])], indexing="ij")
                keep = ((t + z + y + x) % 2 == c["parity"])[..., None, None]
                res[r] = torch.where(keep, _hop(U, eta[r], bool(c["dagger"])), 0)
            elif op in ("dslash", "clover"):
                res[r] = D(eta[r], bool(c["dagger"]))
            elif op == "sign":
                res[r] = _sign(U, eta[r], c["degree"])
            else:
                res[r] = _solve(D, eta[r], 1e-12)
        outs.append(torch.view_as_real(res.reshape(eta.shape[0], -1, 4, 3)))
    return outs
