"""Timed workloads of the overlap library, through its Python entry points.

A case names one operation, its lattice (extents x, y, z, t), its number of
right-hand sides and its arithmetic:

  dslash, kernel   the hopping term H and the kernel K alone
  sign, overlap    sign(K) and D[mu] by the multi-shift CG over 20 poles
  adjoint          D^dagger chi and the link gradient of Re(chi^H D psi)
  solve            D[mu] x = b to 1e-10 by GMRESR(relSUMR), mixed precision

The links are exp(i eps A) with Gaussian A in su(3), eps = 0.25, and the
sources complex Gaussian noise; the Zolotarev interval comes from the library's
Lanczos estimate, as in the benchmark.  Single-precision results are kept as
complex64, which is what they are good for; a solve returns its solution.

Lattices run from 4^4 to 32^3 x 64, one to twelve right-hand sides.
"""
import math

import numpy as np
import torch

import paper_1501_01855_amd as ovl

RHO, MU, EPS, POLES = 1.4, 0.05, 0.25, 20
B_MAX = 8.0 - RHO          # rigorous bound on |K|
A_LOW = 0.3                # below min |K| on these links, for the 64-bit values
ETA = {"f64": 1e-10, "f32": 1e-5}
PREC = {"f64": ovl.F64, "f32": ovl.F32}


def _case(op, x, y, z, t, nrhs, prec, name=None):
    c = {"op": op, "x": x, "y": y, "z": z, "t": t, "nrhs": nrhs, "prec": prec}
    return dict(c, name=name) if name else c


def listed():
    return [
        # latency of one hop on a small lattice: what a user's own Krylov code calls in a loop
        _case("dslash", 8, 8, 8, 16, 1, "f64", "dslash_8c16_f64"),
        # all spin-colour components of a propagator at once, on the benchmark's lattice
        _case("dslash", 24, 24, 24, 48, 12, "f64", "dslash_24c48_12rhs_f64"),
        # extents that no tile divides, a few right-hand sides
        _case("kernel", 15, 9, 21, 27, 3, "f64", "kernel_odd_3rhs_f64"),
        # the stencil at the largest lattice of the benchmark, single precision
        _case("kernel", 32, 32, 32, 64, 1, "f32", "kernel_32c64_f32"),
        # the sign function on the lattice of the derivative workload: launches and waits count
        _case("sign", 8, 8, 8, 16, 1, "f64", "sign_8c16_f64"),
        # relaxed sign calls of an outer solver, twelve sources together
        _case("sign", 16, 16, 16, 32, 12, "f32", "sign_16c32_12rhs_f32"),
        # the operator itself: odd extents, then the benchmark's lattice
        _case("overlap", 15, 9, 21, 27, 1, "f64", "overlap_odd_f64"),
        _case("overlap", 24, 24, 24, 48, 1, "f64", "overlap_24c48_f64"),
        # backward passes: the small double-precision and the large single-precision one
        _case("adjoint", 8, 8, 8, 16, 1, "f64", "adjoint_8c16_f64"),
        _case("adjoint", 32, 32, 32, 64, 1, "f32", "adjoint_32c64_f32"),
        # whole solves in mixed precision (FP16 storage inside): a small and a large lattice
        _case("solve", 8, 8, 8, 16, 1, "mixed", "solve_8c16_mixed"),
        _case("solve", 24, 24, 24, 48, 1, "mixed", "solve_24c48_mixed"),
    ]


# volume times right-hand sides at most, per operation and arithmetic
_MOST = {("dslash", "f64"): 12 * 24**3 * 48, ("dslash", "f32"): 12 * 24**3 * 48,
         ("kernel", "f64"): 12 * 24**3 * 48, ("kernel", "f32"): 12 * 24**3 * 48,
         ("sign", "f64"): 24**3 * 48, ("sign", "f32"): 12 * 16**3 * 32,
         ("overlap", "f64"): 24**3 * 48, ("overlap", "f32"): 12 * 16**3 * 32,
         ("adjoint", "f64"): 16**3 * 32, ("adjoint", "f32"): 32**3 * 64,
         ("solve", "mixed"): 20**3 * 40}


def draw(rng):
    op, prec = rng.choice(sorted(_MOST))
    nrhs = rng.choice([1, 1, 1, 2, 3, 4, 6, 12])
    cap = _MOST[op, prec] // nrhs
    low = 4**4
    v = math.exp(rng.uniform(math.log(low), math.log(max(min(cap, 32**3 * 64), 2 * low))))
    side = (v / 2) ** 0.25            # t is about twice the spatial extents
    d = [max(4, min(32, round(side * rng.uniform(0.75, 1.33)))) for _ in range(3)]
    d.append(max(4, min(64, int(v / (d[0] * d[1] * d[2])))))
    return _case(op, *d, nrhs, prec)


# ---------------------------------------------------------------- inputs
def _dims(c):
    return c["x"], c["y"], c["z"], c["t"]


def _vol(c):
    return c["x"] * c["y"] * c["z"] * c["t"]


def _su3_basis(dev):
    lam = torch.zeros(8, 3, 3, dtype=torch.complex128)
    for k, (a, b) in enumerate([(0, 1), (0, 2), (1, 2)]):
        lam[2 * k, a, b] = lam[2 * k, b, a] = 1
        lam[2 * k + 1, a, b], lam[2 * k + 1, b, a] = -1j, 1j
    lam[6, 0, 0], lam[6, 1, 1] = 1, -1
    lam[7] = torch.diag(torch.tensor([1.0, 1.0, -2.0], dtype=torch.complex128)) / math.sqrt(3.0)
    return (lam / 2).to(dev)


def _mul3(a, b):
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _links(V, gen, dev):
    """exp(i EPS A): Taylor of a quarter of the exponent, squared twice."""
    out = torch.empty(4 * V, 3, 3, dtype=torch.complex128, device=dev)
    basis = _su3_basis(dev).reshape(8, 9)
    eye = torch.eye(3, dtype=torch.complex128, device=dev)
    step = 1 << 20
    for s in range(0, 4 * V, step):
        n = min(step, 4 * V - s)
        g = torch.randn(n, 8, dtype=torch.float64, device=dev, generator=gen)
        x = sum(g[:, k, None] * basis[k] for k in range(8)).reshape(n, 3, 3) * (0.25j * EPS)
        u = eye.expand(n, 3, 3)
        for k in range(14, 0, -1):
            u = eye + _mul3(x, u) / k
        u = _mul3(u, u)
        out[s:s + n] = _mul3(u, u)
    return out.reshape(V, 4, 3, 3)


def _inputs(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    V, n = _vol(case), case["nrhs"]
    U = _links(V, gen, dev)

    def noise():
        return torch.view_as_complex(torch.randn(n, V, 4, 3, 2, dtype=torch.float64, device=dev, generator=gen))

    return U, noise(), noise() if case["op"] == "adjoint" else None


def prepare(case, seed):
    U, psi, chi = _inputs(case, seed)
    ctx = ovl.Context(_dims(case))
    ctx.gauge_load(U)
    st = {"case": case, "ctx": ctx, "psi": psi, "chi": chi}
    if case["op"] in ("sign", "overlap", "adjoint", "solve"):
        lmin, _, _ = ctx.kernel_interval(RHO)
        st["zolo"] = ovl.zolotarev_coeffs(POLES, 0.95 * lmin, B_MAX)
    if case["op"] == "solve":
        ctx.set_option(ovl.OPT_ADAPTIVE_NZ, True)
        st["params"] = ovl.solver_defaults(rho=RHO, mu=MU, tol=1e-10, eta_tilde=3e-3, f32_threshold=1e-6,
                                           half_threshold=3e-3, max_middle=4000)
    return st


def run(st):
    c, ctx = st["case"], st["ctx"]
    op = c["op"]
    if op == "solve":
        x, _, _ = ctx.solve(st["psi"], st["zolo"], st["params"])
        return x
    prec = PREC[c["prec"]]
    if op == "dslash":
        out = ctx.wilson_dslash(st["psi"], prec)
    elif op == "kernel":
        out = ctx.kernel_K_apply(st["psi"], RHO, prec)
    elif op == "sign":
        out, _ = ctx.sign(st["psi"], RHO, st["zolo"], ETA[c["prec"]], prec)
    elif op == "overlap":
        out, _ = ctx.overlap(st["psi"], RHO, MU, st["zolo"], ETA[c["prec"]], prec)
    else:
        dpsi, dU, _ = ctx.overlap_adjoint(st["psi"], st["chi"], RHO, MU, st["zolo"], ETA[c["prec"]], prec)
        out = [dpsi, dU]
    if c["prec"] == "f32":
        return [o.to(torch.complex64) for o in out] if op == "adjoint" else out.to(torch.complex64)
    return out


# ---------------------------------------------------------------- cost
def work(case):
    """Bytes and operations that the method needs: fields in and out of the call
    once; per CG iteration two applications of K (links read twice, the CG's
    four vectors read and three written) and 16 operations per pole and
    component.  A relaxed solve is counted in FP16 storage."""
    V, n, op, prec = _vol(case), case["nrhs"], case["op"], case["prec"]
    hop = 1320.0 * V * n
    io = 2 * 192.0 * V * n
    S = {"f64": 192.0, "f32": 96.0, "mixed": 52.0}[prec] * V * n
    G = {"f64": 576.0, "f32": 192.0, "mixed": 96.0}[prec] * V
    if op in ("dslash", "kernel"):
        return {"bytes": io + G, "flops": hop + (48.0 * V * n if op == "kernel" else 0.0)}
    cond = B_MAX / 0.6                      # |K| in [0.6, 6.6] on these links

    def cg(eta, poles):
        its = 0.5 * cond * math.log(2.0 / eta)
        return its * (2 * G + 7 * S), its * (2 * hop + 12.0 * V * n * (8 * poles + 40))

    if op in ("sign", "overlap"):
        b, f = cg(ETA[prec], POLES / 2)
        return {"bytes": io + b, "flops": f}
    if op == "adjoint":
        b, f = cg(ETA[prec], POLES / 2)
        return {"bytes": 3 * io + 2 * b + 576.0 * V + 4 * POLES * S,
                "flops": 2 * f + POLES * (2 * hop + 4 * 6 * 72.0 * 4 * V * n)}
    steps = math.log(1e10) / -math.log((1 - MU) / (1 + MU))
    b, f = cg(3e-2, 3)
    return {"bytes": io + steps * (b + 12 * 192.0 * V * n), "flops": steps * f}


# ---------------------------------------------------------------- values in 64 bits
_PERM = torch.tensor([[3, 2, 1, 0], [3, 2, 1, 0], [2, 3, 0, 1], [2, 3, 0, 1]])
_PHASE = torch.tensor([[-1j, -1j, 1j, 1j], [-1, 1, 1, -1], [-1j, 1j, 1j, -1j], [1, 1, 1, 1]], dtype=torch.complex128)


class _Lattice:
    """H, K and functions of K in plain torch: fields [n, V, 4, 3], links [V, 4, 3, 3]."""

    def __init__(self, case, U):
        self.d, self.V, self.U = _dims(case), _vol(case), U

    def shift(self, f, mu, by):
        x, y, z, t = self.d
        g = f.reshape(f.shape[0], t, z, y, x, -1)
        return torch.roll(g, by, 4 - mu).reshape(f.shape)

    def hop(self, psi, U=None):
        U = self.U if U is None else U
        out = 0
        for mu in range(4):
            u = U[:, mu]
            pf = self.shift(psi, mu, -1)
            f = sum(u[:, None, :, b] * pf[..., b, None] for b in range(3))
            uc = u.conj()
            b_ = self.shift(sum(uc[:, None, b, :] * psi[..., b, None] for b in range(3)), mu, 1)
            perm, ph = _PERM[mu].to(psi.device), _PHASE[mu].to(psi.device)[:, None]
            out = out + f + b_ + ph * (b_ - f)[:, :, perm]
        return out

    def K(self, psi, U=None):
        o = (4.0 - RHO) * psi - 0.5 * self.hop(psi, U)
        return _g5(o)

    def shifted(self, b, sigma, omega=None):
        """(K^2 + sigma_l)^{-1} b for all l (or their omega-weighted sum), to rounding."""
        L, n = len(sigma), b.shape[0]
        dev = b.device
        sg = torch.tensor(sigma, dtype=torch.float64, device=dev)
        ds = sg - sg[0]
        om = None if omega is None else torch.tensor(omega, dtype=torch.float64, device=dev)

        def dot(u, v):
            return torch.stack([torch.vdot(u[i].flatten(), v[i].flatten()).real for i in range(n)])

        def col(s):
            return s.reshape(n, 1, 1, 1)

        x = torch.zeros_like(b) if om is not None else torch.zeros((L, *b.shape), dtype=b.dtype, device=dev)
        p = b.expand(L, *b.shape).clone()
        r = b.clone()
        rr = dot(r, r)
        bb = rr.clone()
        zeta = torch.ones(L, n, dtype=torch.float64, device=dev)
        zold = torch.ones_like(zeta)
        a_old, b_old = torch.ones_like(rr), torch.zeros_like(rr)
        live = L
        for _ in range(2000):
            w = self.K(self.K(p[0])) + sg[0] * p[0]
            al = rr / dot(p[0], w)
            r -= col(al) * w
            new = dot(r, r)
            be = new / rr
            zn = zeta * zold * a_old / (al * b_old * (zold - zeta) + zold * a_old * (1 + ds[:, None] * al))
            rat = zn / zeta
            for l in range(live):
                c = col(al * rat[l])
                if om is not None:
                    x += (om[l] * c) * p[l]
                else:
                    x[l] += c * p[l]
                p[l] = col(zn[l]) * r + col(be * rat[l] ** 2) * p[l]
            zold, zeta, a_old, b_old, rr = zeta, zn, al, be, new
            while live > 1 and bool((zeta[live - 1] ** 2 * rr <= 1e-30 * bb).all()):
                live -= 1
            if bool((rr <= 1e-26 * bb).all()):
                return x
        return None

    def sign(self, psi):
        sigma, omega = _quadrature(A_LOW, B_MAX)
        y = self.shifted(psi, sigma, omega)
        return None if y is None else self.K(y)


def _g5(f):
    return torch.cat([f[:, :, :2], -f[:, :, 2:]], 2)


def _agm(x, y):
    for _ in range(12):   # converges quadratically
        x, y = 0.5 * (x + y), math.sqrt(x * y)
    return x


def _quadrature(lo, hi):
    """1/|x| = sum omega_l / (x^2 + sigma_l) on [lo, hi] to rounding: the midpoint
    rule for (2/pi) int dt / (x^2 + t^2) under t = lo sn(u)/cn(u), modulus
    k^2 = 1 - (lo/hi)^2, where the integrand is periodic and analytic (the
    conformal-map quadrature of Hale, Higham and Trefethen)."""
    m = 1.0 - (lo / hi) ** 2
    quarter = math.pi / (2 * _agm(1.0, lo / hi))
    # descending Landen / AGM amplitudes
    a, c, b = [1.0], [math.sqrt(m)], lo / hi
    while c[-1] > 1e-17 and len(a) < 20:
        an, cn_ = 0.5 * (a[-1] + b), 0.5 * (a[-1] - b)
        b = math.sqrt(a[-1] * b)
        a.append(an)
        c.append(cn_)
    xs = np.exp(np.linspace(math.log(lo), math.log(hi), 400))
    for n in range(16, 64, 2):
        sigma, omega = [], []
        for j in range(n):
            phi = 2.0 ** (len(a) - 1) * a[-1] * (j + 0.5) * quarter / n
            for k in range(len(a) - 1, 0, -1):
                phi = 0.5 * (phi + math.asin(c[k] / a[k] * math.sin(phi)))
            s, co = math.sin(phi), math.cos(phi)
            dn = math.sqrt(1.0 - m * s * s)
            sigma.append((lo * s / co) ** 2)
            omega.append((2.0 / math.pi) * (quarter / n) * lo * dn / (co * co))
        err = max(abs(1.0 - x * sum(w / (x * x + g) for w, g in zip(omega, sigma))) for x in xs)
        if err < 1e-14:
            break
    return sigma, omega


def exact(case, seed):
    if case["op"] == "solve":
        return None   # thousands of operator applications in this form
    U, psi, chi = _inputs(case, seed)
    lat = _Lattice(case, U)
    op = case["op"]
    if op == "dslash":
        return lat.hop(psi)
    if op == "kernel":
        return lat.K(psi)
    if op == "sign":
        return lat.sign(psi)
    if op == "overlap":
        s = lat.sign(psi)
        return None if s is None else 0.5 * (1 + MU) * psi + 0.5 * (1 - MU) * _g5(s)
    # d/dU of (1 - mu)/2 Re sum_l omega_l [(chi' - K b_l)^H dK a_l - b_l^H dK (K a_l)],
    # chi' = gamma_5 chi, a_l = X_l psi, b_l = X_l K chi', X_l = (K^2 + sigma_l)^{-1}
    sigma, omega = _quadrature(A_LOW, B_MAX)
    cp = _g5(chi)
    dpsi = 0.5 * (1 + MU) * chi
    grad = torch.zeros_like(U)
    leaf = U.clone().requires_grad_(True)
    for f in range(case["nrhs"]):
        s = slice(f, f + 1)
        a = lat.shifted(psi[s], sigma)
        g = lat.shifted(cp[s], sigma)
        if a is None or g is None:
            return None
        for l, w in enumerate(omega):
            b = lat.K(g[l])
            ka = lat.K(a[l])
            left = cp[s] - lat.K(b)
            dpsi[s] += 0.5 * (1 - MU) * w * b
            with torch.enable_grad():
                val = (left.conj() * lat.K(a[l], leaf)).real.sum() - (b.conj() * lat.K(ka, leaf)).real.sum()
                (gu,) = torch.autograd.grad(val, leaf)
            grad += (0.5 * (1 - MU) * w) * gu
    return [dpsi, grad]
