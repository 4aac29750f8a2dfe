"""Calls with less and less device memory (the context's workspace limit): down to
what they cannot do without they succeed, with shorter rings of residuals and of
SUMR's basis vectors (down to none), with the adjoint's two solves one after the
other and without the FP64 two-row links, and stay within the bounds of the call
with memory to spare; below that they say so, and the context goes on."""
import functools

import numpy as np
import pytest

import synth
from gpu_util import require_gpu, to_dev, to_host
from oracle import adjoint, krylov
from oracle.lattice import WilsonKernel, norm
from oracle.zolotarev import Zolotarev

pytestmark = pytest.mark.gpu

DIMS, RHO, MU = (6, 4, 4, 8), 1.4, 0.1
V = int(np.prod(DIMS))
FIELD = 192 * V          # bytes of an FP64 field
SMALL = 512 * 1024       # partial sums, coefficients, flags: small next to fields on real lattices


@functools.lru_cache(maxsize=None)
def _problem():
    U = synth.gauge_field(DIMS, 15, 0.25)
    z = Zolotarev(10, 0.4, 8.0 - RHO)
    k = WilsonKernel(DIMS, U, RHO)
    return U, z, krylov.SignFunction(k, z)


def _context(ovl, limit=None):
    U, z, _ = _problem()
    ctx = ovl.Context(DIMS)
    ctx.set_option(ovl.OPT_AUTOTUNE, 0)   # no scratch for timing
    ctx.gauge_load(to_dev(U))
    if limit is not None:
        ctx.set_option(ovl.OPT_WORKSPACE_KIB, int(limit) // 1024)
    return ctx, ovl.zolo_from(z.nz, z.a, z.b, z.delta, z.omega, z.sigma)


def _links(ovl):
    """Bytes of the loaded links without the FP64 two-row form (480 of 1776 per
    site), which can go."""
    ctx, _ = _context(ovl)
    held = ctx.device_bytes
    ctx.close()
    return held * 1296 // 1776


def _descend(ovl, call, check, least, unit):
    """call(ctx, zolo) under falling limits, each result checked.  least: the
    bytes beside the links with which it has to succeed; unit: the bytes of the
    fields that an optional buffer is made of.  Such a buffer is taken while it
    is at most a quarter of what is left, so the limits go in such steps."""
    links = _links(ovl)
    held = set()
    for extra in (160, 80, 50, 36, 24, 18, 12, 9, 6, 4, 2, 1, 0):
        limit = links + least + SMALL + extra * unit
        ctx, zg = _context(ovl, limit)
        check(call(ctx, zg))
        print("spare units", extra, "held", (ctx.device_bytes - links - least) / unit, flush=True)
        assert ctx.device_bytes <= limit
        held.add(ctx.device_bytes)
        ctx.close()
    assert len(held) >= 4
    ctx, zg = _context(ovl, links + 0.6 * least)
    with pytest.raises(ovl.OvlError) as e:
        call(ctx, zg)
    assert e.value.code == -3
    ctx.set_option(ovl.OPT_WORKSPACE_KIB, 0)
    check(call(ctx, zg))                 # and the context goes on
    ctx.close()


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_sign(prec):
    ovl = require_gpu()
    _, z, sign = _problem()
    eta, own = {0: (1e-11, 1e-12), 1: (1e-5, 1e-5), 2: (2e-2, 1e-2)}[prec]
    psi = np.stack([synth.gaussian_source(DIMS, 60), synth.point_source(DIMS, 3, 1, 2), synth.gaussian_source(DIMS, 61)])
    want = [sign(p, 1e-13) for p in psi]
    dev = to_dev(psi)

    def check(r):
        got = to_host(r[0])
        for f in range(3):
            assert norm(got[f] - want[f]) <= (eta + own) * norm(psi[f]), f

    # input, output, p, t, w, residual, sum and the shift vectors
    fields = 3 * (7 + z.nz) * {0: 1.0, 1: 0.5, 2: 52 / 192}[prec]
    _descend(ovl, lambda ctx, zg: ctx.sign(dev, RHO, zg, eta, prec=prec), check, fields * FIELD,
             3 * FIELD * {0: 1.0, 1: 0.5, 2: 52 / 192}[prec])


def test_sign_after_larger_calls():
    """What larger calls left is given back for one that needs other buffers."""
    ovl = require_gpu()
    _, z, sign = _problem()
    psi = synth.gaussian_source(DIMS, 62)
    dev = to_dev(np.stack([psi] * 4))
    want = sign(psi, 1e-13)
    links = _links(ovl)
    # FP32 of 12 fields, then FP64 of 4, which need about as much each
    ctx, zg = _context(ovl, links + (12 * (8 + z.nz) * 0.5 + 3 * 4) * FIELD + SMALL)
    for _ in range(2):
        ctx.sign(dev.repeat(3, 1, 1, 1), RHO, zg, 1e-5, prec=ovl.F32)
        got = to_host(ctx.sign(dev, RHO, zg, 1e-11)[0])
        for f in range(4):
            assert norm(got[f] - want) <= 2e-11 * norm(psi)
    ctx.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_adjoint_two_rhs(prec):
    ovl = require_gpu()
    U, z, _ = _problem()
    psi = np.stack([synth.gaussian_source(DIMS, 80), synth.point_source(DIMS, 5, 1, 2)])
    chi = np.stack([synth.gaussian_source(DIMS, 81), synth.gaussian_source(DIMS, 82)])
    ref_U = sum(adjoint.link_gradient(DIMS, U, RHO, z, MU, psi[f], chi[f]) for f in range(2))
    ref_psi = [adjoint.psi_gradient(DIMS, U, RHO, z, MU, chi[f]) for f in range(2)]
    eta, tol = (1e-13, 1e-10) if prec == 0 else (1e-6, 2e-5)
    dpsi_in, dchi_in = to_dev(psi), to_dev(chi)

    def check(r):
        assert norm(to_host(r[1]) - ref_U) <= tol * norm(ref_U)
        for f in range(2):
            assert norm(to_host(r[0])[f] - ref_psi[f]) <= tol * norm(ref_psi[f])

    # FP64: three of the call, chi'; in the precision of the solves: two sources
    # (and chi'), a_l, b_l, K a_l, K b_l and one solve's p, t, w, residual, shift vectors
    S = 1.0 if prec == 0 else 0.5
    fields = 2 * (4 + S * (2 + (prec == 1) + 4 * z.nz + 4 + z.nz))
    _descend(ovl, lambda ctx, zg: ctx.overlap_adjoint(dpsi_in, dchi_in, RHO, MU, zg, eta, prec), check, fields * FIELD,
             2 * S * FIELD)


@pytest.mark.parametrize("restarts", [False, True])
@pytest.mark.parametrize("ladder", ["f64", "mixed"])
def test_solve(ladder, restarts):
    ovl = require_gpu()
    _, z, sign = _problem()
    D = krylov.Overlap(sign, MU)
    b = np.stack([synth.gaussian_source(DIMS, 83), np.zeros((V, 4, 3)), synth.z2_source(DIMS, 84)])
    dev = to_dev(b)
    lo = dict(f32_threshold=2.0, half_threshold=3.0) if ladder == "f64" else dict(f32_threshold=1e-6, half_threshold=3e-3)
    p = ovl.solver_defaults(rho=RHO, mu=MU, tol=1e-9, eta_tilde=1e-3, norm_restart=1e-4 if restarts else 0.1, **lo)
    steps = []

    def check(r):
        x, st, code = r
        assert code == 0
        assert st[1].sumr_iters == 0 and (not restarts or st[0].restarts > 0)
        x = to_host(x)
        for f in (0, 2):
            assert norm(b[f] - D(x[f], 1e-14)) <= 1.1e-9 * norm(b[f]), f
        assert not x[1].any()
        steps.append(st[0].gmresr_steps)

    # of the call, GMRESR's, SUMR's (two basis vectors), the sign function's
    # result, two per outer step, and a sign call's p, t, w, residual, sum and
    # shift vectors; a mixed solve holds FP32 input and output and a set for fields
    # of different precisions besides
    ctx, zg = _context(ovl)
    check(ctx.solve(dev, zg, p))
    ctx.close()
    fields = 3 * (2 + 4 + 7 + 1 + 2 * max(steps) + 5 + z.nz + (0 if ladder == "f64" else 2 * 0.5 + 1))
    _descend(ovl, lambda ctx, zg: ctx.solve(dev, zg, p), check, fields * FIELD, 3 * FIELD)


def test_links_and_low_modes_beyond_the_limit():
    """A load of links that the limit does not allow, then one that it does; the
    low modes likewise."""
    ovl = require_gpu()
    U, z, sign = _problem()
    links = _links(ovl)
    ctx = ovl.Context(DIMS)
    ctx.set_option(ovl.OPT_AUTOTUNE, 0)
    ctx.set_option(ovl.OPT_WORKSPACE_KIB, links // 2048)
    for _ in range(2):
        with pytest.raises(ovl.OvlError) as e:
            ctx.gauge_load(to_dev(U))
        assert e.value.code == -3
    ctx.set_option(ovl.OPT_WORKSPACE_KIB, int(links + (7 + z.nz) * FIELD + SMALL) // 1024)
    ctx.gauge_load(to_dev(U))
    psi = synth.gaussian_source(DIMS, 64)
    zg = ovl.zolo_from(z.nz, z.a, z.b, z.delta, z.omega, z.sigma)
    got = to_host(ctx.sign(to_dev(psi), RHO, zg, 1e-11)[0])
    assert norm(got - sign(psi, 1e-13)) <= 2e-11 * norm(psi)
    import torch
    many = torch.zeros((40, V, 4, 3), dtype=torch.complex128, device="cuda")
    with pytest.raises(ovl.OvlError) as e:
        ctx.lowmodes_set([1.0] * 40, many)
    assert e.value.code == -3
    assert np.array_equal(to_host(ctx.sign(to_dev(psi), RHO, zg, 1e-11)[0]), got)
    ctx.close()
