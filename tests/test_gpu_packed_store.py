"""Every stencil launch variant with its packed store and several fields (the
entry points of H and K store in the canonical layout): K and K^2 + sigma with
their dot products inside the sign function of five fields, K y + x with exact
low modes, in every precision, against the oracle."""
import functools

import numpy as np
import pytest

import synth
from gpu_util import require_gpu, rel, to_dev, to_host
from oracle import krylov
from oracle.lattice import WilsonKernel
from oracle.zolotarev import Zolotarev

pytestmark = pytest.mark.gpu

NF = 5   # more than a group of four fields


@functools.lru_cache(maxsize=None)
def _problem(dims):
    U = synth.gauge_field(dims, 17, 0.3)
    k = WilsonKernel(dims, U, 1.4)
    z = Zolotarev(10, 0.3, 6.6)
    psi = np.stack([synth.gaussian_source(dims, 30 + f) for f in range(NF - 1)] + [synth.point_source(dims, 9, 3, 0)])
    sign = krylov.SignFunction(k, z)
    return U, z, psi, [sign(p, 1e-13) for p in psi]


# columns and t chunks fit; none of them does
@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (5, 3, 7, 3)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_every_variant(dims, prec):
    ovl = require_gpu()
    U, z, psi, want = _problem(dims)
    zg = ovl.zolo_from(z.nz, z.a, z.b, z.delta, z.omega, z.sigma)
    eta, tol = {0: (1e-13, 1e-12), 1: (1e-6, 1e-5), 2: (1e-2, 2e-2)}[prec]   # of the call, and with the storage's own
    dev = to_dev(psi)
    ctx = ovl.Context(dims)
    ctx.gauge_load(to_dev(U))
    evals, _ = ctx.lowmodes_compute(1.4, 2, tol=1e-11)
    evecs = ctx.lowmodes_get()
    ctx.close()
    ran = 0
    for v in range(ovl.N_STENCIL_VARIANTS):
        ctx = ovl.Context(dims)
        ctx.gauge_load(to_dev(U))
        try:
            ctx.set_tuning({(prec * 8 + e) * 64 + NF: v for e in (1, 2, 3)})
        except ovl.OvlError:
            ctx.close()
            continue
        ran += 1
        print("case", dims, prec, "variant", v, flush=True)
        got = to_host(ctx.sign(dev, 1.4, zg, eta, prec=prec)[0])
        for f in range(NF):
            assert rel(got[f], want[f]) < tol, (v, f)
        # two exact modes: the same function, the modes' part added by K y + x
        ctx.lowmodes_set(evals, evecs)
        got = to_host(ctx.sign(dev, 1.4, zg, eta, prec=prec)[0])
        for f in range(NF):
            assert rel(got[f], want[f]) < tol + 2 * z.delta, (v, f)
        ctx.close()
    assert ran >= 9
