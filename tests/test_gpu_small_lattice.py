"""The stencil with eight lanes per site (launch variant 22), against the
oracle's operator on lattices whose volume fills its 64-site blocks exactly,
leaves a remainder, or is less than one block."""
import numpy as np
import pytest

import synth
from gpu_util import max_rel_elem, rel, require_gpu, to_dev, to_host
from oracle.lattice import WilsonKernel

pytestmark = pytest.mark.gpu

VARIANT = 22


def _tuning(prec, nf):
    return {(prec * 8 + e) * 64 + nf: VARIANT for e in range(4)}


# 16 sites (a quarter of a block), 72 (a block and a remainder), 3 x 64, 5 x 3 x 7 x 9
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 3, 3, 4), (4, 4, 2, 6), (5, 3, 7, 9)])
@pytest.mark.parametrize("two_row", [True, False])
def test_eight_lanes_per_site(dims, two_row):
    ovl = require_gpu()
    from oracle import krylov
    from oracle.zolotarev import Zolotarev
    U = synth.gauge_field(dims, 21, 0.3)
    ora = WilsonKernel(dims, U, 1.4)
    psi = np.stack([synth.gaussian_source(dims, 50 + i) for i in range(3)])
    psi[2, 1:] = 0.0   # a field that is zero off one site
    z = Zolotarev(12, 0.2, 6.6)
    zg = ovl.zolo_from(z.nz, z.a, z.b, z.delta, z.omega, z.sigma)
    sref = krylov.SignFunction(ora, z)(psi[0], 1e-14)
    tol = {ovl.F64: 1e-14, ovl.F32: 2e-6, ovl.HALF: 5e-3}     # the bounds of the other variants
    stol = {ovl.F64: 1e-12, ovl.F32: 1e-5, ovl.HALF: 1e-2}
    eta = {ovl.F64: 1e-13, ovl.F32: 1e-6, ovl.HALF: 1e-2}
    for prec in (ovl.F64, ovl.F32, ovl.HALF):
        print("case", dims, two_row, prec, flush=True)
        ctx = ovl.Context(dims)
        ctx.set_option(ovl.OPT_TWO_ROW_LINKS, two_row)
        ctx.gauge_load(to_dev(U))
        ctx.set_tuning({**_tuning(prec, 1), **_tuning(prec, 3)})
        h = to_host(ctx.wilson_dslash(to_dev(psi), prec=prec))
        k = to_host(ctx.kernel_K_apply(to_dev(psi), 1.4, prec=prec))
        for f in range(3):
            assert max_rel_elem(h[f], ora.hop(psi[f])) < tol[prec], (prec, f)
            if prec == ovl.HALF:
                assert rel(k[f], ora.K(psi[f])) < 2e-3, (prec, f)
            else:
                assert max_rel_elem(k[f], ora.K(psi[f])) < tol[prec], (prec, f)
        s = to_host(ctx.sign(to_dev(psi[0]), 1.4, zg, eta[prec], prec=prec)[0])
        assert rel(s, sref) < stol[prec], prec
        assert ctx.tuning()[(prec * 8 + 2) * 64 + 1] == VARIANT
        ctx.close()


def test_eight_lanes_limit():
    """Refused above 65536 sites, accepted at the limit."""
    ovl = require_gpu()
    ctx = ovl.Context((16, 16, 16, 16))
    ctx.set_tuning(_tuning(ovl.F32, 1))
    ctx.close()
    ctx = ovl.Context((16, 16, 16, 17))
    with pytest.raises(ovl.OvlError):
        ctx.set_tuning(_tuning(ovl.F32, 1))
    ctx.close()
