"""The grouped updates of the multi-shift CG's shift vectors: sign calls that end
within the first group of iterations, between groups and well past them, with
one pole, few and the most, on fields that stop at different iterations (one of
them zero), and on volumes around the update kernels' block sizes."""
import functools

import numpy as np
import pytest

import synth
from gpu_util import require_gpu, to_dev, to_host
from oracle.lattice import WilsonKernel

pytestmark = pytest.mark.gpu

POLES = (1, 6, 64)


@functools.lru_cache(maxsize=None)
def _reference(dims):
    from oracle import krylov
    from oracle.zolotarev import Zolotarev
    U = synth.gauge_field(dims, 31, 0.25)
    ora = WilsonKernel(dims, U, 1.4)
    V = int(np.prod(dims))
    psi = np.stack([synth.gaussian_source(dims, 80), np.zeros((V, 4, 3)), synth.point_source(dims, V - 1, 2, 1)])
    out = {}
    for nz in POLES:
        z = Zolotarev(nz, 0.3, 6.6)
        sign = krylov.SignFunction(ora, z)
        out[nz] = (z, [sign(p, 1e-13) if p.any() else np.zeros_like(p) for p in psi])
    return U, psi, out


@pytest.mark.parametrize("eta", [0.7, 5e-2, 1e-4, 1e-12])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (3, 3, 3, 3), (4, 4, 4, 5)])   # 16, 81 and 320 sites
def test_groups(dims, eta):
    ovl = require_gpu()
    U, psi, ref = _reference(dims)
    ctx = ovl.Context(dims)
    ctx.gauge_load(to_dev(U))
    # the storage's own error of a sign call, as in the other tests of sign(K)
    own = {ovl.F64: 1e-12, ovl.F32: 1e-5, ovl.HALF: 1e-2}
    for nz in POLES:
        z, want = ref[nz]
        zg = ovl.zolo_from(z.nz, z.a, z.b, z.delta, z.omega, z.sigma)
        for prec in (ovl.F64, ovl.F32, ovl.HALF):
            if eta < 0.1 * own[prec] and prec != ovl.F64:
                continue   # not reachable in that storage
            got = to_host(ctx.sign(to_dev(psi), 1.4, zg, eta, prec=prec)[0])
            for f in range(3):
                err = np.linalg.norm(got[f] - want[f])
                assert err <= (eta + own[prec]) * np.linalg.norm(psi[f]), (nz, prec, f, err)
    ctx.close()


def test_batches_match_single_fields():
    """Six FP32 fields of 16^3 x 32, which are solved in two batches (their
    multi-shift CG would leave the Infinity Cache): each as in a call of its own,
    which differs by at most the accuracy of either call and the storage."""
    import torch
    ovl = require_gpu()
    dims, eta = (16, 16, 16, 32), 1e-4
    ctx = ovl.Context(dims)
    ctx.gauge_generate(5, 0.25)
    z = ovl.zolotarev_coeffs(12, 0.5, 6.6)
    psi = torch.stack([ctx.source(ovl.SRC_GAUSS, seed=90 + i) for i in range(6)])
    psi[4] = 0.0
    got, st = ctx.sign(psi, 1.4, z, eta, prec=ovl.F32)
    its = 0
    for f in range(6):
        one, s1 = ctx.sign(psi[f], 1.4, z, eta, prec=ovl.F32)
        its += s1.mscg_iters
        assert float((got[f] - one).norm()) <= (2 * eta + 2e-5) * float(psi[f].norm()), f
    assert abs(st.mscg_iters - its) <= 6   # a stop may move by one iteration with the launch shape
    ctx.close()
