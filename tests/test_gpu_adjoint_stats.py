"""Counters of the adjoint: D^dagger chi takes one application of the sign
function per field, whether the link gradient is wanted with it (whose solutions
give it) or not."""
import pytest

import synth
from gpu_util import require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [1, 2])
@pytest.mark.parametrize("want_links", [True, False])
def test_sign_calls(nrhs, want_links):
    import torch
    ovl = require_gpu()
    dims = (4, 4, 4, 4)
    ctx = ovl.Context(dims)
    ctx.gauge_load(to_dev(synth.gauge_field(dims, 11, 0.3)))
    z = ovl.zolotarev_coeffs(10, 0.25, 6.6)
    f = torch.stack([to_dev(synth.gaussian_source(dims, 80 + i)) for i in range(nrhs)])
    for prec, eta in ((ovl.F64, 1e-10), (ovl.F32, 1e-5)):
        _, _, st = ctx.overlap_adjoint(f, f, 1.4, 0.05, z, eta, prec, want_links=want_links)
        assert st.sign_calls[prec] == nrhs and sum(st.sign_calls) == nrhs
        assert st.mscg_iters > 0
        _, _, st = ctx.overlap_adjoint(f, f, 1.4, 0.05, z, eta, prec, want_psi=not want_links, want_links=want_links)
        assert sum(st.sign_calls) == (0 if want_links else nrhs)
    ctx.close()
