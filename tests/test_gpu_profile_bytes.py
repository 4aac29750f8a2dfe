"""The bytes that the profile of a stencil launch counts: the packed input once,
the links once per launch, and the output as it is stored -- complex128 in the
canonical layout for the entry points of H and K, whatever the precision."""
import numpy as np
import pytest

import synth
from gpu_util import require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf", [1, 3])
@pytest.mark.parametrize("two_row", [True, False])
def test_bytes_of_h_and_k(nf, two_row):
    ovl = require_gpu()
    dims = (4, 4, 4, 6)
    V = int(np.prod(dims))
    ctx = ovl.Context(dims)
    ctx.set_option(ovl.OPT_TWO_ROW_LINKS, two_row)
    ctx.gauge_load(to_dev(synth.gauge_field(dims, 8, 0.25)))
    psi = to_dev(np.stack([synth.gaussian_source(dims, 90 + i) for i in range(nf)]))
    site = {ovl.F64: 192, ovl.F32: 96, ovl.HALF: 52}
    links = {ovl.F64: (480, 576), ovl.F32: (192, 288), ovl.HALF: (96, 144)}
    for prec in (ovl.F64, ovl.F32, ovl.HALF):
        for call in (lambda: ctx.wilson_dslash(psi, prec), lambda: ctx.kernel_K_apply(psi, 1.4, prec)):
            call()   # the launch shapes are timed here
            ctx.profile(True)
            call()
            got = ctx.profile_read(ovl.KERN_STENCIL, prec)
            assert got["launches"] == 1
            assert got["bytes"] == V * (links[prec][0 if two_row else 1] + nf * (site[prec] + 192)), prec
            ctx.profile(False)
    ctx.close()
