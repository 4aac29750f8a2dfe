"""Several FP16 fields on lattices whose volume is no multiple of four: a
field's scales (four bytes per site) then end inside a 16-byte word, and the
next field must start after it."""
import numpy as np
import pytest

import synth
from gpu_util import max_rel_elem, require_gpu, to_dev, to_host
from oracle.lattice import WilsonKernel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(5, 3, 7, 9), (3, 3, 3, 2), (3, 5, 3, 7)])   # remainders 1, 2, 3
def test_fp16_fields_do_not_overlap(dims):
    ovl = require_gpu()
    U = synth.gauge_field(dims, 21, 0.3)
    ora = WilsonKernel(dims, U, 1.4)
    psi = np.stack([synth.gaussian_source(dims, 60 + i) for i in range(3)])
    ctx = ovl.Context(dims)
    ctx.gauge_load(to_dev(U))
    h = to_host(ctx.wilson_dslash(to_dev(psi), prec=ovl.HALF))
    for f in range(3):
        assert max_rel_elem(h[f], ora.hop(psi[f])) < 5e-3, f   # the storage's bound, as for one field
    ctx.close()
