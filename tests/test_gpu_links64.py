"""The FP64 stencil on two rows of each link and the third row's difference from
its rebuild: the same operator as on the full links, and the full links where
the difference does not fit."""
import numpy as np
import pytest

import synth
from gpu_util import max_rel_elem, require_gpu, to_dev, to_host
from oracle.lattice import WilsonKernel

pytestmark = pytest.mark.gpu


# links in SU(3) to rounding; off by 2^-44 (just inside the limit of 2^-43); off
# by 2^-40 (outside it: full links, while FP32 and FP16 still use two rows)
@pytest.mark.parametrize("off", [0.0, 2.0**-44, 2.0**-40])
@pytest.mark.parametrize("dims", [(5, 3, 7, 9), (8, 8, 8, 16)])
def test_fp64_links(dims, off):
    ovl = require_gpu()
    U = synth.gauge_field(dims, 23, 0.3)
    rng = np.random.default_rng(3)
    U[:, :, 2] += off * rng.uniform(-1.0, 1.0, U[:, :, 2].shape)
    psi = np.stack([synth.gaussian_source(dims, 70 + i) for i in range(2)])
    ora = WilsonKernel(dims, U, 1.4)
    ctx = ovl.Context(dims)
    ctx.gauge_load(to_dev(U))
    assert ctx.gauge_info()[1]
    two = to_host(ctx.wilson_dslash(to_dev(psi)))
    ctx.set_option(ovl.OPT_TWO_ROW_LINKS, 0)
    full = to_host(ctx.wilson_dslash(to_dev(psi)))
    for f in range(2):
        assert max_rel_elem(two[f], ora.hop(psi[f])) < 1e-14, f
        assert max_rel_elem(full[f], ora.hop(psi[f])) < 1e-14, f
        # eight hops of three products each, links equal to 2^-54, |psi| up to the
        # field's largest component: at most 24 * 2 * 2^-54 = 2.7e-15 of it
        assert max_rel_elem(two[f], full[f]) < 2.7e-15, f
        if off == 2.0**-40:
            assert np.array_equal(two[f], full[f]), f
    ctx.close()
