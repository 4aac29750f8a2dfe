"""The launch shape of H and K with the store of the entry points (canonical
layout) is timed with that store and kept apart from that of K inside the sign
function; a table that has K only once sets both."""
import numpy as np
import pytest

import synth
from gpu_util import require_gpu, to_dev

pytestmark = pytest.mark.gpu

K, K_CANON = 1, 4


def _key(prec, epi, nf):
    return (prec * 8 + epi) * 64 + nf


def test_k_of_the_entry_point_has_its_own_choice():
    ovl = require_gpu()
    dims = (4, 4, 4, 6)
    ctx = ovl.Context(dims)
    ctx.gauge_load(to_dev(synth.gauge_field(dims, 8, 0.25)))
    psi = to_dev(synth.gaussian_source(dims, 90))
    z = ovl.zolotarev_coeffs(8, 0.5, 6.6)
    for prec in (ovl.F64, ovl.F32, ovl.HALF):
        ctx.sign(psi, 1.4, z, 1e-2, prec)
        assert _key(prec, K, 1) in ctx.tuning() and _key(prec, K_CANON, 1) not in ctx.tuning()
        ctx.kernel_K_apply(psi, 1.4, prec)
        assert _key(prec, K_CANON, 1) in ctx.tuning()
        # a table with one choice for K, then one with both
        ctx.set_tuning({_key(prec, K, 1): 3})
        assert ctx.tuning()[_key(prec, K, 1)] == ctx.tuning()[_key(prec, K_CANON, 1)] == 3
        ctx.set_tuning({_key(prec, K, 1): 0, _key(prec, K_CANON, 1): 2})
        assert (ctx.tuning()[_key(prec, K, 1)], ctx.tuning()[_key(prec, K_CANON, 1)]) == (0, 2)
    ctx.close()


def test_canonical_store_is_what_is_timed():
    """The timing of H in FP16 stores complex128 rows, so its scratch is a field
    of those (192 bytes per site; a packed field has 52)."""
    ovl = require_gpu()
    dims = (8, 8, 8, 16)
    V = int(np.prod(dims))
    ctx = ovl.Context(dims)
    ctx.gauge_load(to_dev(synth.gauge_field(dims, 8, 0.25)))
    psi = to_dev(synth.gaussian_source(dims, 90))
    before = ctx.device_bytes
    ctx.wilson_dslash(psi, ovl.HALF)
    assert ctx.device_bytes - before >= V * (52 + 192)   # packed input, timed output
    ctx.close()
