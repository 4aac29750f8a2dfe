"""The FP64 stencil sees every link exactly as loaded, whichever form of the links
it reads: a hop of a point source is one entry of a link (times a phase), and
has to be that entry to the last bit -- on links near one, whose third rows hold
many small entries, and on links whose third row does not fit the two-row form
(exact zeros, whose rebuild is a negative zero), which are read in full."""
import numpy as np
import pytest

import synth
from gpu_util import require_gpu, to_dev, to_host
from oracle.lattice import WilsonKernel

pytestmark = pytest.mark.gpu


# eps of the links; perturbation of the third rows; two-row form expected
CASES = [(0.3, 0.0, True), (1e-3, 0.0, True), (1e-3, 2.0**-50, True), (0.0, 0.0, False)]


@pytest.mark.parametrize("eps,off,two_row", CASES)
@pytest.mark.parametrize("dims", [(3, 3, 3, 4), (5, 3, 7, 9)])
def test_links_bit_for_bit(dims, eps, off, two_row):
    ovl = require_gpu()
    V = int(np.prod(dims))
    if eps:
        U = synth.gauge_field(dims, 41, eps)
    else:
        U = np.tile(np.eye(3, dtype=np.complex128), (V, 4, 1, 1))
    rng = np.random.default_rng(6)
    U[:, :, 2] += off * rng.uniform(-1.0, 1.0, U[:, :, 2].shape)
    ora = WilsonKernel(dims, U, 1.4)
    ctx = ovl.Context(dims)
    ctx.gauge_load(to_dev(U))
    sites = [0, V // 2, V - 1]
    src = np.stack([synth.point_source(dims, s, sp, c) for s in sites for sp in (0, 3) for c in range(3)][:16])
    for variant in (0, 2, 22):
        ctx.set_tuning({(ovl.F64 * 8 + 0) * 64 + len(src): variant})
        got = to_host(ctx.wilson_dslash(to_dev(src)))
        for f in range(len(src)):
            assert np.array_equal(got[f], ora.hop(src[f])), (variant, f)
    # the form that was read, from the bytes of a launch: the links once, 192 in
    # and 192 out per site and field
    ctx.profile(True)
    ctx.wilson_dslash(to_dev(src))
    link_bytes = ctx.profile_read(ovl.KERN_STENCIL, ovl.F64)["bytes"] / V - 384 * len(src)
    assert link_bytes == (480 if two_row else 576)
    ctx.close()


@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (5, 3, 7, 9)])
def test_same_bits_on_either_form(dims):
    """H and K on fields of noise, in every launch variant: the two-row form and
    the full links give the same values to the last bit."""
    ovl = require_gpu()
    psi = to_dev(np.stack([synth.gaussian_source(dims, 50 + f) for f in range(3)]))
    U = to_dev(synth.gauge_field(dims, 41, 0.3))
    ran = 0
    for v in range(ovl.N_STENCIL_VARIANTS):
        out = []
        for two_row in (1, 0):
            ctx = ovl.Context(dims)
            ctx.set_option(ovl.OPT_TWO_ROW_LINKS, two_row)
            ctx.gauge_load(U)
            try:
                ctx.set_tuning({(ovl.F64 * 8 + e) * 64 + 3: v for e in (0, 1)})
            except ovl.OvlError:
                ctx.close()
                break
            out.append([to_host(ctx.wilson_dslash(psi)), to_host(ctx.kernel_K_apply(psi, 1.4))])
            ctx.close()
        if len(out) == 2:
            ran += 1
            for a, b in zip(*out):
                assert np.array_equal(a, b), v
    assert ran >= 9
