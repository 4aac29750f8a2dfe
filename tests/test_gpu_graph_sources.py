"""Graphs of the multi-shift CG under sources that lie in other buffers from call
to call (the basis vectors of an FP64 solve go round a ring): a recorded chunk
does not read the source, so one graph serves them all, with the values of
direct launches bit for bit, also with several right-hand sides that stop at
different iterations."""
import numpy as np
import pytest

import synth
from gpu_util import require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf", [1, 3])
def test_fp64_solve_with_graphs(nf):
    ovl = require_gpu()
    dims = (4, 4, 4, 6)
    U = to_dev(synth.gauge_field(dims, 9, 0.25))
    b = np.stack([synth.gaussian_source(dims, 33 + f) for f in range(nf)])
    if nf > 1:
        b[1] = synth.point_source(dims, 7, 1, 2)
    z = ovl.zolotarev_coeffs(12, 0.4, 6.6)
    p = ovl.solver_defaults(rho=1.4, mu=0.1, tol=1e-9, eta_tilde=1e-3, f32_threshold=2.0, half_threshold=3.0)
    xs = []
    for graphs in (True, False):
        ctx = ovl.Context(dims)
        ctx.gauge_load(U)
        ctx.set_option(ovl.OPT_AUTOTUNE, 0)   # one launch variant: the same tile sums
        ctx.set_option(ovl.OPT_GRAPHS, graphs)
        x, st, code = ctx.solve(to_dev(b), z, p)
        x2, _, _ = ctx.solve(to_dev(b), z, p)   # every graph cached
        assert code == 0 and st[0].sumr_iters > 6
        xs += [to_host(x), to_host(x2)]
        ctx.close()
    for x in xs[1:]:
        assert np.array_equal(x, xs[0])
