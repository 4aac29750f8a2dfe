"""Right-hand sides that are skipped (here: zero ones, which are solved from the
start) do not split a sign call into batches: twelve right-hand sides of which
two are non-zero, apart from each other, take the updates that the two take
alone; and where batches are made, one without any active field costs none."""
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

DIMS = (16, 16, 16, 32)   # four FP32 fields of it make a batch


def _solve(ovl, which, n):
    import torch
    ctx = ovl.Context(DIMS)
    ctx.gauge_generate(5, 0.25)
    z = ovl.zolotarev_coeffs(10, 0.5, 6.6)
    b = torch.zeros((n, ctx.V, 4, 3), dtype=torch.complex128, device="cuda")
    for k, f in enumerate(which):
        b[f] = ctx.source(ovl.SRC_GAUSS, seed=40 + k)
    # FP32 throughout: two short middle solves
    p = ovl.solver_defaults(rho=1.4, mu=0.2, tol=1e-2, eta_tilde=1e-1, f32_threshold=1e-9, half_threshold=2.0)
    ctx.profile(True)
    x, st, _ = ctx.solve(b, z, p)
    launches = ctx.profile_read(ovl.KERN_SHIFT, ovl.F32)["launches"]
    out = x[list(which)].cpu()
    for f in set(range(n)) - set(which):
        assert not x[f].any()
    ctx.close()
    return out, launches, st


def test_two_active_of_twelve():
    ovl = require_gpu()
    alone, l2, _ = _solve(ovl, (0, 1), 2)
    among, l12, st = _solve(ovl, (0, 11), 12)
    for f in range(2):   # each solved to 1e-2 in FP32
        assert float((alone[f] - among[f]).norm()) <= 4e-2 / 0.2 * float(alone[f].norm())
    assert all(st[f].mscg_iters == 0 for f in range(1, 11))
    # one launch shape differs from the other: a sign call may stop an iteration
    # (of some thirty) earlier or later
    assert l12 <= 1.1 * l2, (l2, l12)


def test_batch_without_an_active_field():
    ovl = require_gpu()
    six, l6, _ = _solve(ovl, (0, 1, 2, 3, 4, 5), 6)        # two batches of three
    among, l12, _ = _solve(ovl, (0, 1, 2, 3, 4, 5), 12)    # two batches of six, the second without any
    for f in range(6):
        assert float((six[f] - among[f]).norm()) <= 4e-2 / 0.2 * float(six[f].norm())
    assert l12 <= l6, (l6, l12)
