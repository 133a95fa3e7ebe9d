"""Vector kernels of the constrained apply and of PCG at the edges of their launches.

ndof 8 (one partial wave), 512 (one whole block of a reduction), 729 (a second, partial block)
and 531441 (1025 reductions' worth for the 1024 blocks; not a multiple of a wave or of the
mask's 32-bit words).  PCG stops on its recursive residual at 1e-10; the recomputed residual
of these well conditioned mass systems differs from it by rounding of the iterates (iterations
x eps x condition, below 1e-11), so 2e-10 is the bar.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (7, 1), (4, 2), (40, 2)]


@pytest.mark.parametrize("n,p", SIZES)
def test_constrained_apply(n, p):
    """y is x on the essential DOFs and A (x without them) elsewhere, also where x is NaN there
    or the buffers are only 8-byte aligned."""
    import torch
    from paper_2603_09038_amd import hexpa as hx
    mesh = synth.box_mesh(n, perturb=0.1, seed=p)
    free = hx.PAOperator(mesh, p, p + 1, ops=hx.PA_MASS)
    op = hx.PAOperator(mesh, p, p + 1, ops=hx.PA_MASS, ess_mode=1)
    k = np.arange(op.ndof)
    M = n * p + 1
    ess = np.zeros(op.ndof, bool)
    for s in (1, M, M * M):
        ess |= (k // s % M == 0) | (k // s % M == M - 1)
    ess = torch.tensor(ess, device="cuda")
    buf = torch.tensor(synth.rand_x(op.ndof + 1, p), device="cuda")
    for off in (0, 1):
        x = buf[off:off + op.ndof]
        want = torch.where(ess, x, free.apply(torch.where(ess, 0.0, x)))
        out = torch.full((op.ndof + 1,), np.nan, dtype=torch.float64, device="cuda")
        got = op.apply_constrained(x, out[off:off + op.ndof])
        assert torch.equal(got[ess], x[ess])
        assert (got - want).norm() <= 1e-13 * want.norm()  # sums of <= 8 elements in any order
        bad = torch.where(ess, np.nan, x)
        got = op.apply_constrained(bad)
        assert got[ess].isnan().all() and (got - want)[~ess].norm() <= 1e-13 * want.norm()
    op.close()
    free.close()


@pytest.mark.parametrize("n,p", SIZES)
@pytest.mark.parametrize("constrained", [False, True])
def test_pcg_residual(n, p, constrained):
    import torch
    from paper_2603_09038_amd import hexpa as hx
    op = hx.PAOperator(synth.box_mesh(n, perturb=0.1, seed=p), p, p + 1, ops=hx.PA_MASS, ess_mode=int(constrained))
    b = torch.tensor(synth.rand_x(op.ndof, 5), device="cuda")
    for mode in (hx.PA_CG_PLAIN, hx.PA_CG_JACOBI):
        x = torch.zeros_like(b)
        hx.cg_solve(op.h, b, x, rtol=1e-10, max_it=2000, mode=mode, check_every=3, constrained=constrained)
        r = b - (op.apply_constrained(x) if constrained else op.apply(x))
        assert r.norm() <= 2e-10 * b.norm(), (mode, float(r.norm() / b.norm()))
    op.close()
