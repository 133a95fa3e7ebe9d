"""Every run length of the chained MFMA apply (orders p >= 5).

The length follows from the elements of a resident workgroup: 64 elements on 1 to 64 workgroups
are 64 to 1 each, on both sides of every step of the rule (2, 3, 5 and 32), so each order, Q and
operator runs its kernel without runs and, where the rule has them, every length of runs.
Reference: the CPU oracle; the bar is the parity tests' 1e-12 (sums of at most ~10^3 products
in FP64).
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [5, 6, 7, 8])
@pytest.mark.parametrize("dq", [1, 2])
def test_run_lengths(p, dq):
    import torch
    from paper_2603_09038_amd import hexpa as hx
    mesh = synth.box_mesh(4, perturb=0.1, seed=p)
    for ops in (hx.PA_MASS, hx.PA_DIFFUSION, hx.PA_MASS | hx.PA_DIFFUSION):
        op = hx.PAOperator(mesh, p, p + dq, ops=ops)
        op.set_variant(hx.PA_VARIANT_MFMA)
        x = synth.rand_x(op.ndof, p)
        ref = oracle.Problem(mesh, p, p + dq, ops=ops).apply(x)
        xt = torch.tensor(x, device="cuda")
        for cap in (1, 2, 3, 9, 12, 16, 21, 32, 64):
            op.set_grid_cap(cap)
            err = np.linalg.norm(op.apply(xt).cpu().numpy() - ref) / np.linalg.norm(ref)
            assert err <= 1e-12, (p, dq, ops, cap, err)
        op.close()
