"""The coloured apply of the chained MFMA kernel (orders p >= 5): one element at a time, each
thread adding its own nodes to y with a plain load and store.  One element, 27 and 125 on one,
two and five workgroups (coloured meshes are boxes); nodes fewer and more than the
threads of a workgroup (216 to 729).  Reference: the CPU oracle, the parity tests' 1e-12; the
result is the same bits every time and for every grid, and adds to what y holds.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [5, 6, 7, 8])
@pytest.mark.parametrize("dq", [1, 2])
def test_coloured_elements(p, dq):
    import torch
    from paper_2603_09038_amd import hexpa as hx
    for n in (1, 3, 5) if p < 7 else (1, 3):
        mesh = synth.box_mesh(n, perturb=0.1, seed=p)
        for ops in (hx.PA_MASS, hx.PA_DIFFUSION, hx.PA_MASS | hx.PA_DIFFUSION):
            ref_op = oracle.Problem(mesh, p, p + dq, ops=ops)
            x = synth.rand_x((n * p + 1) ** 3, p)
            ref = ref_op.apply(x)
            xt = torch.tensor(x, device="cuda")
            op = hx.PAOperator(mesh, p, p + dq, ops=ops)
            op.set_variant(hx.PA_VARIANT_MFMA_COLORED)
            first = None
            for cap in (0, 1, 2, 5):
                op.set_grid_cap(cap)
                y = op.apply(xt)
                first = y if first is None else first
                assert torch.equal(y, first)
                err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
                assert err <= 1e-12, (p, dq, ops, n, cap, err)
            hx.pa_apply_add(op.h, xt, y)
            assert (y - 2 * first).norm() <= 1e-14 * first.norm()
            op.close()
