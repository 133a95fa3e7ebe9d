"""The vector-ALU apply with z in registers (orders p <= 4) where its groups can go wrong.

A workgroup takes 4 to 64 elements at a time (the pencils that fill its threads): one element,
27 and 125 give a single short group, a short last group, several groups on one, two and five
workgroups and groups that cross element rows; shuffled elements have no neighbours to merge.
Reference: the CPU oracle; the bar is the parity tests' 1e-12 (sums of at most ~10^3 products
in FP64).
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("dq", [1, 2])
def test_groups_of_elements(p, dq):
    import torch
    from paper_2603_09038_amd import hexpa as hx
    for n in (1, 3, 5):
        mesh = synth.box_mesh(n, perturb=0.1, seed=p)
        perm = np.random.default_rng([p, 9]).permutation(n ** 3)
        for ops in (hx.PA_MASS, hx.PA_DIFFUSION, hx.PA_MASS | hx.PA_DIFFUSION):
            ref_op = oracle.Problem(mesh, p, p + dq, ops=ops)
            x = synth.rand_x((n * p + 1) ** 3, p)
            ref = ref_op.apply(x)
            xt = torch.tensor(x, device="cuda")
            for shuffled in (False, True):
                if shuffled:
                    op = hx.PAOperator({"n": 0, "vert": mesh["vert"], "hex": mesh["hex"][perm]}, p, p + dq, ops=ops,
                                       structured=False, elem_dofs=ref_op.elem_dofs[perm], ndof=x.size)
                else:
                    op = hx.PAOperator(mesh, p, p + dq, ops=ops)
                op.set_variant(hx.PA_VARIANT_VALU)
                for cap in (0, 1, 2, 5):
                    op.set_grid_cap(cap)
                    y = op.apply(xt).cpu().numpy()
                    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
                    assert err <= 1e-12, (p, dq, ops, n, shuffled, cap, err)
                op.close()


def test_a_nan_stays_in_its_elements():
    """A NaN at one node reaches the outputs of the elements that hold it and no others, although
    a workgroup's LDS goes from one group to the next."""
    import torch
    from paper_2603_09038_amd import hexpa as hx
    for p, q in ((1, 2), (2, 4), (3, 4), (4, 5), (4, 6)):
        n = 5
        mesh = synth.box_mesh(n, perturb=0.1, seed=1)
        for ops in (hx.PA_MASS, hx.PA_DIFFUSION, hx.PA_MASS | hx.PA_DIFFUSION):
            op = hx.PAOperator(mesh, p, q, ops=ops)
            dofs = hx.pa_get_elem_dofs(op.h)
            x = synth.rand_x(op.ndof, 3)
            bad = dofs[62][(p + 1) ** 3 // 2]
            x[bad] = np.nan
            hit = np.unique(dofs[(dofs == bad).any(axis=1)])
            op.set_variant(hx.PA_VARIANT_VALU)
            op.set_grid_cap(3)
            y = op.apply(torch.tensor(x, device="cuda")).cpu().numpy()
            assert np.isnan(y[hit]).all()
            assert np.isfinite(np.delete(y, hit)).all(), (p, q, ops)
            op.close()
