"""The first application of a preconditioner runs its coarse solve kernel by kernel, later ones
as a captured graph; so does the first one after a change of the iteration count or of the
operator.  Same kernels in the same order: the results are the same bits.  (A binding anew sums
the coarse stencil by atomics: there the coarse level's 1e-9 is the bar.)
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,n", [(2, 3), (4, 4)])
def test_first_and_later_applications_agree(p, n):
    import torch
    from paper_2603_09038_amd import hexpa as hx
    mesh = synth.box_mesh(n, perturb=0.1, seed=p)
    ops = [hx.PAOperator(mesh, p, p + 2, ops=hx.PA_DIFFUSION, ess_mode=1,
                         coeff={"kind": hx.PA_COEFF_SINE, "value": v, "amp": 0.5, "freq": 2.0}) for v in (1.0, 3.0)]
    r = torch.tensor(synth.rand_x(ops[0].ndof, 1), device="cuda")
    seen = []

    def thrice(f):
        a = f().clone()
        for _ in range(2):
            assert torch.equal(f(), a)
        seen.append(a)

    lp = hx.LearnedPreconditioner(ops[0], use_net=False, use_coarse=True, coarse_iters=4)
    thrice(lambda: lp.apply(r))
    lp.configure(use_net=False, use_coarse=True, coarse_iters=7)
    thrice(lambda: lp.coarse(r))
    thrice(lambda: lp.apply(r))
    lp.bind(ops[1])
    thrice(lambda: lp.apply(r))
    lp.bind(ops[0])
    thrice(lambda: lp.apply(r))
    assert (seen[2] - seen[4]).norm() <= 1e-9 * seen[2].norm()
    assert not torch.equal(seen[0], seen[2]) and not torch.equal(seen[2], seen[3])
    lp.close()
    for op in ops:
        op.close()
