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


@pytest.mark.parametrize("used_before", [False, True])
def test_application_in_a_captured_graph(used_before):
    """An application that the caller captures is part of the graph, whether the handle has its
    own graph already or not: replays on new residuals, with eager work between them."""
    import torch
    from paper_2603_09038_amd import hexpa as hx
    op = hx.PAOperator(synth.box_mesh(4, perturb=0.1, seed=1), 2, 4, ops=hx.PA_DIFFUSION, ess_mode=1)
    lp = hx.LearnedPreconditioner(op, use_net=False, use_coarse=True)
    want = hx.LearnedPreconditioner(op, use_net=False, use_coarse=True)
    r, z = (torch.zeros(op.ndof, dtype=torch.float64, device="cuda") for _ in range(2))
    if used_before:
        lp.apply(r, z)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        lp.apply(r, z)
    for seed in range(4):
        r.copy_(torch.tensor(synth.rand_x(op.ndof, seed)))
        z.fill_(np.nan)
        g.replay()
        ref = want.apply(r)
        torch.cuda.synchronize()
        # two handles: their stencils are summed by atomics
        assert (z - ref).norm() <= 1e-9 * ref.norm()
    for h in (lp, want, op):
        h.close()
