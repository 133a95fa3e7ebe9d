"""The batched loops of PCG's vector kernels: a thread takes four entries a grid apart in one go
once n exceeds 3 x 1024 x 256, and the rest one by one.  105^3 = 1,157,625 entries run one
batched turn (4 x 262,144) and a tail that ends inside a block.

Solves stop on the recursive residual at 1e-10, or 1e-8 in mixed precision, where the residual
is the FP64 one; the recomputed residual differs from it by rounding of the iterates
(iterations x eps x condition of these well conditioned mass systems, below 1e-11), so twice
the tolerance is the bar.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

N, P = 52, 2


@pytest.fixture(scope="module")
def hx():
    import torch  # noqa: F401
    from paper_2603_09038_amd import hexpa
    return hexpa


def _residual(op, b, x, constrained):
    r = b - (op.apply_constrained(x) if constrained else op.apply(x))
    return float(r.norm() / b.norm())


@pytest.mark.parametrize("constrained", [False, True])
def test_fp64_solves(hx, constrained):
    import torch
    op = hx.PAOperator(synth.box_mesh(N, perturb=0.1, seed=1), P, P + 1, ops=hx.PA_MASS, ess_mode=int(constrained))
    assert op.ndof == 105 ** 3
    b = torch.tensor(synth.rand_x(op.ndof, 5), device="cuda")
    iters = {}
    for mode in (hx.PA_CG_PLAIN, hx.PA_CG_JACOBI):
        for check in (1, 7):
            x = torch.tensor(synth.rand_x(op.ndof, 6), device="cuda")
            res = hx.cg_solve(op.h, b, x, rtol=1e-10, max_it=2000, mode=mode, check_every=check, constrained=constrained)
            rel = _residual(op, b, x, constrained)
            assert rel <= 2e-10, (mode, check, rel)
            assert abs(res["rel_res_true"] - rel) <= 1e-12
            iters[mode, check] = res["iters"]
    # the host looks one check late, so both stop within a check of each other
    for mode in (hx.PA_CG_PLAIN, hx.PA_CG_JACOBI):
        assert abs(iters[mode, 7] - iters[mode, 1]) <= 14
    op.close()


@pytest.mark.parametrize("constrained", [False, True])
@pytest.mark.parametrize("mode", ["PA_CG_MIXED_RU", "PA_CG_MIXED_IR", "PA_CG_MIXED_FCG"])
def test_fp32_vectors(hx, mode, constrained):
    """FP32 vectors with the 16-bit apply; reliable updates end each chunk with an update of x
    beside the residual (the one caller of that form)."""
    import torch
    op = hx.PAOperator(synth.box_mesh(N, perturb=0.1, seed=1), P, P + 2, ops=hx.PA_MASS | hx.PA_DIFFUSION,
                       ess_mode=int(constrained))
    b = torch.tensor(synth.rand_x(op.ndof, 5), device="cuda")
    x = torch.zeros_like(b)
    hx.cg_solve(op.h, b, x, rtol=1e-8, max_it=4000, mode=getattr(hx, mode), constrained=constrained, inner_max=40)
    rel = _residual(op, b, x, constrained)
    assert rel <= 2e-8, rel
    op.close()
