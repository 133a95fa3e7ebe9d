"""Rounding of the weight-gradient sums of the network's middle layer.

The inputs make every summand of a weight's gradient the same number: r = 1 gives tiles of +1
and -1, layer 1 passes them on through its centre taps (the tiles of -1 are cut off by the
ReLU), layer 2 is open (bias 1, no weights), and a target proportional to the number of
elements at a node makes the gradient at the output constant.  Rounding then has one sign along a chain of
additions, so a chain of k additions is off by about k units and a long one shows, while the
exact sum is a product.

A wave adds 4 N products in FP32 to a part, and the parts of its rows and items (a tap has at
most N rows of an item, and two of its four parts hold tiles of +1) in FP32; the sums of the
waves are FP64.  With u = 2^-24 the bar is u times that number of additions, one rounding of the row of
a workgroup and one of the result.  (One chain over all products of a wave: 72 to 200 an item.)
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,n", [(2, 3), (2, 32), (3, 26), (4, 2), (4, 24)])
def test_equal_summands(p, n):
    import torch
    from paper_2603_09038_amd import hexpa as hx
    N, rng = p + 1, np.random.default_rng([p, n])
    op = hx.PAOperator(synth.box_mesh(n, perturb=0.1, seed=p), p, p + 2, ops=hx.PA_DIFFUSION)
    lp = hx.LearnedPreconditioner(op, use_net=True, use_coarse=False, loss=hx.PA_LP_LOSS_L2)
    w1, w3 = (rng.uniform(0.5, 1.0, 16).astype(np.float32) for _ in range(2))
    W1, b1, W2, b2, W3, b3 = (np.zeros(s, np.float32) for s in ((16, 2, 27), 16, (16, 16, 27), 16, (16, 27), 1))
    W1[:, 0, 13], b2[:], W3[:, 13] = w1, 1.0, w3
    lp.set_params(np.concatenate([a.ravel() for a in (W1, b1, W2, b2, W3, b3)]))
    mult = np.bincount(hx.pa_get_elem_dofs(op.h).ravel(), minlength=op.ndof)  # 1, 2, 4 or 8
    t = mult / 3.0
    _, g = lp.loss_grad(torch.ones(op.ndof, dtype=torch.float64, device="cuda"), torch.tensor(t, device="cuda"))
    gout = np.float32(-t[0] / mult[0] / (t @ t))
    ga2 = w3 * gout  # FP32
    inside = np.array([N - 1, N, N - 1], dtype=np.float64)
    count = n ** 3 * np.einsum("z,y,x->zyx", inside, inside, inside).ravel()
    want = ga2.astype(np.float64)[:, None, None] * w1.astype(np.float64)[None, :, None] * count
    got = g[W1.size + 16:][:W2.size].reshape(W2.shape)
    items = np.ceil(np.ceil(n ** 3 / 64) * N / (256 // (3 * N - 2) * N))  # output planes of a wave
    bar = 2.0 ** -24 * (4 * N + 2 * N * items + 2)
    err = np.abs(got / want - 1).max()
    print(f"p={p} n={n}: error {err:.2e}, bar {bar:.2e}")
    assert err <= bar
    lp.close()
    op.close()
