"""Rows and columns of unequal size on the split GEMMs: every row and column of
dW is right to its own size, as fp32 products give it, whatever lies beside it
in the same 32 rows.  The oracle's product is the reference, in float64."""
import math

import numpy as np
import pytest
import torch

import oracle as O
from paper_2306_01685_amd import Params, harness as H
from tests.parity import oparams

# The bar of the whole-matrix tests (4e-6 without, 2e-5 after updates), here
# for each row and each column by its own norm: an fp32 product of K <= 600
# terms rounds to about sqrt(K) 2^-24 = 1.5e-6 of it.
TOL, TOL_STEP = 4e-6, 2e-5
EXPS = np.array([0, -10, -20, -26, -30, -42])


def sizes(rng, d, mixed):
    """1, or powers of two from 2^0 to 2^-42 mixed within any 32."""
    return 2.0 ** rng.choice(EXPS, d) if mixed else np.ones(d)


def coupled(rng, d, s):
    """Near the identity, i and j coupled by s_i s_j, as a rank-1 update by
    means of size s leaves them; bitwise symmetric fp32."""
    q = (rng.standard_normal(d) * s).astype(np.float32)
    P = (np.float32(0.1) * np.outer(q, q)).astype(np.float32)
    P[np.arange(d), np.arange(d)] = (1.0 + 0.1 * rng.random(d)).astype(np.float32)
    return P


def worst(got, ref, axis):
    n = np.linalg.norm(ref, axis=axis)
    e = np.linalg.norm(np.asarray(got, np.float64) - ref, axis=axis)
    assert np.all(e[n == 0] == 0)
    return float((e[n > 0] / n[n > 0]).max())


def check(got, ref, tol, *ctx):
    r, c = worst(got, ref, 1), worst(got, ref, 0)
    assert r <= tol, (*ctx, "row", r)
    assert c <= tol, (*ctx, "column", c)


SHAPES = [(64, 128), (320, 192), (192, 320), (257, 100), (99, 514)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("factors", ["identity", "coupled"])
@pytest.mark.parametrize("grad_dtype", ["fp32", "bf16"])
def test_rows_and_columns_of_unequal_size(grad_dtype, factors, rows, cols):
    rng = np.random.default_rng(5)
    layers = H.allocate_layers(SHAPES, grad_dtype)
    st, ins = [], []
    for L, s in zip(layers, SHAPES):
        sr, sc = sizes(rng, s[0], rows), sizes(rng, s[1], cols)
        if factors == "identity":
            Li, Ri = np.eye(s[0], dtype=np.float32), np.eye(s[1], dtype=np.float32)
        else:
            Li, Ri = coupled(rng, s[0], sr), coupled(rng, s[1], sc)
        a = (rng.standard_normal(s[0]) * sr * 0.2).astype(np.float32)
        g = (rng.standard_normal(s[1]) * sc * 0.2).astype(np.float32)
        G = (rng.standard_normal(s) * 1e-3 * sr[:, None] * sc[None, :]).astype(np.float32)
        if grad_dtype == "bf16":
            G = torch.from_numpy(G).bfloat16().float().numpy()
        H.set_factors(L, Li, Ri)
        H.set_inputs(L, a, g, G)
        st.append([Li.astype(np.float64), Ri.astype(np.float64)])
        ins.append((a, g, G))
    plan = H.make_plan(layers)
    p = Params(eps=math.inf, rescale=False)
    plan.precondition(p)   # no pending term
    torch.cuda.synchronize()
    for L, (Li, Ri), (_, _, G) in zip(layers, st, ins):
        check(H.get_dW(L), O.precondition(Li, G.astype(np.float64), Ri), TOL, G.shape)
    # one term, two (a factor written every other step), the stabiliser's
    # shift of the diagonal
    for t, eps in enumerate((math.inf, math.inf, 0.0, math.inf)):
        p = Params(eps=eps, rescale=False)
        plan.step(p)
        torch.cuda.synchronize()
        for i, (L, (a, g, G)) in enumerate(zip(layers, ins)):
            st[i][0], st[i][1], dW, _ = O.layer_step(st[i][0], st[i][1], a, g, G, oparams(p))
            check(H.get_dW(L), dW, TOL_STEP, SHAPES[i], t)
