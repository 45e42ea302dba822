"""The scaled fp16 pairs that carry the fp32 operands of the split GEMMs:
their error bounds on the CPU, and on the GPU the row maxima behind the scales
wherever they come from (the SM pass, its lazy and rank-r forms, the operand
preparation of a call without an update, the first GEMM's output), ragged
sizes on both tile sizes, and the one kernel of small layers.
"""
import math

import numpy as np
import pytest
import torch

import oracle as O
from oracle.rank import layer_step_rank
from paper_2306_01685_amd import Params, harness as H
from tests.parity import TOL_STEP, check_close, fillers, has_tile, oparams, rel, spd


def split_exp(m):
    """The exponent that puts m into [2^14, 2^15), at most 126; 0 for 0 and inf."""
    m = np.float32(m)
    if not (m > 0 and np.isfinite(m)):
        return 0
    return min(14 + 127 - int(m.view(np.uint32) >> 23), 126)


def pair(x):
    """x (a float32 row) -> its two fp16 planes, scaled back, in float64."""
    e = split_exp(np.abs(x).max())
    xs = np.ldexp(x.astype(np.float64), e)   # exact: a power of two
    h = xs.astype(np.float16)
    l = (xs - h.astype(np.float64)).astype(np.float16)
    assert np.isfinite(h).all()
    return np.ldexp(h.astype(np.float64), -e), np.ldexp(l.astype(np.float64), -e)


@pytest.mark.parametrize("emin,emax", [(-1, 1), (-14, 0), (-40, 40), (-149, -100), (100, 127)])
def test_fp16_pair_error(emin, emax):
    """Within a row with largest entry m: |x - (h + l)| <= 2^-23 |x| + 2^-39 m
    (l keeps 11 of the remainder's at most 13 bits: half a unit of its last
    place, or half of fp16's spacing 2^-24 under the scale m <= 2^15)."""
    rng = np.random.default_rng(emax + 200)
    x = (rng.choice([-1.0, 1.0], 200_000) * np.ldexp(rng.uniform(1, 2, 200_000), rng.integers(emin, emax, 200_000)))
    x = x.astype(np.float32)
    h, l = pair(x)
    x = x.astype(np.float64)
    assert np.all(np.abs(x - (h + l)) <= 2.0 ** -23 * np.abs(x) + 2.0 ** -39 * np.abs(x).max())
    assert np.all(np.abs(l) <= 2.0 ** -11 * np.abs(x) + 2.0 ** -39 * np.abs(x).max())   # l l' is left out
    # 75 % of the mantissas of a well-scaled row are held exactly
    if emax - emin == 2:
        assert np.mean(x == h + l) > 0.7


@pytest.mark.gpu
@pytest.mark.parametrize("grad_dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", [(64, 64), (320, 64), (64, 320), (576, 320), (1088, 64), (64, 1088)])
def test_block_scales_follow_the_buffers(shape, grad_dtype):
    """Buffers refilled between calls, without and after an update: the scales
    come from what the call reads.  Blocks of very different sizes, zeros."""
    d_in, d_out = shape
    p = Params(eps=math.inf, rescale=False)
    L = H.allocate_layers([shape], grad_dtype, gemm_path="split")[0]
    plan = H.make_plan([L])
    rng = np.random.default_rng(d_in + d_out)
    a = (rng.standard_normal(d_in) / math.sqrt(d_in)).astype(np.float32)
    g = (rng.standard_normal(d_out) / math.sqrt(d_out)).astype(np.float32)
    for fs, gs in ((1.0, 1.0), (2.0 ** -40, 2.0 ** 20), (2.0 ** 30, 2.0 ** -60)):
        Li, Ri = spd(1, d_in) * np.float32(fs), spd(2, d_out) * np.float32(fs)
        Li[32:64] *= np.float32(2.0 ** 20)   # one block of rows and columns far larger
        Li[:, 32:64] *= np.float32(2.0 ** 20)
        G = (rng.standard_normal(shape) * gs).astype(np.float32)
        G[:32] *= np.float32(2.0 ** -25)
        if d_out > 64:
            G[:, 64:96] = 0.0
        if grad_dtype == "bf16":
            G = torch.from_numpy(G).bfloat16().float().numpy()
        H.set_factors(L, Li, Ri)
        H.set_inputs(L, a, g, G)
        plan.precondition(p)   # no pending term: maxima from the preparation
        torch.cuda.synchronize()
        check_close(H.get_dW(L), O.precondition(Li.astype(np.float64), G.astype(np.float64), Ri.astype(np.float64)),
                    4e-6, shape, fs)
    Li, Ri = spd(3, d_in), spd(4, d_out)
    H.set_factors(L, Li, Ri)
    st = [Li.astype(np.float64), Ri.astype(np.float64)]
    for t in range(5):   # pass with nothing pending, one term, lazily two terms
        plan.step(p)
        torch.cuda.synchronize()
        st[0], st[1], dW, _ = O.layer_step(st[0], st[1], a, g, G, oparams(p))
        check_close(H.get_dW(L), dW, TOL_STEP, shape, t)
    plan.sync_factors()
    torch.cuda.synchronize()
    H.set_factors(L, Li * np.float32(2.0 ** 50), Ri)   # allowed after a sync
    plan.precondition(p)
    torch.cuda.synchronize()
    check_close(H.get_dW(L), O.precondition(Li * 2.0 ** 50, G.astype(np.float64), Ri.astype(np.float64)), 4e-6, shape)


@pytest.mark.gpu
def test_block_scales_of_rank_r_factors_and_switched_layers():
    shapes = [(128, 192), (192, 64)]
    p = Params(eps=math.inf, rescale=False)
    layers = H.allocate_layers(shapes[:1], "fp32", rank=3) + H.allocate_layers(shapes[1:], "bf16")
    rng = np.random.default_rng(7)
    state, ins = [], []
    for i, L in enumerate(layers):
        d_in, d_out = shapes[i]
        Li, Ri = spd(20 + i, d_in) * np.float32(2.0 ** 24), spd(30 + i, d_out)
        H.set_factors(L, Li, Ri)
        state.append([Li.astype(np.float64), Ri.astype(np.float64)])
        r = 3 if i == 0 else 1
        a = (rng.standard_normal((r, d_in)) / d_in).astype(np.float32)
        g = (rng.standard_normal((r, d_out)) / d_out).astype(np.float32)
        G = torch.from_numpy(rng.standard_normal(shapes[i]).astype(np.float32)).bfloat16().float().numpy()
        ins.append((a if r > 1 else a[0], g if r > 1 else g[0], G))
        H.set_inputs(L, *ins[-1])
    plan = H.make_plan(layers)
    plan.set_second_order([1, 0])
    for t in range(3):
        if t == 2:   # the second layer's factors were never passed over so far
            plan.set_second_order([1, 1])
            plan.precondition(p)
        else:
            plan.step(p)
        torch.cuda.synchronize()
        a, g, G = ins[0]
        Ln, Rn, dW, _ = layer_step_rank(state[0][0], state[0][1], a.T, g.T, G, oparams(p), update=t < 2)
        state[0] = [Ln, Rn]
        check_close(H.get_dW(layers[0]), dW, TOL_STEP, t)
    ref = O.precondition(state[1][0], ins[1][2].astype(np.float64), state[1][1])
    assert rel(H.get_dW(layers[1]), ref) <= 2e-6


@pytest.mark.gpu
@pytest.mark.parametrize("grad_dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", [(64, 65), (65, 64), (67, 96), (129, 127), (255, 321), (769, 100), (100, 769), (514, 258)])
def test_ragged_layers_on_the_split(shape, grad_dtype):
    """AUTO layers of 64 or more that are not multiples of 64: partial slabs,
    unaligned rows, edges of the 128 x 128 tiles; precondition alone, then steps
    with the stabiliser off, on some and on every factor, then a sync."""
    d_in, d_out = shape
    L = H.allocate_layers([shape], grad_dtype)[0]
    rng = np.random.default_rng(d_in * 1000 + d_out)
    a = (rng.standard_normal(d_in) / math.sqrt(d_in)).astype(np.float32)
    g = (rng.standard_normal(d_out) / math.sqrt(d_out)).astype(np.float32)
    G = rng.standard_normal(shape).astype(np.float32) * np.float32(1e-3)
    if grad_dtype == "bf16":
        G = torch.from_numpy(G).bfloat16().float().numpy()
    Li, Ri = spd(5, d_in), spd(6, d_out)
    H.set_factors(L, Li, Ri)
    H.set_inputs(L, a, g, G)
    plan = H.make_plan([L])
    p = Params(eps=math.inf, rescale=False)
    plan.precondition(p)
    torch.cuda.synchronize()
    ref = O.precondition(Li.astype(np.float64), G.astype(np.float64), Ri.astype(np.float64))
    check_close(H.get_dW(L), ref, 4e-6, shape)
    st = [Li.astype(np.float64), Ri.astype(np.float64)]
    for t, eps in enumerate((math.inf, 0.0, 2.0, math.inf)):
        p = Params(eps=eps)
        plan.step(p)
        torch.cuda.synchronize()
        st[0], st[1], dW, ost = O.layer_step(st[0], st[1], a, g, G, oparams(p))
        check_close(H.get_dW(L), dW, TOL_STEP, shape, t)
        s = H.get_stats(L)
        assert s["norm_G"] == pytest.approx(ost.norm_G, rel=1e-6)
        assert s["norm_dW_hat"] == pytest.approx(ost.norm_dW_hat, rel=1e-5)
    plan.sync_factors()
    torch.cuda.synchronize()
    Lg, Rg = H.get_factors(L)
    check_close(Lg, st[0], TOL_STEP, shape)
    check_close(Rg, st[1], TOL_STEP, shape)


@pytest.mark.gpu
@pytest.mark.parametrize("grad_dtype", ["fp32", "bf16"])
def test_edges_of_large_tiles(grad_dtype):
    """Ragged and aligned layers among enough others that the plan keeps tiles
    of 256 x 256 (a bf16 G: 128 x 512), with and without the stabiliser's shift
    of the diagonal, one and two pending terms."""
    shapes = [(64, 65), (65, 64), (129, 127), (255, 321), (769, 100), (514, 258), (320, 576), (576, 320), (257, 513)]
    layers = H.allocate_layers(shapes, grad_dtype)
    plan = H.make_plan(layers + fillers())
    assert has_tile(plan, 4, 3, 0) and not has_tile(plan, 4, 6, 0)   # 769 rows: four large tiles, seven small
    rng = np.random.default_rng(21)
    st, ins = [], []
    for i, (L, s) in enumerate(zip(layers, shapes)):
        Li, Ri = spd(2 * i, s[0]), spd(2 * i + 1, s[1])
        G = (rng.standard_normal(s) * 1e-3).astype(np.float32)
        if grad_dtype == "bf16":
            G = torch.from_numpy(G).bfloat16().float().numpy()
        ins.append(((rng.standard_normal(s[0]) / math.sqrt(s[0])).astype(np.float32),
                    (rng.standard_normal(s[1]) / math.sqrt(s[1])).astype(np.float32), G))
        H.set_factors(L, Li, Ri)
        H.set_inputs(L, *ins[-1])
        st.append([Li.astype(np.float64), Ri.astype(np.float64)])
    plan.precondition(Params(eps=math.inf, rescale=False))
    torch.cuda.synchronize()
    for L, (Li, Ri), (_, _, G) in zip(layers, st, ins):
        check_close(H.get_dW(L), O.precondition(Li, G.astype(np.float64), Ri), 4e-6, G.shape)
    for t, eps in enumerate((math.inf, 0.0, math.inf)):
        p = Params(eps=eps)
        plan.step(p)
        torch.cuda.synchronize()
        for i, (L, (a, g, G)) in enumerate(zip(layers, ins)):
            st[i][0], st[i][1], dW, ost = O.layer_step(st[i][0], st[i][1], a, g, G, oparams(p))
            check_close(H.get_dW(L), dW, TOL_STEP, shapes[i], t)
            s = H.get_stats(L)
            assert s["norm_G"] == pytest.approx(ost.norm_G, rel=1e-6)
            assert s["norm_dW_hat"] == pytest.approx(ost.norm_dW_hat, rel=1e-5)


@pytest.mark.gpu
def test_tile_sizes_give_the_same_bits():
    """A few layers take small tiles, among many others large ones: the same
    sums in the same order (an output's and ||dW_hat||^2's)."""
    shapes = [(320, 576), (576, 320), (321, 515)]
    rng = np.random.default_rng(3)
    p = Params(eps=math.inf)

    def run(grad_dtype, others):
        layers = H.allocate_layers(shapes, grad_dtype, stats=False)
        plan = H.make_plan(layers + others)
        # (576 rows: five small tiles, and no more than four of 128 x 512 either way)
        assert has_tile(plan, 0, 4, 2) == (not others)
        for i, L in enumerate(layers):
            H.set_factors(L, *fac[i])
            H.set_inputs(L, *ins[i])
        for _ in range(3):
            plan.step(p)
        torch.cuda.synchronize()
        return [L["dW"].clone() for L in layers]

    fac = [(spd(2 * i, s[0]), spd(2 * i + 1, s[1])) for i, s in enumerate(shapes)]
    ins = [((rng.standard_normal(s[0]) / s[0]).astype(np.float32), (rng.standard_normal(s[1]) / s[1]).astype(np.float32),
            torch.from_numpy(rng.standard_normal(s).astype(np.float32)).bfloat16().float().numpy()) for s in shapes]
    many = fillers()
    for gd in ("fp32", "bf16"):
        alone, among = run(gd, []), run(gd, many)
        for x, y in zip(alone, among):
            assert torch.equal(x, y)


@pytest.mark.gpu
@pytest.mark.parametrize("grad_dtype", ["fp32", "bf16"])
def test_layers_of_at_most_64(grad_dtype):
    """Both products in one kernel: edges of its 4 x 4 outputs and eight-deep
    sums, with and without a pending term and the stabiliser's shift; fp32
    sums of eight within fp64 ones keep dW within a few roundings."""
    shapes = [(1, 1), (1, 64), (64, 1), (3, 5), (7, 8), (9, 16), (33, 31), (63, 62), (64, 64)]
    layers = H.allocate_layers(shapes, grad_dtype)
    rng = np.random.default_rng(11)
    st, ins = [], []
    for i, (L, s) in enumerate(zip(layers, shapes)):
        Li, Ri = spd(i, s[0]), spd(50 + i, s[1])
        a = (rng.standard_normal(s[0]) / s[0]).astype(np.float32)
        g = (rng.standard_normal(s[1]) / s[1]).astype(np.float32)
        G = torch.from_numpy(rng.standard_normal(s).astype(np.float32)).bfloat16().float().numpy()
        H.set_factors(L, Li, Ri)
        H.set_inputs(L, a, g, G)
        st.append([Li.astype(np.float64), Ri.astype(np.float64)])
        ins.append((a, g, G))
    plan = H.make_plan(layers)
    plan.precondition(Params(eps=math.inf, rescale=False))
    torch.cuda.synchronize()
    for L, (Li, Ri), (_, _, G) in zip(layers, st, ins):
        check_close(H.get_dW(L), O.precondition(Li, G.astype(np.float64), Ri), 1e-6, G.shape)
    for t, eps in enumerate((math.inf, 0.0, math.inf)):
        p = Params(eps=eps)
        plan.step(p)
        torch.cuda.synchronize()
        for i, (L, (a, g, G)) in enumerate(zip(layers, ins)):
            st[i][0], st[i][1], dW, ost = O.layer_step(st[i][0], st[i][1], a, g, G, oparams(p))
            check_close(H.get_dW(L), dW, 1e-5, shapes[i], t)
            assert H.get_stats(L)["norm_dW_hat"] == pytest.approx(ost.norm_dW_hat, rel=1e-5)
