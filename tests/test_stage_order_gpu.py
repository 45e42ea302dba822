"""mkor_run_stage beyond the order of a step."""
import math

import numpy as np
import pytest
import torch

from paper_2306_01685_amd import Params, harness as H
from tests.parity import spd

pytestmark = pytest.mark.gpu

MEANS, PASS, FINALIZE, PREP, XT, DW, RESCALE = range(7)
# both associations of a bf16 G, ragged rows, an fp32 G, bf16 factors, one kernel
SPECS = [((128, 192), "bf16", {}), ((320, 64), "bf16", {}), ((130, 75), "bf16", {}), ((192, 128), "fp32", {}),
         ((128, 64), "bf16", dict(factor_dtype="bf16")), ((40, 24), "bf16", {})]


def build():
    rng = np.random.default_rng(12)
    layers = []
    for k, (s, gd, kw) in enumerate(SPECS):
        L = H.allocate_layers([s], gd, **kw)[0]
        if not kw:
            H.set_factors(L, spd(2 * k, s[0]), spd(2 * k + 1, s[1]))
        H.set_inputs(L, (rng.standard_normal(s[0]) / s[0]).astype(np.float32),
                     (rng.standard_normal(s[1]) / s[1]).astype(np.float32),
                     torch.from_numpy(rng.standard_normal(s).astype(np.float32)).bfloat16().float().numpy())
        layers.append(L)
    return layers, H.make_plan(layers)


def run(plan, p, *stages):
    for s in stages:
        plan.run_stage(p, s)
    torch.cuda.synchronize()


def test_gemms_repeat_without_a_new_preparation():
    """The first GEMM's operand lies where the second one writes: it is there
    all the same."""
    layers, plan = build()
    p = Params(eps=math.inf)
    for _ in range(2):
        plan.step(p)
    torch.cuda.synchronize()
    once = [L["dW"].clone() for L in layers]
    for _ in range(2):
        run(plan, p, XT, DW, RESCALE)
        for L, x, s in zip(layers, once, SPECS):
            assert torch.equal(L["dW"], x), s


def test_preparation_between_pass_and_finalize():
    """The preparation's maxima leave the pass's sums alone."""
    p = Params(eps=0.0)
    a, pa = build()
    b, pb = build()
    for _ in range(3):
        run(pa, p, MEANS, PASS, FINALIZE, PREP, XT, DW, RESCALE)
        run(pb, p, MEANS, PASS, PREP, FINALIZE, PREP, XT, DW, RESCALE)
    pa.sync_factors()
    pb.sync_factors()
    torch.cuda.synchronize()
    for x, y, s in zip(a, b, SPECS):
        for k in ("Linv", "Rinv", "dW"):
            assert torch.equal(x[k], y[k]), (s, k)
