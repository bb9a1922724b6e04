"""Backward launches that hold a data gradient, a weight gradient and the sums behind the row kernels and the biases, vs
the fp64 oracle: every pair of tile sizes, edges of tiles, partial K slabs, one and two streams, accumulation."""
import pytest
import torch

import workloads as W
from gpu_util import DEV, TOL, captured, err, to_np
from paper_2302_08005_amd import binding as B
from test_gpu_layer import run_case

pytestmark = pytest.mark.gpu


def cfg(name, batch, seq, hidden, heads, ffn, dtype=W.BF16, **kw):
    return W.LayerConfig(name, batch, seq, hidden, heads, ffn, **{**dict(causal=0, dropout_p=0.1, dtype=dtype, config_id=81), **kw})


# names: tiles of the data / the weight gradient of the feed-forward block's products
CASES = [
    cfg("64x64-64x64-half-ragged", 3, 67, 256, 4, 1000, W.FP16, len_lo=20, len_hi=67),
    cfg("64x64-64x64-one-token", 1, 1, 128, 2, 72),
    cfg("64x64-128x64", 1, 130, 1024, 8, 3848, len_lo=100, len_hi=130),
    cfg("64x64-128x128-preln", 2, 35, 1536, 12, 6144, pre_ln=1, causal=1),
    cfg("128x64-128x64-two-streams", 4, 523, 512, 8, 2048),
    cfg("128x64-128x128-two-streams", 1, 264, 1536, 24, 6152),
    cfg("fp32-16x16-preln", 2, 33, 64, 1, 72, W.FP32, pre_ln=1, causal=1),
    cfg("fp32-32x32", 3, 45, 320, 5, 328, W.FP32, len_lo=9, len_hi=45),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_paired_gradients(c):
    errs, layer, (xd, sld, dyd, _, dx) = run_case(c, check_saved=False)
    bad = {k: v for k, v in errs.items() if not v <= TOL[c.dtype]}
    assert not bad, (bad, errs)
    first, dx = {k: v.clone() for k, v in layer.grads.items()}, dx.clone()
    layer.desc.accumulate_grads = 1
    dx2 = layer.backward(xd, sld, dyd)
    assert torch.equal(dx, dx2)
    for k in W.PARAM_NAMES:
        # g + (g + rounding): one rounding of the storage type more than twice the first result
        assert err(layer.grads[k], 2 * to_np(first[k])) <= TOL[c.dtype] / 2, k


def test_input_gradient_on_top_of_the_input():
    """dx may lie on x, which the weight gradient of the QKV projection still reads: the two then do not share a launch."""
    c = CASES[2]
    errs, layer, (xd, sld, dyd, _, dx) = run_case(c, check_saved=False)
    want = {k: v.clone() for k, v in layer.grads.items()}
    x2 = xd.clone()
    B.slapo_layer_bwd(layer.desc, layer.params, x2, sld, dyd, layer.saved, x2, layer.grads, layer.scratch)
    torch.cuda.synchronize()
    assert err(x2, to_np(dx)) <= TOL[c.dtype]
    for k in W.PARAM_NAMES:
        assert err(layer.grads[k], to_np(want[k])) <= TOL[c.dtype], k


@pytest.mark.parametrize("c", [
    cfg("paired-two-streams", 4, 523, 512, 8, 2048), cfg("paired-two-streams-no-dropout", 4, 523, 512, 8, 2048, dropout_p=0.0),
    cfg("forked", 5, 1000, 512, 8, 1024), cfg("forked-half-checkpoint", 5, 1000, 512, 8, 1024, W.FP16)], ids=lambda c: c.name)
def test_input_gradient_on_top_of_the_input_on_two_streams(c):
    """The weight gradient of the QKV projection, on the helper stream, has read x before dx is written there."""
    layer = B.Layer(c, W.make_params(c), checkpoint=int("checkpoint" in c.name))
    gen = torch.Generator(device=DEV).manual_seed(5)
    x, dy = (torch.randn(c.batch, c.seq, c.hidden, device=DEV, generator=gen).to(layer.dt) for _ in range(2))
    layer.forward(x)
    dx = layer.backward(x, None, dy)
    want = {k: v.clone() for k, v in layer.grads.items()}
    if "forked" in c.name:   # captured, the same launches have one dependence more
        step = lambda out: B.slapo_layer_bwd(layer.desc, layer.params, x, None, dy, layer.saved, out, layer.grads, layer.scratch)
        (nodes, edges), (nodes2, edges2) = captured(lambda: step(dx)), captured(lambda: step(x))
        assert nodes2 == nodes and edges2 == edges + 1
    for _ in range(3):
        x2 = x.clone()
        B.slapo_layer_bwd(layer.desc, layer.params, x2, None, dy, layer.saved, x2, layer.grads, layer.scratch)
        torch.cuda.synchronize()
        if "forked" in c.name:   # the same launches, ordered
            assert torch.equal(x2, dx) and all(torch.equal(layer.grads[k], want[k]) for k in W.PARAM_NAMES)
        assert err(x2, to_np(dx)) <= TOL[c.dtype]
        for k in W.PARAM_NAMES:
            assert err(layer.grads[k], to_np(want[k])) <= TOL[c.dtype], k


# few tokens, many weights: beyond 64 million the gradients have a launch each (fp32: never)
@pytest.mark.parametrize("hidden,tokens,dtype,paired", [(2048, 128, W.BF16, True), (2304, 16, W.FP16, True), (2560, 16, W.BF16, False),
                                                        (2560, 16, W.FP32, True)])
def test_which_calls_pair_their_gradients(hidden, tokens, dtype, paired):
    c = cfg("few-tokens", 1, tokens, hidden, hidden // 128, 4 * hidden, dtype, pre_ln=1, causal=1)
    errs, layer, (x, _, dy, _, dx) = run_case(c, check_saved=False)
    assert all(v <= TOL[dtype] for v in errs.values()), errs
    launches = captured(lambda: B.slapo_layer_bwd(layer.desc, layer.params, x, None, dy, layer.saved, dx, layer.grads, layer.scratch), grids=True)
    # three row kernels, four products with the gradients beside them, the last sums, attention (one to three), the gradient
    # of the output projection if it is forked; else eight products (and the second kernels of K ranges) and six sums
    assert len(launches) <= 12 if paired else len(launches) >= 17
