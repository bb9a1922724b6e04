"""Layers that drop nothing: a branch's gradient and the residual's are one array, dy itself in front of a pre-LN layer's
feed-forward block. Against the fp64 oracle, on one and two streams, with dx on top of dy, and as stacks."""
import pytest
import torch

import workloads as W
from gpu_util import DEV, TOL, captured, err, to_np
from paper_2302_08005_amd import binding as B
from test_gpu_layer import run_case
from test_gpu_stack import test_stack_matches_oracle_chain_and_single_layer_calls as stack_matches

pytestmark = pytest.mark.gpu


def cfg(name, batch, seq, hidden, heads, ffn, **kw):
    return W.LayerConfig(name, batch, seq, hidden, heads, ffn, **{**dict(causal=1, dropout_p=0.0, dtype=W.BF16, pre_ln=1, config_id=91), **kw})


CASES = [
    cfg("preln", 2, 67, 256, 4, 1000), cfg("preln-narrow-branches-fp16", 3, 40, 512, 1, 72, attn_dim=64, dtype=W.FP16),
    cfg("postln", 3, 67, 256, 4, 520, pre_ln=0, causal=0, len_lo=20, len_hi=67), cfg("preln-fp32", 2, 33, 320, 5, 328, dtype=W.FP32),
    cfg("preln-two-streams", 4, 523, 512, 8, 2048), cfg("postln-two-streams-forked", 5, 1000, 512, 8, 1024, pre_ln=0, causal=0),
    cfg("preln-two-streams-forked", 5, 1000, 512, 8, 1024),
    cfg("preln-shared", 4, 500, 1024, 16, 4096), cfg("postln-shared-blocks-fp16", 4, 756, 1152, 18, 3456, pre_ln=0, causal=0, dtype=W.FP16),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_layers_without_dropout(c):
    errs, layer, (xd, sld, dyd, _, dx) = run_case(c, check_saved=False)
    bad = {k: v for k, v in errs.items() if not v <= TOL[c.dtype]}
    assert not bad, (bad, errs)
    want, dy = {k: v.clone() for k, v in layer.grads.items()}, dyd.clone()
    B.slapo_layer_bwd(layer.desc, layer.params, xd, sld, dy, layer.saved, dy, layer.grads, layer.scratch)   # dx on top of dy
    torch.cuda.synchronize()
    assert torch.equal(dy, dx)
    for k in W.PARAM_NAMES:
        assert err(layer.grads[k], to_np(want[k])) <= TOL[c.dtype], k


@pytest.mark.parametrize("c", [
    cfg("stack-preln", 2, 72, 256, 4, 520, config_id=92), cfg("stack-preln-forked", 5, 1000, 256, 4, 512, config_id=93),
    cfg("stack-postln", 2, 72, 256, 4, 520, pre_ln=0, causal=0, config_id=94),
    cfg("stack-llama", 2, 72, 256, 4, 344, ln_eps=1e-6, arch=W.LLAMA, config_id=95)], ids=lambda c: c.name)
def test_stacks_without_dropout(c):
    stack_matches(c)


@pytest.mark.parametrize("c", [cfg("one-stream", 2, 67, 256, 4, 1000), cfg("forked", 5, 1000, 512, 8, 1024),
                               cfg("shared", 4, 500, 1024, 16, 4096)], ids=lambda c: c.name)
def test_input_gradient_partly_on_top_of_dy(c):
    """dx from 40 rows into dy on: as with dx on dy, no launch beside the one that writes dx reads dy."""
    layer, T = B.Layer(c, W.make_params(c)), c.batch * c.seq
    gen = torch.Generator(device=DEV).manual_seed(6)
    x, both = (torch.randn(rows, c.hidden, device=DEV, generator=gen).to(layer.dt) for rows in (T, T + 40))
    dy, dx = both[:T], both[40:]
    layer.forward(x)
    whole = dy.clone()
    step = lambda g, out: B.slapo_layer_bwd(layer.desc, layer.params, x, None, g, layer.saved, out, layer.grads, layer.scratch)
    step(whole, whole)                                   # dx on dy
    want, grads = whole.clone(), {k: v.clone() for k, v in layer.grads.items()}
    assert captured(lambda: step(dy, dx)) == captured(lambda: step(whole, whole))
    step(dy, dx)
    torch.cuda.synchronize()
    assert torch.equal(dx, want)
    for k in W.PARAM_NAMES:
        assert torch.equal(layer.grads[k], grads[k]), k
