"""Layers of few tokens, whose long products are computed in K ranges that the row kernels add up, vs the fp64 oracle."""
import pytest
import torch

import workloads as W
from oracle import layer as L
from oracle import llama_layer as LL
from paper_2302_08005_amd import binding as B
from gpu_util import DEV, TOL, err

pytestmark = pytest.mark.gpu

# (a product has ranges from K = 2048 on while its 64x64 tiles are at most 32, from 6144 on while they are at most 64)
CASES = [
    # last range short (17 slabs of 128 in ranges of 5, 5, 5, 2) and its last slab partial; the attention block's K is below the line
    W.LayerConfig("postln-short-last-range", 1, 61, 512, 8, 2056, dropout_p=0.1, dtype=W.BF16, len_lo=20, len_hi=61, config_id=61),
    # every product in ranges, the layer's own input gradient too
    W.LayerConfig("postln-all", 2, 64, 1024, 16, 4096, dropout_p=0.1, dtype=W.BF16, config_id=62),
    W.LayerConfig("preln-fp16-d128", 2, 64, 1024, 8, 2600, causal=1, dropout_p=0.1, dtype=W.FP16, pre_ln=1, config_id=63),
    W.LayerConfig("preln-keeps-all", 3, 8, 1024, 16, 2048, causal=1, dropout_p=0.0, dtype=W.BF16, pre_ln=1, config_id=64),
    # a hidden size that is no multiple of a tile, one token per row block
    W.LayerConfig("ragged-hidden", 1, 3, 536, 8, 2048, causal=1, dropout_p=0.1, dtype=W.BF16, pre_ln=1, attn_dim=512, config_id=65),
    # the last size with 32 tiles and the first beyond it
    W.LayerConfig("32-tiles", 1, 256, 512, 8, 2048, dropout_p=0.1, dtype=W.BF16, config_id=66),
    W.LayerConfig("40-tiles", 1, 257, 512, 8, 2048, dropout_p=0.1, dtype=W.BF16, config_id=67),
    # 64 tiles: K = 6144 has ranges, 6136 has none (49 and 48 slabs of 128)
    W.LayerConfig("64-tiles", 2, 64, 2048, 32, 6144, causal=1, dropout_p=0.1, dtype=W.BF16, pre_ln=1, config_id=68),
    W.LayerConfig("64-tiles-short", 2, 64, 2048, 16, 6136, dropout_p=0.0, dtype=W.BF16, config_id=69),
    # the widest rows that have ranges (whole blocks of eight wavefronts in backward)
    W.LayerConfig("widest", 1, 60, 4096, 32, 6200, causal=1, dropout_p=0.1, dtype=W.BF16, pre_ln=1, config_id=70),
    # the same as a post-LN layer: the residual gradient is the row kernel's to add, outside of the paired launches (more than 64 M weights)
    W.LayerConfig("widest-postln", 1, 60, 4096, 32, 6200, dropout_p=0.1, dtype=W.BF16, config_id=72),
    W.LayerConfig("gated", 1, 100, 1024, 8, 2048, causal=1, dropout_p=0.1, dtype=W.BF16, pre_ln=1, ln_eps=1e-6, arch=W.LLAMA, config_id=71),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_layer_of_few_tokens(cfg):
    n = 2
    O = LL if cfg.arch == W.LLAMA else L
    params = [W.make_params(cfg, layer_id=l, perturbed=True) for l in range(n)]
    x, dy, sl = W.make_inputs(cfg)
    ref = O.layer_forward(cfg, params[0], x, sl)
    gref = O.layer_backward(cfg, params[0], ref, dy)
    layers = [B.Layer(cfg, params[l], layer_id=l) for l in range(n)]
    xd, dyd = layers[0].to_device(x), layers[0].to_device(dy)
    sld = None if sl is None else torch.from_numpy(sl).to(DEV)
    y = layers[0].forward(xd, sld)
    layers[0].scratch.fill_(0x5A)
    dx = layers[0].backward(xd, sld, dyd)
    errs = {"y": err(y, ref["y"]), "dx": err(dx, gref["dx"])}
    errs.update({"d" + k: err(layers[0].grads[k], gref[k]) for k in W.param_names(cfg)})
    bad = {k: v for k, v in errs.items() if not v <= TOL[cfg.dtype]}
    assert not bad, (bad, errs)

    # two layers as a stack and as a checkpointed one: the bits of the layers called one at a time
    y1 = layers[1].forward(y, sld)
    g1 = layers[1].backward(y, sld, dyd)
    g0 = layers[0].backward(xd, sld, g1)
    for checkpoint in (0, 1):
        st = B.Stack(cfg, params, checkpoint=checkpoint)
        assert torch.equal(st.forward(xd, sld), y1)
        assert torch.equal(st.backward(xd, sld, dyd), g0)
        for l in range(n):
            for k in W.param_names(cfg):
                assert torch.equal(st.grads[l][k], layers[l].grads[k]), (checkpoint, l, k)


# dx written over x: products and gradients in launches of their own, sums in another order than with dx elsewhere
@pytest.mark.parametrize("cfg", [c for c in CASES if c.name in ("postln-short-last-range", "postln-all", "widest-postln")], ids=lambda c: c.name)
def test_input_gradient_on_top_of_the_input(cfg):
    params = W.make_params(cfg, perturbed=True)
    x, dy, sl = W.make_inputs(cfg)
    ref = L.layer_forward(cfg, params, x, sl)
    gref = L.layer_backward(cfg, params, ref, dy)
    layer = B.Layer(cfg, params)
    xd, dyd = layer.to_device(x), layer.to_device(dy)
    sld = None if sl is None else torch.from_numpy(sl).to(DEV)
    layer.forward(xd, sld)
    B.slapo_layer_bwd(layer.desc, layer.params, xd, sld, dyd, layer.saved, xd, layer.grads, layer.scratch)
    errs = {"dx": err(xd, gref["dx"]), **{"d" + k: err(layer.grads[k], gref[k]) for k in W.param_names(cfg)}}
    bad = {k: v for k, v in errs.items() if not v <= TOL[cfg.dtype]}
    assert not bad, (bad, errs)
