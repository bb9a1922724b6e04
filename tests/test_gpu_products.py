"""Backward whose weight gradients share launches of 256x256 tiles with each other and with data gradients: vs the fp64 oracle, and
vs the same layer with a launch for each (dx on top of x). Ragged tokens, widths and K."""
import pytest
import torch

import test_gpu_layer
import workloads as W
from gpu_util import DEV, TOL, captured, err, shared_launches, to_np
from paper_2302_08005_amd import binding as B
from test_gpu_layer import run_case
from test_gpu_llama import run_case as run_gated

pytestmark = pytest.mark.gpu


def cfg(name, batch, seq, hidden, heads, ffn, dtype=W.BF16, **kw):
    return W.LayerConfig(name, batch, seq, hidden, heads, ffn, **{**dict(causal=0, dropout_p=0.1, dtype=dtype, config_id=96), **kw})


def tiles(*products):
    return sum(((m + 255) // 256) * ((n + 255) // 256) for m, n in products)


def with_quarters(whole, cut):
    """The grid of a launch of `whole` tiles, `cut` of them in quarters."""
    return whole - cut + (cut + 7) // 8 * 32, 1, 1


def launches(layer, x, dy, dx):
    return captured(lambda: B.slapo_layer_bwd(layer.desc, layer.params, x, None, dy, layer.saved, dx, layer.grads, layer.scratch), grids=True)


# the input gradient and all weight gradients behind attention; `cut`: tiles in quarters, of weight gradients, or of the input gradient
# where that is the shortest (its K, 960, is no multiple of a quarter's slabs)
@pytest.mark.parametrize("c,cut", [
    (cfg("postln-ragged", 4, 525, 1024, 16, 4104, len_lo=100, len_hi=525), 0),
    (cfg("gated-half-ragged", 4, 775, 1024, 8, 2728, W.FP16, causal=1, pre_ln=1, dropout_p=0.0, ln_eps=1e-6, arch=W.LLAMA), 0),
    (cfg("weights-in-quarters-half", 4, 500, 1536, 24, 6152, W.FP16), 28),
    (cfg("input-in-quarters", 4, 650, 1536, 5, 4104, attn_dim=320, causal=1, pre_ln=1), 18)], ids=lambda v: getattr(v, "name", v))
def test_gradients_behind_attention(c, cut):
    errs, layer, (x, sl, dy, _, dx) = (run_gated if c.arch == W.LLAMA else run_case)(c, check_saved=False)
    assert all(v <= TOL[c.dtype] for v in errs.values()), errs
    T, H, F, F1, A = c.batch * c.seq, c.hidden, c.ffn, c.ffn * (2 if c.arch == W.LLAMA else 1), c.attn_dim or c.hidden
    assert launches(layer, x, dy, dx).count(with_quarters(tiles((T, H), (H, F), (F1, H), (H, A), (3 * A, H)), cut)) == 1
    first, dx = {k: v.clone() for k, v in layer.grads.items()}, dx.clone()
    layer.desc.accumulate_grads = 1
    assert torch.equal(layer.backward(x, sl, dy), dx)
    for k in W.param_names(c):   # one rounding of the storage type more than twice the first result
        assert err(layer.grads[k], 2 * to_np(first[k])) <= TOL[c.dtype] / 2, k


# each block's with the gradient of its input
@pytest.mark.parametrize("dtype", [W.BF16, W.FP16])
def test_gradients_of_each_block(dtype):
    c = cfg("blocks", 4, 750, 1536, 16, 4104, dtype, attn_dim=1024)
    layer, T, H, F, A = B.Layer(c, W.make_params(c)), 3000, 1536, 4104, 1024
    gen = torch.Generator(device=DEV).manual_seed(9)
    x, dy = (torch.randn(c.batch, c.seq, H, device=DEV, generator=gen).to(layer.dt) for _ in range(2))
    layer.forward(x)
    dx = layer.backward(x, None, dy)
    want = {k: v.clone() for k, v in layer.grads.items()}
    grids = launches(layer, x, dy, dx)
    assert with_quarters(tiles((T, H), (H, F), (F, H)), 20) in grids and with_quarters(tiles((T, H), (H, A), (3 * A, H)), 0) in grids
    x2 = x.clone()   # dx on top of x: a launch for each
    assert len(launches(layer, x2, dy, x2)) > len(grids)
    B.slapo_layer_bwd(layer.desc, layer.params, x2, None, dy, layer.saved, x2, layer.grads, layer.scratch)
    torch.cuda.synchronize()
    assert err(x2, to_np(dx)) <= TOL[c.dtype]   # (the same sums in another order, rounded once more on the way)
    for k in W.PARAM_NAMES:
        assert err(layer.grads[k], to_np(want[k])) <= TOL[c.dtype], k
        layer.grads[k].copy_(want[k])
    layer.desc.accumulate_grads = 1
    assert torch.equal(layer.backward(x, None, dy), dx)
    for k in W.PARAM_NAMES:   # one rounding of the storage type more than twice the first result
        assert err(layer.grads[k], 2 * to_np(want[k])) <= TOL[c.dtype] / 2, k


# the first feed-forward bias's gradient: column sums that the product of the activation gradient leaves behind, by its tiles
@pytest.mark.parametrize("hidden,heads,ffn,dtype,attn_dim,tile", [
    (768, 1, 776, W.BF16, 64, "<1, 128, 128, 64, 2, 4, 1, 4,"), (768, 1, 1032, W.FP16, 64, "<1, 192, 128,"),
    (768, 1, 1544, W.BF16, 64, "<1, 256, 128,"), (768, 1, 2056, W.BF16, 64, "<1, 192, 256,"),
    (768, 1, 3080, W.FP16, 64, "<1, 256, 256,"), (1024, 16, 4104, W.BF16, 0, "quarters_kernel<1,")])
def test_column_sums_of_the_activation_gradient(hidden, heads, ffn, dtype, attn_dim, tile):
    c = cfg("sums", 3, 1391, hidden, heads, ffn, dtype, attn_dim=attn_dim)
    T = c.batch * c.seq
    assert tile in B.slapo_gemm_kernel_name(dtype, B.NN, B.EPI_DACT, T, ffn, hidden, flags=0 if "quarters" in tile else B.GEMM_SHARED)
    errs, layer, (x, sl, dy, _, dx) = run_case(c, check_saved=False)
    assert all(v <= TOL[dtype] for v in errs.values()), errs
    grids = launches(layer, x, dy, dx)
    assert ((ffn + 255) // 256, 64, 1) not in grids                                       # no pass over that array ...
    assert ((3 * (attn_dim or hidden) + 255) // 256, 64, 1) in grids                      # ... as there is over the gradient of QKV


# in IEEE half a gradient that overflows its storage is an infinity in the bias gradient too, whatever its column adds up to: gradients
# in launches of their own, in shared ones, and beside data gradients (where the sums are a pass over the stored array)
@pytest.mark.parametrize("batch,seq,hidden", [(16, 500, 512), (4, 500, 1024), (2, 200, 512)])
def test_overflow_of_the_activation_gradient_shows_in_the_bias_gradient(batch, seq, hidden):
    c = cfg("overflow", batch, seq, hidden, hidden // 64, 4 * hidden, W.FP16, pre_ln=1, causal=1, act=W.RELU, dropout_p=0.0)
    params = W.make_params(c)
    params["w2"][:, :2], params["b1"][:2] = (8.0, -8.0), 100.0   # (two gates that are always open)
    layer = B.Layer(c, params)
    x, dy = torch.randn(batch, seq, hidden, device=DEV).to(layer.dt), torch.zeros(batch, seq, hidden, dtype=layer.dt, device=DEV)
    dy[0, 0], dy[0, 1] = 9216.0 / hidden, -4608.0 / hidden   # times 8 and summed: 73728, beyond the largest half, and half of that
    layer.forward(x)
    layer.backward(x, None, dy)
    b1 = layer.grads["b1"].float()
    assert b1[:2].tolist() == [float("inf"), -float("inf")] and bool(torch.isfinite(b1[2:]).all())


# which layers share launches: small ones and those that leave most of the chip idle do not
@pytest.mark.parametrize("batch,seq,hidden,together", [(12, 24, 256, False), (6, 200, 768, False), (6, 381, 768, True), (3, 500, 1024, False), (4, 500, 1024, True),
                                                       (16, 500, 512, False)])
def test_which_layers_share_launches(batch, seq, hidden, together):
    c, T, H, F = cfg("lines", batch, seq, hidden, hidden // 64, 4 * hidden), batch * seq, hidden, 4 * hidden
    layer = B.Layer(c, W.make_params(c))
    x = torch.zeros(batch, seq, hidden, dtype=layer.dt, device=DEV)
    layer.forward(x)
    dx = torch.empty_like(x)
    assert shared_launches(lambda: B.slapo_layer_bwd(layer.desc, layer.params, x, None, x, layer.saved, dx, layer.grads, layer.scratch)) == together
    assert (with_quarters(tiles((T, H), (H, F), (F, H), (H, H), (3 * H, H)), 0) in launches(layer, x, x, dx)) == together


# checkpointing, and two host threads with a helper stream between them, at sizes that share launches behind attention and by block
SHARING = [cfg("threads-behind", 4, 500, 1024, 16, 4096, causal=1, pre_ln=1), cfg("threads-blocks", 4, 756, 1152, 18, 3456)]


@pytest.mark.parametrize("c,n", list(zip(SHARING, (1, 2))), ids=lambda v: getattr(v, "name", v))
def test_shared_launches_accumulate_and_recompute(c, n, monkeypatch):
    layer = B.Layer(c, W.make_params(c))
    x = torch.zeros(c.batch, c.seq, c.hidden, dtype=layer.dt, device=DEV)
    layer.forward(x)
    dx = torch.empty_like(x)
    assert shared_launches(lambda: B.slapo_layer_bwd(layer.desc, layer.params, x, None, x, layer.saved, dx, layer.grads, layer.scratch)) == n
    monkeypatch.setattr(test_gpu_layer, "SMALL", [c] * 5)
    test_gpu_layer.test_layer_is_deterministic_and_accumulates()
    test_gpu_layer.test_checkpoint_mode_recomputes_to_the_same_bits(0)


def test_two_host_threads_with_shared_launches(monkeypatch):
    monkeypatch.setattr(test_gpu_layer, "SMALL", [None] * 4 + SHARING)
    test_gpu_layer.test_backward_from_two_host_threads_on_one_device()
