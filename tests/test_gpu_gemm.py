"""GPU parity of the GEMMs and their fused epilogues vs fp64 products of the same stored inputs."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import layer as L
from paper_2302_08005_amd import binding as B
from gpu_util import DEV, TOL, err, store, tdtype, to_dev, to_np

pytestmark = pytest.mark.gpu


# the activation and its derivative are the oracle's own (pinned in tests/test_oracle_layer.py), not a second copy
_act, _dact = L._act, L._act_grad


# the last three reach the direct-load kernels with ragged edge tiles: 128x128 tiles fed by loader wavefronts
# (long K, one round of tiles), 256x256 tiles, and 128x64 tiles (long K, few tiles)
SHAPES = [(256, 256, 128), (296, 264, 200), (128, 128, 64), (1024, 768, 512), (520, 136, 72), (4096, 1024, 1024),
          (1664, 1672, 2048), (3592, 3336, 256), (520, 136, 2048)]


@pytest.mark.parametrize("dtype", [W.BF16, W.FP32, W.FP16])
@pytest.mark.parametrize("layout", [B.NT, B.NN, B.TN])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_layouts(dtype, layout, M, N, K):
    rng = np.random.default_rng(M + 3 * N + 7 * K + layout)
    a = store(rng.standard_normal((M, K)), dtype)
    b = store(rng.standard_normal((K, N)) * 0.1, dtype)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    A = to_dev(a if layout != B.TN else a.T.copy(), dtype)
    Bm = to_dev(b.T.copy() if layout == B.NT else b, dtype)
    Cout = torch.empty(M, N, dtype=A.dtype, device=DEV)
    B.slapo_gemm(dtype, layout, B.EPI_NONE, 0, M, N, K, A, Bm, Cout)
    assert err(Cout, ref) <= {W.BF16: 5e-3, W.FP16: 1e-3}.get(dtype, 1e-5)


@pytest.mark.parametrize("dtype", [W.BF16, W.FP32, W.FP16])
@pytest.mark.parametrize("act", [W.GELU, W.RELU])
def test_gemm_epilogues(dtype, act):
    M, N, K = 392, 520, 256
    rng = np.random.default_rng(5)
    a = store(rng.standard_normal((M, K)), dtype)
    w = store(rng.standard_normal((N, K)) * 0.1, dtype)
    bias = store(rng.standard_normal(N), dtype)
    aux = store(rng.standard_normal((M, N)), dtype)
    acc = a.astype(np.float64) @ w.astype(np.float64).T
    A, Wt, bd, auxd = to_dev(a, dtype), to_dev(w, dtype), to_dev(bias, dtype), to_dev(aux, dtype)
    tol = TOL[dtype]
    Cout = torch.empty(M, N, dtype=A.dtype, device=DEV)
    U = torch.empty_like(Cout)
    B.slapo_gemm(dtype, B.NT, B.EPI_BIAS, act, M, N, K, A, Wt, Cout, bias=bd)
    assert err(Cout, acc + bias) <= tol
    B.slapo_gemm(dtype, B.NT, B.EPI_BIAS_ACT, act, M, N, K, A, Wt, Cout, bias=bd, aux_out=U)   # U receives act'(pre)
    if act == W.GELU:   # (the ReLU gate is a 0/1 decision at pre = 0 +- rounding: compared where it is decided)
        assert err(U, _dact(acc + bias, act)) <= tol
    else:
        clear = np.abs(acc + bias) > 1e-2
        assert np.array_equal(to_np(U)[clear], _dact(acc + bias, act)[clear])
    assert err(Cout, _act(acc + bias, act)) <= tol
    if act == W.RELU:   # the derivative store is optional: the gate can be read off the output
        C0 = torch.empty_like(Cout)
        B.slapo_gemm(dtype, B.NT, B.EPI_BIAS_ACT, act, M, N, K, A, Wt, C0, bias=bd)
        assert torch.equal(C0, Cout)
    B.slapo_gemm(dtype, B.NT, B.EPI_DACT, act, M, N, K, A, Wt, Cout, aux_in=auxd)
    # GeLU: C = acc * aux_in; ReLU: C = acc * [aux_in > 0], the same for aux_in = relu(u) and aux_in = relu'(u)
    assert err(Cout, acc * (aux > 0 if act == W.RELU else aux.astype(np.float64))) <= tol
    B.slapo_gemm(dtype, B.NT, B.EPI_ADD, act, M, N, K, A, Wt, Cout, aux_in=auxd)
    assert err(Cout, acc + aux) <= tol
    C2 = auxd.clone()                          # in-place accumulate (aux_in aliases C)
    B.slapo_gemm(dtype, B.NT, B.EPI_ADD, act, M, N, K, A, Wt, C2, aux_in=C2)
    assert err(C2, acc + aux) <= tol


# (M, N, K): tile-starved weight gradients that take the several-K-ranges path (4, 2 and 8 ranges, ragged edges),
# and two that must not (K too short to cut up, enough tiles)
@pytest.mark.parametrize("dtype", [W.BF16, W.FP16, W.FP32])
@pytest.mark.parametrize("M,N,K,split", [(1024, 1024, 16384, True), (136, 264, 8192, True), (264, 136, 24576, True),
                                         (1024, 1024, 4096, False), (2048, 1536, 1024, False)])
def test_weight_gradient_in_k_ranges(dtype, M, N, K, split):
    rng = np.random.default_rng(M + K)
    a = store(rng.standard_normal((K, M)), dtype)
    b = store(rng.standard_normal((K, N)) * 0.05, dtype)
    c0 = store(rng.standard_normal((M, N)), dtype)
    ref = a.astype(np.float64).T @ b.astype(np.float64)
    nbytes = B.slapo_weight_grad_workspace(dtype, M, N, K)
    assert (nbytes > 0) == (split and dtype != W.FP32)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device=DEV)
    A, Bt = to_dev(a, dtype), to_dev(b, dtype)
    out = torch.empty(M, N, dtype=A.dtype, device=DEV)
    B.slapo_weight_grad(dtype, 0, M, N, K, A, Bt, out, ws)
    tol = TOL[dtype]
    assert err(out, ref) <= tol
    ws.fill_(0x7F)                                   # stale workspace contents must not matter
    out2 = torch.empty_like(out)
    B.slapo_weight_grad(dtype, 0, M, N, K, A, Bt, out2, ws)
    assert torch.equal(out, out2)                    # bit for bit, whichever workgroup finishes first
    acc = to_dev(c0, dtype)
    B.slapo_weight_grad(dtype, 1, M, N, K, A, Bt, acc, ws)
    assert err(acc, ref + c0) <= tol
    plain = torch.empty_like(out)                    # the one-range kernel: same product, other summation order
    B.slapo_gemm(dtype, B.TN, B.EPI_NONE, 0, M, N, K, A, Bt, plain)
    assert err(plain, to_np(out)) <= tol


# Grids of 256x256 tiles that end in a thin round (272 and 289 tiles on 256 CUs, ragged edges in the second case):
# with a workspace the tiles beyond the full round are computed in several K ranges and added by a second kernel.
@pytest.mark.parametrize("dtype", [W.BF16, W.FP16])
@pytest.mark.parametrize("layout", [B.NT, B.NN, B.TN])
@pytest.mark.parametrize("M,N,K", [(4352, 4096, 2048), (4296, 4200, 3072)])
def test_thin_last_round_in_k_ranges(dtype, layout, M, N, K):
    nbytes = B.slapo_gemm_workspace(dtype, layout, B.EPI_NONE, M, N, K)
    assert nbytes > 0 and nbytes == B.slapo_gemm_workspace(dtype, layout, B.EPI_ADD, M, N, K)
    assert B.slapo_gemm_workspace(dtype, layout, B.EPI_BIAS, M, N, K) == 0          # plain and add epilogues only
    assert B.slapo_gemm_workspace(dtype, layout, B.EPI_NONE, 4096, 4096, K) == 0     # a full round: nothing to do
    assert "K ranges" in B.slapo_gemm_kernel_name(dtype, layout, B.EPI_NONE, M, N, K, flags=B.GEMM_SHARED, with_ws=1)
    rng = np.random.default_rng(M + N + K + layout)
    a = store(rng.standard_normal((M, K)), dtype)
    b = store(rng.standard_normal((K, N)) * 0.1, dtype)
    aux = store(rng.standard_normal((M, N)), dtype)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    A = to_dev(a if layout != B.TN else a.T.copy(), dtype)
    Bm = to_dev(b.T.copy() if layout == B.NT else b, dtype)
    auxd = to_dev(aux, dtype)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    out = torch.empty(M, N, dtype=A.dtype, device=DEV)
    B.slapo_gemm_ex(dtype, layout, B.EPI_NONE, 0, M, N, K, A, Bm, out, ws=ws, flags=B.GEMM_SHARED)
    tol = {W.BF16: 5e-3, W.FP16: 1e-3}[dtype]
    assert err(out, ref) <= tol
    ws.fill_(0x7F)                                   # stale workspace contents must not matter
    out2 = torch.empty_like(out)
    B.slapo_gemm_ex(dtype, layout, B.EPI_NONE, 0, M, N, K, A, Bm, out2, ws=ws, flags=B.GEMM_SHARED)
    assert torch.equal(out, out2)                    # bit for bit, whichever workgroup finishes first
    plain = torch.empty_like(out)                    # without a workspace: every tile in one piece
    B.slapo_gemm(dtype, layout, B.EPI_NONE, 0, M, N, K, A, Bm, plain)
    assert err(plain, to_np(out)) <= tol and not torch.equal(plain, out)   # (the tail tiles sum in another order)
    acc = auxd.clone()                               # add epilogue, in place
    B.slapo_gemm_ex(dtype, layout, B.EPI_ADD, 0, M, N, K, A, Bm, acc, aux_in=acc, ws=ws, flags=B.GEMM_SHARED)
    assert err(acc, ref + aux) <= tol
    with pytest.raises(B.SlapoError) as e:           # a workspace that is too small is refused, not half used
        B.slapo_gemm_ex(dtype, layout, B.EPI_NONE, 0, M, N, K, A, Bm, out, ws=ws[:nbytes // 2])
    assert e.value.status == -5


# The same for the smaller tiles (NT and NN only): 272 tiles of 128x128 with 16 in the tail, 304 with ragged edges and a
# partial last slab, and grids of 128x64 tiles that are all tail: 16 tiles in 8 ranges, 9 ragged ones in 8, one row.
@pytest.mark.parametrize("dtype", [W.BF16, W.FP16])
@pytest.mark.parametrize("layout", [B.NT, B.NN])
@pytest.mark.parametrize("M,N,K", [(2176, 2048, 2048), (2331, 2040, 4104), (128, 1024, 4096), (300, 136, 6152), (1, 64, 4096)])
def test_small_tiles_in_k_ranges(dtype, layout, M, N, K):
    nbytes = B.slapo_gemm_workspace(dtype, layout, B.EPI_NONE, M, N, K)
    assert nbytes > 0 and nbytes == B.slapo_gemm_workspace(dtype, layout, B.EPI_ADD, M, N, K)
    assert B.slapo_gemm_workspace(dtype, layout, B.EPI_BIAS, M, N, K) == 0
    assert "K ranges" in B.slapo_gemm_kernel_name(dtype, layout, B.EPI_NONE, M, N, K, with_ws=1)
    rng = np.random.default_rng(M + N + K + layout)
    a = store(rng.standard_normal((M, K)), dtype)
    b = store(rng.standard_normal((K, N)) * 0.1, dtype)
    aux = store(rng.standard_normal((M, N)), dtype)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    A, Bm, auxd = to_dev(a, dtype), to_dev(b.T.copy() if layout == B.NT else b, dtype), to_dev(aux, dtype)
    ws = torch.full((nbytes,), 0x7F, dtype=torch.uint8, device=DEV)
    out = torch.empty(M, N, dtype=A.dtype, device=DEV)
    B.slapo_gemm_ex(dtype, layout, B.EPI_NONE, 0, M, N, K, A, Bm, out, ws=ws)
    tol = {W.BF16: 5e-3, W.FP16: 1e-3}[dtype]
    assert err(out, ref) <= tol
    out2 = torch.empty_like(out)
    B.slapo_gemm_ex(dtype, layout, B.EPI_NONE, 0, M, N, K, A, Bm, out2, ws=ws)
    assert torch.equal(out, out2)
    acc = auxd.clone()
    B.slapo_gemm_ex(dtype, layout, B.EPI_ADD, 0, M, N, K, A, Bm, acc, aux_in=acc, ws=ws)
    assert err(acc, ref + aux) <= tol
    small = torch.empty_like(out)                    # a workspace that does not hold the partial tiles is left alone
    B.slapo_gemm_ex(dtype, layout, B.EPI_NONE, 0, M, N, K, A, Bm, small, ws=ws[:16])
    plain = torch.empty_like(out)
    B.slapo_gemm(dtype, layout, B.EPI_NONE, 0, M, N, K, A, Bm, plain)
    assert torch.equal(small, plain) and err(plain, ref) <= tol


# K that is no multiple of the 64-deep slab: fewer than one slab, one element piece over, one under, odd (token counts of
# weight gradients), against 256x256 tiles, 128x128 tiles and 128x64 tiles (all with ragged edges). The K-range forms are
# above, split slabs and short K in layout TN below (test_gemm_partial_last_slab_tn).
@pytest.mark.parametrize("layout,Ks", [(B.NT, (8, 72, 200, 1016)), (B.NN, (8, 72, 200, 1016)), (B.TN, (1, 63, 65, 203, 1013))])
@pytest.mark.parametrize("M,N", [(3592, 3336), (1664, 2056), (520, 136)])
def test_gemm_partial_last_slab(layout, Ks, M, N):
    for K in Ks:
        rng = np.random.default_rng(K + M)
        a = store(rng.standard_normal((M, K)), W.BF16)
        b = store(rng.standard_normal((K, N)) * 0.1, W.BF16)
        ref = a @ b                                   # fp32 on the host: far below one bf16 rounding
        a[5] = np.nan                                 # the pieces beyond K are zeros, not the next row: only row 5 may show it
        A = to_dev(a if layout != B.TN else a.T.copy(), W.BF16)
        Bm = to_dev(b.T.copy() if layout == B.NT else b, W.BF16)
        Cout = torch.empty(M, N, dtype=A.dtype, device=DEV)
        B.slapo_gemm(W.BF16, layout, B.EPI_NONE, 0, M, N, K, A, Bm, Cout)
        got = to_np(Cout)
        assert np.isnan(got[5]).all()
        got[5] = ref[5]
        assert err(got, ref) <= 5e-3, K


@pytest.mark.parametrize("M,N,K", [(136, 264, 8191), (4352, 4096, 1999), (1024, 1024, 12289)])
def test_weight_gradient_in_k_ranges_of_odd_length(M, N, K):
    rng = np.random.default_rng(K)
    a = store(rng.standard_normal((K, M)), W.BF16)
    b = store(rng.standard_normal((K, N)) * 0.05, W.BF16)
    ws = torch.empty(max(B.slapo_weight_grad_workspace(W.BF16, M, N, K), 16), dtype=torch.uint8, device=DEV)
    out = torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
    B.slapo_weight_grad(W.BF16, 0, M, N, K, to_dev(a, W.BF16), to_dev(b, W.BF16), out, ws)
    assert err(out, a.T @ b) <= 5e-3


# fp32: tiles of 32 x 32 with K in 16-deep chunks over eight wavefronts: fewer rows than a tile, one over, one piece of
# columns over; K below one chunk, below eight, between, and odd where K runs along the rows of both operands.
@pytest.mark.parametrize("layout,Ks", [(B.NT, (8, 24, 136, 264, 1000)), (B.NN, (8, 24, 136, 264, 1000)), (B.TN, (1, 17, 127, 129, 999))])
@pytest.mark.parametrize("M,N", [(1, 8), (33, 40), (77, 264), (256, 1024)])
def test_gemm_fp32_tiles(layout, Ks, M, N):
    if layout == B.TN:
        M = -(-M // 8) * 8
    for K in Ks:
        rng = np.random.default_rng(K + M)
        a = rng.standard_normal((M, K)).astype(np.float32)
        b = rng.standard_normal((K, N)).astype(np.float32)
        ref, mag = a.astype(np.float64) @ b, np.abs(a).astype(np.float64) @ np.abs(b)
        if M > 5:
            a[5] = np.nan                             # only row 5 may show it
        A = to_dev(a if layout != B.TN else a.T.copy(), W.FP32)
        Bm = to_dev(b.T.copy() if layout == B.NT else b, W.FP32)
        Cout = torch.empty(M, N, dtype=torch.float32, device=DEV)
        B.slapo_gemm(W.FP32, layout, B.EPI_NONE, 0, M, N, K, A, Bm, Cout)
        got = to_np(Cout).astype(np.float64)
        if M > 5:
            assert np.isnan(got[5]).all()
            got[5] = ref[5]
        assert (np.abs(got - ref) <= (K + 8) * 2.0 ** -24 * mag + 1e-30).all(), K   # K rounded additions and the 8 partial sums


# Operands whose contraction index is strided, with rows so long that the byte offset of a slab's row beyond K leaves 32
# bits (less than one slab of K), or comes close to it in front of the slab's own offset (one row over a slab). The rows
# beyond K are zeros in the other operand: only an element that does not belong there, here a NaN, shows them.
@pytest.mark.parametrize("layout,long,K", [(B.TN, 40_000_000, 8), (B.NN, 40_000_000, 8), (B.TN, 33_000_000, 65), (B.NN, 29_000_000, 72)])
def test_gemm_rows_of_more_than_2_gib(layout, long, K):
    M, N = (long, 8) if layout == B.TN else (8, long)
    wide = torch.ones(K, long, dtype=torch.bfloat16, device=DEV)
    cols = torch.tensor([5, 13_000_000, 20_000_008, 25_032_704, long - 1], device=DEV)
    wide[:, cols] = float("nan")
    other = torch.arange(8 * K, device=DEV).remainder(5).to(torch.bfloat16)   # small whole numbers: exact sums
    other = other.view(K, 8) if layout == B.TN else other.view(8, K)
    out = torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
    B.slapo_gemm(W.BF16, layout, B.EPI_NONE, 0, M, N, K, *((wide, other) if layout == B.TN else (other, wide)), out)
    want = other.float().sum(0 if layout == B.TN else 1)
    got = out if layout == B.TN else out.t()                                  # [long, 8]
    assert torch.equal(torch.isnan(got).any(1).nonzero().flatten(), cols)
    clean = torch.ones(long, dtype=torch.bool, device=DEV)
    clean[cols] = False
    assert bool((got[clean] == want.to(torch.bfloat16)).all())


# K no multiple of 128 under a grid of 256x256 tiles with a thin last round: the K ranges are an offer there, and a
# workspace that does not hold them is left alone. (K multiples of 128 refuse one: test_thin_last_round_in_k_ranges.)
@pytest.mark.parametrize("layout", [B.NT, B.NN, B.TN])
def test_small_workspace_is_left_alone_where_k_ranges_are_an_offer(layout):
    M, N, K = 4296, 4200, 3000
    assert B.slapo_gemm_workspace(W.BF16, layout, B.EPI_NONE, M, N, K) > 16
    gen = torch.Generator(device=DEV).manual_seed(1)
    A = torch.randn((K, M) if layout == B.TN else (M, K), device=DEV, generator=gen).to(torch.bfloat16)
    Bm = torch.randn((N, K) if layout == B.NT else (K, N), device=DEV, generator=gen).to(torch.bfloat16)
    small, plain = (torch.empty(M, N, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    B.slapo_gemm_ex(W.BF16, layout, B.EPI_NONE, 0, M, N, K, A, Bm, small, ws=torch.empty(16, dtype=torch.uint8, device=DEV), flags=B.GEMM_SHARED)
    B.slapo_gemm_ex(W.BF16, layout, B.EPI_NONE, 0, M, N, K, A, Bm, plain, flags=B.GEMM_SHARED)
    assert torch.equal(small, plain)


# Shapes that can use a workspace but whose K used to keep them off it run without one: thin last rounds of 256x256 tiles
# with K no multiple of 128, and few output tiles with K no multiple of 256.
OFFERED = [(4296, 4200, 3000), (7680, 2560, 4000), (264, 136, 8191), (1024, 1024, 16384 - 128)]


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("M,N,K", OFFERED)
def test_weight_gradient_without_the_offered_workspace(M, N, K, accumulate):
    assert B.slapo_weight_grad_workspace(W.BF16, M, N, K) > 0
    gen = torch.Generator(device=DEV).manual_seed(K)
    A, Bm, C0 = (torch.randn(*s, device=DEV, generator=gen).to(torch.bfloat16) for s in ((K, M), (K, N), (M, N)))
    out, plain = C0.clone(), C0.clone()
    B.slapo_weight_grad(W.BF16, accumulate, M, N, K, A, Bm, out, None)
    B.slapo_gemm_ex(W.BF16, B.TN, B.EPI_ADD if accumulate else B.EPI_NONE, 0, M, N, K, A, Bm, plain, aux_in=plain if accumulate else None, flags=B.GEMM_SHARED)
    assert torch.equal(out, plain)


# Every epilogue in every tile form, with ragged edges, without and with a partial last slab: 256x256 tiles, 128x128 with
# four LDS stages (layout TN: split slabs from K > 1024 on) and with two, 128x64. Pairs of layout and epilogue that no
# layer uses come as 128x128 tiles only. Bound: rounding of the stored result (2^-9 of it in bf16, 2^-12 in half) and of
# the sums, doubled.
FORMS = {"256x256": (3592, 3344, "256, 256, 64, 2, 4, 1, 2, 0"), "128x128-4": (1664, 2064, "128, 128, 64, 2, 4, 1, 4, 4"),
         "128x128-2": (2336, 2064, "128, 128, 64, 2, 4, 1, 2, 4"), "128x64": (520, 144, "128, 64, 64, 2, 2, 1, 4, 4")}
PAIRED = {B.NT: (B.EPI_NONE, B.EPI_BIAS, B.EPI_BIAS_ACT, B.EPI_GATE), B.NN: (B.EPI_NONE, B.EPI_DACT, B.EPI_ADD, B.EPI_DGATE),
          B.TN: (B.EPI_NONE, B.EPI_ADD)}


@pytest.mark.parametrize("dtype", [W.BF16, W.FP16])
@pytest.mark.parametrize("layout", [B.NT, B.NN, B.TN])
@pytest.mark.parametrize("form", list(FORMS))
def test_epilogues_of_every_tile_form(form, layout, dtype):
    M, N, name = FORMS[form]
    tol = {W.BF16: 4e-3, W.FP16: 5e-4}[dtype]
    for K in (192, 203 if layout == B.TN else 200) + ((1088, 2286) if form == "128x128-4" and layout == B.TN else ()):
        if K > 1024:
            name = "128, 128, 64, 2, 2, 2, 4, 4"
        rng = np.random.default_rng(M + K + layout)
        a = store(rng.standard_normal((M, K)), dtype)
        b = store(rng.standard_normal((K, N)) * K ** -0.5, dtype)
        bias, aux = store(rng.standard_normal(N), dtype), store(rng.standard_normal((M, 2 * N)), dtype)
        acc = (torch.from_numpy(a) @ torch.from_numpy(b)).double().numpy()
        A = to_dev(a.T.copy() if layout == B.TN else a, dtype)
        Bm = to_dev(b.T.copy() if layout == B.NT else b, dtype)
        bd, auxd, aux1 = to_dev(bias, dtype), to_dev(aux, dtype), to_dev(aux[:, :N].copy(), dtype)

        def run(epi, act=W.GELU, width=N, aux_in=None, aux_out=None):
            got = B.slapo_gemm_kernel_name(dtype, layout, epi, M, N, K)
            assert name in got or epi not in PAIRED[layout] and "128, 128, 64, 2, 4, 1, %d, 4" % (2 if form in ("256x256", "128x128-2") else 4) in got, (epi, got)
            out = torch.full((M, width), 7.0, dtype=A.dtype, device=DEV)
            B.slapo_gemm(dtype, layout, epi, act, M, N, K, A, Bm, out, bias=bd, aux_in=aux_in, aux_out=aux_out)
            return out

        pre, keep = acc + bias, torch.empty(M, N, dtype=A.dtype, device=DEV)
        errs = {"none": err(run(B.EPI_NONE), acc), "bias": err(run(B.EPI_BIAS), pre), "add": err(run(B.EPI_ADD, aux_in=aux1), acc + aux[:, :N]),
                "dgelu": err(run(B.EPI_DACT, aux_in=aux1), acc * aux[:, :N]),
                "drelu": err(run(B.EPI_DACT, W.RELU, aux_in=aux1), acc * (aux[:, :N] > 0)),
                "dgate": err(run(B.EPI_DGATE, width=2 * N, aux_in=auxd), np.repeat(acc, 2, 1) * aux),
                "relu": err(run(B.EPI_BIAS_ACT, W.RELU), np.maximum(pre, 0)),
                "gelu": err(run(B.EPI_BIAS_ACT, aux_out=keep), _act(pre, W.GELU))}
        errs["gelu'"] = err(keep, _dact(pre, W.GELU))
        gate, up = acc[:, ::2], acc[:, 1::2]
        sig = 1 / (1 + np.exp(-gate))
        errs["gate"] = err(run(B.EPI_GATE, width=N // 2, aux_out=keep), gate * sig * up)
        errs["gate'"] = err(keep, np.stack([up * sig * (1 + gate * (1 - sig)), gate * sig], 2).reshape(M, N))
        assert all(v <= tol for v in errs.values()), (K, errs)


# layout TN from K > 1024 on (split slabs), and short K in several rounds (two LDS stages)
@pytest.mark.parametrize("M,N,Ks,name", [(768, 3072, (1025, 1087, 2286), "2, 2, 2, 4, 4"), (5120, 1280, (7, 65, 1000), "2, 4, 1, 2, 4")])
def test_gemm_partial_last_slab_tn(M, N, Ks, name):
    for K in Ks:
        assert name in B.slapo_gemm_kernel_name(W.BF16, B.TN, B.EPI_NONE, M, N, K)
    test_gemm_partial_last_slab(B.TN, Ks, M, N)


# 64x64 tiles with 128-deep slabs: K of whole slabs, one piece more, one less, odd slab counts; ragged edges
@pytest.mark.parametrize("layout", [B.NT, B.NN])
@pytest.mark.parametrize("M,N", [(64, 64), (65, 8), (129, 200), (9, 2048)])
def test_gemm_64x64_tiles(layout, M, N):
    Ks = (256, 264, 376, 640, 1016)
    for K in Ks:
        assert "64, 64, 128, 2, 2, 1, 3, 4, " + ("false" if K % 128 == 0 else "true") in B.slapo_gemm_kernel_name(W.BF16, layout, B.EPI_NONE, M, N, K)
    test_gemm_partial_last_slab(layout, Ks, M, N)


@pytest.mark.parametrize("dtype", [W.BF16, W.FP16])
@pytest.mark.parametrize("layout", [B.NT, B.NN])
def test_epilogues_of_64x64_tiles(layout, dtype):
    """The bound of test_epilogues_of_every_tile_form, at the K that these tiles start from."""
    M, N, name = 264, 144, "64, 64, 128, 2, 2, 1, 3, 4"
    for K in (256, 328):
        rng = np.random.default_rng(K + layout)
        a, b = store(rng.standard_normal((M, K)), dtype), store(rng.standard_normal((K, N)) * K ** -0.5, dtype)
        bias, aux = store(rng.standard_normal(N), dtype), store(rng.standard_normal((M, 2 * N)), dtype)
        acc = a.astype(np.float64) @ b.astype(np.float64)
        A, Bm = to_dev(a, dtype), to_dev(b.T.copy() if layout == B.NT else b, dtype)
        keep = torch.empty(M, N, dtype=A.dtype, device=DEV)

        def run(epi, act=W.GELU, width=N, aux_in=None, aux_out=None):
            assert name in B.slapo_gemm_kernel_name(dtype, layout, epi, M, N, K)
            out = torch.full((M, width), 7.0, dtype=A.dtype, device=DEV)
            B.slapo_gemm(dtype, layout, epi, act, M, N, K, A, Bm, out, bias=to_dev(bias, dtype), aux_in=aux_in, aux_out=aux_out)
            return out

        if layout == B.NT:
            gate, up = acc[:, ::2], acc[:, 1::2]
            errs = {"bias": err(run(B.EPI_BIAS), acc + bias), "gelu": err(run(B.EPI_BIAS_ACT, aux_out=keep), _act(acc + bias, W.GELU))}
            errs["gelu'"] = err(keep, _dact(acc + bias, W.GELU))
            errs["gate"] = err(run(B.EPI_GATE, width=N // 2, aux_out=keep), gate / (1 + np.exp(-gate)) * up)
        else:
            aux1 = to_dev(aux[:, :N].copy(), dtype)
            errs = {"add": err(run(B.EPI_ADD, aux_in=aux1), acc + aux[:, :N]), "dgelu": err(run(B.EPI_DACT, aux_in=aux1), acc * aux[:, :N]),
                    "dgate": err(run(B.EPI_DGATE, width=2 * N, aux_in=to_dev(aux, dtype)), np.repeat(acc, 2, 1) * aux)}
        assert all(v <= {W.BF16: 4e-3, W.FP16: 5e-4}[dtype] for v in errs.values()), (K, errs)


# a thin last round in quarters of tiles (a product that has the chip to itself): the bits of whole tiles (GEMM_SHARED). One row or
# eight columns beyond whole tiles (quarters without rows or columns), 1 to 128 tiles beyond a round, partial slabs of 128 and of 64.
@pytest.mark.parametrize("M,N,K", [(4097, 4096, 256), (4096, 4104, 264), (65700, 240, 320), (4200, 4200, 392), (2331, 8192, 512), (4096, 6144, 1032)])
@pytest.mark.parametrize("layout,epi", [(B.NT, B.EPI_NONE), (B.NT, B.EPI_BIAS), (B.NT, B.EPI_BIAS_ACT), (B.NT, B.EPI_GATE), (B.NN, B.EPI_NONE), (B.NN, B.EPI_DACT),
                                        (B.NN, B.EPI_ADD), (B.NN, B.EPI_DGATE)])
def test_gemm_thin_round_in_quarters(layout, epi, M, N, K):
    dtype = W.FP16 if K % 16 else W.BF16
    if epi == B.EPI_GATE:
        N = (N + 15) // 16 * 16   # (pairs in whole 16-byte pieces of the gated output: other N are refused)
    name = B.slapo_gemm_kernel_name(dtype, layout, epi, M, N, K)
    assert "quarters" in name and "quarters" not in B.slapo_gemm_kernel_name(dtype, layout, epi, M, N, K, flags=B.GEMM_SHARED)
    g = torch.Generator(device=DEV).manual_seed(M + K)
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=g).mul_(0.25).to(tdtype(dtype))
    a, b = rnd(M, K), rnd(N, K) if layout == B.NT else rnd(K, N)
    kw = {}
    if epi in (B.EPI_BIAS, B.EPI_BIAS_ACT):
        kw["bias"] = rnd(N)
    if epi in (B.EPI_DACT, B.EPI_ADD, B.EPI_DGATE):
        kw["aux_in"] = rnd(M, N * (2 if epi == B.EPI_DGATE else 1))
    got = []
    for flags in (0, B.GEMM_SHARED):
        c = torch.full((M, 2 * N if epi == B.EPI_DGATE else N // 2 if epi == B.EPI_GATE else N), float("nan"), dtype=a.dtype, device=DEV)
        aux = torch.full((M, N), float("nan"), dtype=a.dtype, device=DEV) if epi in (B.EPI_BIAS_ACT, B.EPI_GATE) else None
        B.slapo_gemm_ex(dtype, layout, epi, W.GELU, M, N, K, a, b, c, aux_out=aux, flags=flags, **kw)
        got.append((c, aux))
    assert torch.isfinite(got[0][0]).all() and torch.equal(got[0][0], got[1][0])
    assert got[0][1] is None or torch.equal(got[0][1], got[1][1])
    if epi in (B.EPI_NONE, B.EPI_ADD):   # one in 16 rows against a product of its own
        rows = torch.arange((M - 1) % 16, M, 16, device=DEV)
        bt = b.float().t().contiguous() if layout == B.NT else b.float()
        ref = a[rows].float() @ bt + (kw["aux_in"][rows].float() if epi == B.EPI_ADD else 0)
        assert err(got[0][0][rows], to_np(ref)) <= TOL[dtype]


# tiles that make the product one round: two rows and eight columns beyond whole tiles, partial slabs
@pytest.mark.parametrize("dtype", [W.BF16, W.FP16])
@pytest.mark.parametrize("layout", [B.NT, B.NN])
@pytest.mark.parametrize("M,N,name", [(2306, 2192, "192, 128, 64, 2, 4, 1, 3, 4"), (2050, 3472, "256, 128, 64, 2, 4, 1, 3, 4"), (3266, 3344, "192, 256, 64, 2, 4, 1, 2, 0")])
def test_epilogues_of_one_round_tiles(M, N, name, layout, dtype):
    """The bound of test_epilogues_of_every_tile_form."""
    for K in (768, 840):
        rng = np.random.default_rng(K + layout + M)
        a, b = store(rng.standard_normal((M, K)), dtype), store(rng.standard_normal((K, N)) * K ** -0.5, dtype)
        bias, aux = store(rng.standard_normal(N), dtype), store(rng.standard_normal((M, 2 * N)), dtype)
        acc = (torch.from_numpy(a) @ torch.from_numpy(b)).double().numpy()
        A, Bm = to_dev(a, dtype), to_dev(b.T.copy() if layout == B.NT else b, dtype)
        keep = torch.empty(M, N, dtype=A.dtype, device=DEV)

        def run(epi, act=W.GELU, width=N, aux_in=None, aux_out=None):
            assert name in B.slapo_gemm_kernel_name(dtype, layout, epi, M, N, K)
            out = torch.full((M + 1, width), 7.0, dtype=A.dtype, device=DEV)
            B.slapo_gemm(dtype, layout, epi, act, M, N, K, A, Bm, out[:M], bias=to_dev(bias, dtype), aux_in=aux_in, aux_out=aux_out)
            assert (out[M] == 7).all()
            return out[:M]

        errs = {"none": err(run(B.EPI_NONE), acc)}
        if layout == B.NT:
            gate, up = acc[:, ::2], acc[:, 1::2]
            errs.update({"bias": err(run(B.EPI_BIAS), acc + bias), "gelu": err(run(B.EPI_BIAS_ACT, aux_out=keep), _act(acc + bias, W.GELU))})
            errs["gelu'"] = err(keep, _dact(acc + bias, W.GELU))
            errs["gate"] = err(run(B.EPI_GATE, width=N // 2, aux_out=keep), gate / (1 + np.exp(-gate)) * up)
        else:
            aux1 = to_dev(aux[:, :N].copy(), dtype)
            errs.update({"add": err(run(B.EPI_ADD, aux_in=aux1), acc + aux[:, :N]), "dgelu": err(run(B.EPI_DACT, aux_in=aux1), acc * aux[:, :N]),
                         "dgate": err(run(B.EPI_DGATE, width=2 * N, aux_in=to_dev(aux, dtype)), np.repeat(acc, 2, 1) * aux)})
        assert all(v <= {W.BF16: 4e-3, W.FP16: 5e-4}[dtype] for v in errs.values()), (K, errs)


# 64x32 tiles: from 33 tiles of 64x64 to 256 of 64x32; ragged edges, partial slabs, one slab count more and less than the stages
@pytest.mark.parametrize("M,N", [(64, 2056), (65, 1032), (129, 2608), (256, 2048)])
def test_gemm_64x32_tiles(M, N):
    Ks = (256, 264, 376, 504, 640, 1016)
    for K in Ks:
        assert "64, 32, 128, 2, 2, 1, 4, 4, " + ("false" if K % 128 == 0 else "true") in B.slapo_gemm_kernel_name(W.BF16, B.NT, B.EPI_NONE, M, N, K)
    for M_, N_ in ((64, 2048), (257, 2048)):
        assert "64, 32, " not in B.slapo_gemm_kernel_name(W.BF16, B.NT, B.EPI_NONE, M_, N_, 256)
    test_gemm_partial_last_slab(B.NT, Ks, M, N)


@pytest.mark.parametrize("dtype", [W.BF16, W.FP16])
def test_epilogues_of_64x32_tiles(dtype):
    """The bound of test_epilogues_of_every_tile_form, in the products that have these tiles."""
    M, N = 130, 1040
    for K in (256, 328):
        rng = np.random.default_rng(K)
        a, b, bias = store(rng.standard_normal((M, K)), dtype), store(rng.standard_normal((K, N)) * K ** -0.5, dtype), store(rng.standard_normal(N), dtype)
        acc = a.astype(np.float64) @ b.astype(np.float64)
        A, Bm, keep = to_dev(a, dtype), to_dev(b.T.copy(), dtype), torch.empty(M, N, dtype=to_dev(a, dtype).dtype, device=DEV)

        def run(epi, act=W.GELU, width=N, aux_out=None):
            assert "64, 32, 128" in B.slapo_gemm_kernel_name(dtype, B.NT, epi, M, N, K)
            out = torch.full((M, width), 7.0, dtype=A.dtype, device=DEV)
            B.slapo_gemm(dtype, B.NT, epi, act, M, N, K, A, Bm, out, bias=to_dev(bias, dtype), aux_out=aux_out)
            return out

        gate, up = acc[:, ::2], acc[:, 1::2]
        errs = {"bias": err(run(B.EPI_BIAS), acc + bias), "gelu": err(run(B.EPI_BIAS_ACT, aux_out=keep), _act(acc + bias, W.GELU))}
        errs["gelu'"] = err(keep, _dact(acc + bias, W.GELU))
        errs["gate"] = err(run(B.EPI_GATE, width=N // 2, aux_out=keep), gate / (1 + np.exp(-gate)) * up)
        assert all(v <= {W.BF16: 4e-3, W.FP16: 5e-4}[dtype] for v in errs.values()), (K, errs)
