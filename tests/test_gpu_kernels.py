"""GPU parity of single kernels (through the C ABI) against their plain definitions in fp64."""
import math

import numpy as np
import pytest
import torch
from scipy.special import erf

import paper_2403_10616_amd as dp
from oracle import dipaco_oracle as orc
from gpu_util import DEV, dev, fma32, host, median_us, rel_l2

pytestmark = pytest.mark.gpu

TDT = {dp.F32: torch.float32, dp.BF16: torch.bfloat16}


def _rand(shape, seed, dtype):
    """fp32 draws, rounded to the kernel's operand type so that the fp64 reference sees the same values."""
    x = np.random.default_rng(seed).standard_normal(shape).astype(np.float32)
    t = torch.from_numpy(x).to(TDT[dtype])
    return t.to(DEV), t.to(torch.float64).numpy()


@pytest.fixture(params=[0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14], ids=lambda t: f"tile{t}")
def gemm_tile(request):
    """Every workgroup tile shape must reach the same parity; 0 is the library's own choice."""
    dp.dipaco_k_set_gemm_tile(request.param)
    yield request.param
    dp.dipaco_k_set_gemm_tile(0)


# (M, N, K): several tiles with ragged tails in every direction; K not a multiple of the K tile
GEMM_SHAPES = [(128, 128, 64), (200, 136, 72), (1, 8, 8), (300, 264, 520), (64, 512, 1000), (520, 776, 160),
               (257, 8, 32),
               # widths that are multiples of 224: the tile shape with columns every 224 takes them (tile 10)
               (300, 448, 544), (520, 224, 160), (257, 896, 64),
               # short contractions around the depth of the LDS rings (K tiles of 64 in a ring of two, of 32 in a ring of
               # four): one to five K tiles of either size, so that every prologue / steady / tail split runs
               (130, 72, 128), (300, 264, 192), (264, 520, 320), (200, 136, 96), (72, 264, 384)]


@pytest.mark.parametrize("dtype", [dp.F32, dp.BF16])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_forward_layout_with_epilogues(dtype, M, N, K, gemm_tile):
    print(f"gemm fwd tile={gemm_tile} dtype={dtype} M={M} N={N} K={K}", flush=True)
    A, Ar = _rand((M, K), 1, dtype)
    B, Br = _rand((K, N), 2, dtype)
    bias, br = _rand((N,), 3, dtype)
    resid, rr = _rand((M, N), 4, dtype)
    tol = 1e-5 if dtype == dp.F32 else 6e-3
    scale = math.sqrt(K)
    # plain
    C = torch.empty((M, N), dtype=TDT[dtype], device=DEV)
    dp.dipaco_k_gemm(dtype, False, False, False, M, N, K, A, B, C)
    ref = Ar @ Br
    assert np.abs(host(C) - ref).max() <= tol * scale * 4
    assert rel_l2(host(C), ref) <= tol
    # bias + residual
    dp.dipaco_k_gemm(dtype, False, False, False, M, N, K, A, B, C, bias=bias, resid=resid)
    assert rel_l2(host(C), ref + br + rr) <= tol
    # bias + GELU, pre-activation saved
    U = torch.empty_like(C)
    dp.dipaco_k_gemm(dtype, False, False, False, M, N, K, A, B, C, bias=bias, aux_out=U, act=1)
    u_ref = ref + br
    assert rel_l2(host(U), u_ref) <= tol
    u_seen = host(U).astype(np.float64)
    g_ref = 0.5 * u_seen * (1 + erf(u_seen / math.sqrt(2)))
    assert rel_l2(host(C), g_ref) <= tol
    # bias + GELU, derivative saved (what the path step uses): both from the unrounded pre-activation
    dp.dipaco_k_gemm(dtype, False, False, False, M, N, K, A, B, C, bias=bias, aux_out=U, act=3)
    assert rel_l2(host(C), 0.5 * u_ref * (1 + erf(u_ref / math.sqrt(2)))) <= tol
    d_ref = 0.5 * (1 + erf(u_ref / math.sqrt(2))) + u_ref * np.exp(-0.5 * u_ref * u_ref) / math.sqrt(2 * math.pi)
    assert rel_l2(host(U), d_ref) <= tol
    with pytest.raises(dp.DipacoError):
        dp.dipaco_k_gemm(dtype, False, False, False, M, N, K, A, B, C, act=1)   # no aux_out: refused on the host


@pytest.mark.parametrize("dtype", [dp.F32, dp.BF16])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_input_gradient_layout(dtype, M, N, K, gemm_tile):
    print(f"gemm dX tile={gemm_tile} dtype={dtype} M={M} N={N} K={K}", flush=True)
    A, Ar = _rand((M, K), 5, dtype)
    Bt, Btr = _rand((N, K), 6, dtype)          # B stored [N, K]
    U, Ur = _rand((M, N), 7, dtype)
    tol = 1e-5 if dtype == dp.F32 else 6e-3
    C = torch.empty((M, N), dtype=TDT[dtype], device=DEV)
    dp.dipaco_k_gemm(dtype, False, True, False, M, N, K, A, Bt, C)
    ref = Ar @ Btr.T
    assert rel_l2(host(C), ref) <= tol
    dp.dipaco_k_gemm(dtype, False, True, False, M, N, K, A, Bt, C, aux_in=U, act=2)
    gp = 0.5 * (1 + erf(Ur / math.sqrt(2))) + Ur * np.exp(-0.5 * Ur * Ur) / math.sqrt(2 * math.pi)
    assert rel_l2(host(C), ref * gp) <= tol
    dp.dipaco_k_gemm(dtype, False, True, False, M, N, K, A, Bt, C, aux_in=U, act=4)   # plain multiplication
    assert rel_l2(host(C), ref * Ur) <= tol


@pytest.mark.parametrize("dtype", [dp.F32, dp.BF16])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES + [(1000, 264, 64)])
def test_gemm_column_sums_of_the_output(dtype, M, N, K, gemm_tile):
    """The bias gradient taken in the epilogue: column sums of what the product writes (here the input-gradient
    layout with the saved-operand multiplication, as in the step)."""
    print(f"gemm colsum tile={gemm_tile} dtype={dtype} M={M} N={N} K={K}", flush=True)
    A, Ar = _rand((M, K), 11, dtype)
    Bt, Btr = _rand((N, K), 12, dtype)
    U, Ur = _rand((M, N), 13, dtype)
    C = torch.empty((M, N), dtype=TDT[dtype], device=DEV)
    cs = torch.full((N,), 77.0, dtype=torch.float32, device=DEV)
    scratch = torch.full((((M + 31) // 32) * N,), float("nan"), dtype=torch.float32, device=DEV)
    dp.dipaco_k_gemm_colsum(dtype, False, True, M, N, K, A, Bt, C, None, None, None, U, 4, cs, scratch)
    ref = (Ar @ Btr.T) * Ur
    tol = 1e-5 if dtype == dp.F32 else 6e-3
    assert rel_l2(host(C), ref) <= tol
    want = ref.sum(0)
    scale = np.abs(ref).sum(0).max()
    assert np.abs(host(cs) - want).max() <= (2e-6 if dtype == dp.F32 else 2e-3) * scale
    # forward layout with bias: same sums
    B2, B2r = _rand((K, N), 14, dtype)
    bias, biasr = _rand((N,), 15, dtype)
    dp.dipaco_k_gemm_colsum(dtype, False, False, M, N, K, A, B2, C, bias, None, None, None, 0, cs, scratch)
    ref2 = Ar @ B2r + biasr
    assert np.abs(host(cs) - ref2.sum(0)).max() <= (2e-6 if dtype == dp.F32 else 2e-3) * np.abs(ref2).sum(0).max()


@pytest.mark.parametrize("dtype", [dp.F32, dp.BF16])
@pytest.mark.parametrize("M,N,K,splits", [(128, 128, 64, 1), (200, 136, 77, 1), (72, 264, 1000, 4), (8, 8, 5, 1),
                                          (136, 64, 4099, 16), (264, 520, 1024, 5), (8, 776, 96, 1),
                                          (896, 1024, 2048, 8), (384, 1160, 512, 3)])
def test_gemm_weight_gradient_layout_and_split_k(dtype, M, N, K, splits, gemm_tile):
    print(f"gemm dW tile={gemm_tile} dtype={dtype} M={M} N={N} K={K} splits={splits}", flush=True)
    At, Atr = _rand((K, M), 8, dtype)          # A stored [K, M]: contraction over rows (tokens)
    B, Br = _rand((K, N), 9, dtype)
    C = torch.empty((M, N), dtype=torch.float32, device=DEV)
    partial = torch.empty((splits, M, N), dtype=torch.float32, device=DEV) if splits > 1 else None
    dp.dipaco_k_gemm(dtype, True, False, True, M, N, K, At, B, C, splits=splits, partial=partial)
    ref = Atr.T @ Br
    assert rel_l2(host(C), ref) <= 2e-6
    first = host(C).copy()
    dp.dipaco_k_gemm(dtype, True, False, True, M, N, K, At, B, C, splits=splits, partial=partial)
    assert np.array_equal(first, host(C))       # fixed summation order: bit-identical from call to call


def _attn_ref(qkv, B, S, H, dh):
    a = orc.Arch((1,), H * dh, H, dh, 8, 8, S)
    A = H * dh
    o = np.empty((B * S, A))
    lse = np.empty((B, H, S))
    probs = []
    for b in range(B):
        x = qkv[b * S:(b + 1) * S]
        ob, pb = orc._attention(x[:, :A], x[:, A:2 * A], x[:, 2 * A:], a)
        o[b * S:(b + 1) * S] = ob
        probs.append(pb)
        for h in range(H):
            s = (x[:, h * dh:(h + 1) * dh] @ x[:, A + h * dh:A + (h + 1) * dh].T) / math.sqrt(dh)
            s = np.where(np.tril(np.ones((S, S), bool)), s, -np.inf)
            mx = s.max(-1)
            lse[b, h] = mx + np.log(np.exp(s - mx[:, None]).sum(-1))
    return a, o, lse, probs


@pytest.fixture(params=[1, 0], ids=["single_block", "paired_blocks"])
def attn_blocks(request):
    """Both ways of dealing the causal triangle's blocks to workgroups; 1 is the default."""
    dp.dipaco_k_set_attention_blocks(request.param)
    yield request.param
    dp.dipaco_k_set_attention_blocks(1)


@pytest.mark.parametrize("dtype", [dp.F32, dp.BF16])
@pytest.mark.parametrize("B,S,H,dh", [(2, 64, 2, 32), (1, 200, 3, 64), (2, 77, 1, 128), (1, 1, 2, 64), (1, 333, 2, 64),
                                      (2, 1024, 2, 64), (1, 130, 1, 64), (1, 900, 1, 64), (1, 2048, 2, 64),
                                      (1, 1100, 1, 64)])
def test_attention_forward_backward(dtype, B, S, H, dh, attn_blocks):
    print(f"attention dtype={dtype} B={B} S={S} H={H} dh={dh} blocks={attn_blocks}", flush=True)
    A = H * dh
    qkv, qr = _rand((B * S, 3 * A), 10, dtype)
    d_o, gr = _rand((B * S, A), 11, dtype)
    o = torch.empty((B * S, A), dtype=TDT[dtype], device=DEV)
    lse = torch.empty((B, H, S), dtype=torch.float32, device=DEV)
    dp.dipaco_k_attention_fwd(dtype, qkv, o, lse, B, S, H, dh)
    a, o_ref, lse_ref, probs = _attn_ref(qr, B, S, H, dh)
    tol = 2e-5 if dtype == dp.F32 else 1e-2
    assert rel_l2(host(o), o_ref) <= tol
    # every element: with head size 64 the probabilities enter the second product rounded to bf16 (relative 2^-9 each,
    # averaging out over a row), and the result is rounded once more
    o_err = np.abs(host(o) - o_ref).max() / np.abs(o_ref).max()
    assert o_err <= (1e-5 if dtype == dp.F32 else 8e-3), o_err
    assert np.abs(host(lse) - lse_ref).max() <= (1e-5 if dtype == dp.F32 else 2e-2)
    dqkv = torch.empty_like(qkv)
    dsum = torch.empty(2 * B * H * ((S + 127) // 128 * 128), dtype=torch.float32, device=DEV)
    cs = torch.full((3 * A,), 55.0, dtype=torch.float32, device=DEV)
    cs_scratch = torch.full((max((B * S + 255) // 256, B * ((S + 127) // 128)) * 3 * A,), float("nan"),
                            dtype=torch.float32, device=DEV)
    dp.dipaco_k_attention_bwd(dtype, qkv, o, d_o, lse, dqkv, dsum, B, S, H, dh, colsum_out=cs, colsum_scratch=cs_scratch)
    ref = np.empty((B * S, 3 * A))
    for b in range(B):
        x = qr[b * S:(b + 1) * S]
        dq, dk, dv = orc._attention_bwd(gr[b * S:(b + 1) * S], x[:, :A], x[:, A:2 * A], x[:, 2 * A:], probs[b], a)
        ref[b * S:(b + 1) * S] = np.concatenate([dq, dk, dv], axis=1)
    got = host(dqkv)
    for name, sl in (("dq", slice(0, A)), ("dk", slice(A, 2 * A)), ("dv", slice(2 * A, 3 * A))):
        assert rel_l2(got[:, sl], ref[:, sl]) <= (2e-5 if dtype == dp.F32 else 2e-2), name
        top = np.abs(ref[:, sl]).max()
        worst = np.abs(got[:, sl] - ref[:, sl]).max() / (top if top > 0 else 1.0)      # S = 1: dq and dk are zero
        print(f"  {name}: max-abs error / max |{name}| = {worst:.2e}, o: {o_err:.2e}", flush=True)
        assert worst <= (2e-5 if dtype == dp.F32 else 2e-2), (name, worst)
    # column sums of dqkv (the QKV bias gradient), taken in the kernels' epilogues where the matrix-core path runs
    scale = np.abs(ref).sum(0).max()
    assert np.abs(host(cs) - ref.sum(0)).max() <= (1e-5 if dtype == dp.F32 else 1e-2) * scale
    dqkv2 = torch.empty_like(qkv)
    dp.dipaco_k_attention_bwd(dtype, qkv, o, d_o, lse, dqkv2, dsum, B, S, H, dh)            # without the sums
    assert torch.equal(dqkv2, dqkv)


@pytest.mark.parametrize("dtype", [dp.F32, dp.BF16])
@pytest.mark.parametrize("B,S,H,dh", [(1, 1, 1, 32), (2, 31, 3, 32), (1, 129, 2, 32), (1, 515, 1, 32), (1, 1, 1, 128),
                                      (2, 33, 1, 128), (1, 64, 2, 128), (1, 127, 1, 128), (2, 256, 2, 128),
                                      (1, 515, 3, 128), (3, 17, 1, 64), (1, 96, 5, 64)])
def test_attention_head_sizes_at_tile_edges(dtype, B, S, H, dh):
    """Head sizes 32 (half a panel) and 128 (two panels; one 32-query block at a time in dK/dV) and the fp32 kernels'
    16-row waves: one position, one row past a wave / tile / block, several blocks with a ragged last one."""
    test_attention_forward_backward(dtype, B, S, H, dh, 1)


@pytest.mark.parametrize("B,S,H,dh", [(1, 385, 1, 32), (1, 385, 2, 64), (1, 385, 1, 128), (2, 640, 3, 32), (2, 641, 3, 64), (1, 700, 2, 128),
                                      (8, 400, 11, 64), (8, 400, 12, 64), (8, 400, 12, 32), (8, 400, 12, 128)])
def test_attention_with_two_groups_of_waves_a_block(B, S, H, dh, attn_blocks):
    """Four blocks long or longer and few of them: two groups take a block's tiles in turn; 352 and 384 blocks of 128 rows lie on the two
    sides of that rule.  Odd and even numbers of tiles, the last one ragged."""
    test_attention_forward_backward(dp.BF16, B, S, H, dh, attn_blocks)


# ---- the benchmarked kernels at the step's own shapes, element by element ---------------------------------------
def _bf16_ulp(x):
    """Spacing of bf16 numbers at |x| (8 significant bits)."""
    mag = np.maximum(np.abs(x), 2.0 ** -126)
    return 2.0 ** (np.floor(np.log2(mag)) - 7)


def _assert_within_one_bf16_ulp(got, ref, what):
    """The kernels accumulate exactly representable bf16 products in fp32 and round once: the stored value is the
    fp64 result rounded to bf16, give or take the fp32 accumulation error (which can tip a rounding, and is all that
    is left of elements near zero: 2e-5 of the result's typical magnitude covers it)."""
    got = got.astype(np.float64)
    slack = 2e-5 * math.sqrt(float(np.mean(ref * ref)))
    excess = np.abs(got - ref) - (_bf16_ulp(np.maximum(np.abs(ref), np.abs(got))) + slack)
    worst = int(np.argmax(excess))
    assert excess.flat[worst] <= 0, (what, np.unravel_index(worst, ref.shape), got.flat[worst], ref.flat[worst])


STEP_M = 32768
# (name, M, N, K): the forward products of one block at config 2 and a 4096-row slice of the vocabulary head
STEP_FORWARD = [("qkv", STEP_M, 2688, 896), ("out_proj", STEP_M, 896, 896), ("mlp_up", STEP_M, 3584, 896),
                ("mlp_down", STEP_M, 896, 3584), ("head_rows", 4096, 32000, 896)]


@pytest.mark.parametrize("name,M,N,K", STEP_FORWARD, ids=[s[0] for s in STEP_FORWARD])
def test_bf16_forward_products_of_the_step_element_by_element(name, M, N, K):
    print(f"step-shape forward product {name} M={M} N={N} K={K}", flush=True)
    A, Ar = _rand((M, K), 21, dp.BF16)
    B, Br = _rand((K, N), 22, dp.BF16)
    Br *= 0.05                                   # weight-sized entries keep GELU in its curved range
    B = torch.from_numpy(Br).to(torch.bfloat16)
    Br = B.to(torch.float64).numpy()
    B = B.to(DEV)
    bias, br = _rand((N,), 23, dp.BF16)
    resid, rr = _rand((M, N), 24, dp.BF16)
    ref = Ar @ Br
    C = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    if name == "head_rows":                      # plain product
        dp.dipaco_k_gemm(dp.BF16, False, False, False, M, N, K, A, B, C)
        _assert_within_one_bf16_ulp(host(C), ref, name)
        return
    if name == "mlp_up":                         # + bias, GELU out, GELU' saved
        U = torch.empty_like(C)
        dp.dipaco_k_gemm(dp.BF16, False, False, False, M, N, K, A, B, C, bias=bias, aux_out=U, act=3)
        u = ref + br
        cdf = 0.5 * (1 + erf(u / math.sqrt(2)))
        _assert_within_one_bf16_ulp(host(C), u * cdf, name + " GELU")
        _assert_within_one_bf16_ulp(host(U), cdf + u * np.exp(-0.5 * u * u) / math.sqrt(2 * math.pi), name + " GELU'")
        return
    if name == "qkv":                            # + bias
        dp.dipaco_k_gemm(dp.BF16, False, False, False, M, N, K, A, B, C, bias=bias)
        _assert_within_one_bf16_ulp(host(C), ref + br, name)
        return
    dp.dipaco_k_gemm(dp.BF16, False, False, False, M, N, K, A, B, C, bias=bias, resid=resid)   # + bias + residual
    _assert_within_one_bf16_ulp(host(C), ref + br + rr, name)


# input-gradient products dX = dY W^T (W stored [N_out = rows here, K]) of one block, and a slice of the head's
STEP_INPUT_GRAD = [("d_qkv_in", STEP_M, 896, 2688), ("d_out_proj_in", STEP_M, 896, 896), ("d_mlp_up_in", STEP_M, 896, 3584),
                   ("d_mlp_down_in", STEP_M, 3584, 896), ("d_head_in_rows", 4096, 896, 32000)]


@pytest.mark.parametrize("name,M,N,K", STEP_INPUT_GRAD, ids=[s[0] for s in STEP_INPUT_GRAD])
def test_bf16_input_gradient_products_of_the_step_element_by_element(name, M, N, K):
    print(f"step-shape input-gradient product {name} M={M} N={N} K={K}", flush=True)
    A, Ar = _rand((M, K), 25, dp.BF16)
    Bt, Btr = _rand((N, K), 26, dp.BF16)
    ref = Ar @ Btr.T
    C = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    if name != "d_mlp_down_in":
        dp.dipaco_k_gemm(dp.BF16, False, True, False, M, N, K, A, Bt, C)
        _assert_within_one_bf16_ulp(host(C), ref, name)
        return
    # the product that writes dU: multiplied by the saved GELU', with the column sums (the gradient of b_up)
    U, Ur = _rand((M, N), 27, dp.BF16)
    cs = torch.full((N,), 77.0, dtype=torch.float32, device=DEV)
    scratch = torch.full((((M + 31) // 32) * N,), float("nan"), dtype=torch.float32, device=DEV)
    dp.dipaco_k_gemm_colsum(dp.BF16, False, True, M, N, K, A, Bt, C, None, None, None, U, 4, cs, scratch)
    ref = ref * Ur
    _assert_within_one_bf16_ulp(host(C), ref, name)
    assert np.abs(host(cs) - ref.sum(0)).max() <= 1e-5 * np.abs(ref).sum(0).max()   # fp32 sums of unrounded values


STEP_WEIGHT_GRAD = [("d_w_qkv", 896, 2688), ("d_w_o", 896, 896), ("d_w_up", 896, 3584), ("d_w_down", 3584, 896)]


@pytest.mark.parametrize("name,M,N", STEP_WEIGHT_GRAD, ids=[s[0] for s in STEP_WEIGHT_GRAD])
def test_bf16_weight_gradient_products_of_the_step_element_by_element(name, M, N):
    """dW = X^T dY over the 32768 tokens, fp32 out, with the split-K plan the step launches them with."""
    K = STEP_M
    print(f"step-shape weight-gradient product {name} M={M} N={N} K={K}", flush=True)
    At, Atr = _rand((K, M), 28, dp.BF16)
    B, Br = _rand((K, N), 29, dp.BF16)
    plan = dp.dipaco_k_gemm_split_plan(M, N, K, 32)
    splits = max(plan["slices"]) if plan["tile"][0] else 8
    C = torch.empty((M, N), dtype=torch.float32, device=DEV)
    partial = torch.empty((splits, M, N), dtype=torch.float32, device=DEV)
    dp.dipaco_k_gemm(dp.BF16, True, False, True, M, N, K, At, B, C, splits=splits, partial=partial)
    ref = Atr.T @ Br
    rms = math.sqrt(float(np.mean(ref * ref)))
    err = np.abs(host(C).astype(np.float64) - ref)
    assert err.max() <= 1e-4 * rms, (name, np.unravel_index(int(np.argmax(err)), ref.shape), err.max() / rms)


# Edges of the fitted tiles (heights 32, 64, 96, 128, 160; widths 64 and 128), of a group's 64 bytes of K and of a stage of two
# or eight groups; contractions that end inside a group.  Bounds: fp32 sums of K products, 2^-24 sqrt(K) each side, and one
# bf16 rounding (2^-9) of the output.
@pytest.mark.parametrize("dtype", [dp.F32, dp.BF16])
@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 14])
@pytest.mark.parametrize("M,N,K", [(33, 72, 8), (65, 136, 24), (161, 128, 40), (320, 264, 264), (159, 120, 520), (97, 8, 2056),
                                   (160, 1160, 96)])
def test_gemm_fitted_tiles_at_their_edges(dtype, tile, M, N, K):
    print(f"gemm fit dtype={dtype} tile={tile} M={M} N={N} K={K}", flush=True)
    g = torch.Generator().manual_seed(M + N + K)
    mk = lambda *shape: torch.randn(shape, generator=g).to(TDT[dtype]).to(DEV)
    A, B, Bt, R = mk(M, K), mk(K, N), mk(N, K), mk(M, N)
    X, Y = mk(K + 5, ((M + 7) // 8) * 8), mk(K + 5, N)        # weight gradient: the contraction need not be a multiple of 8
    C = torch.empty((M, N), dtype=TDT[dtype], device=DEV)
    W = torch.empty((X.shape[1], N), device=DEV)
    P = torch.empty((3,) + tuple(W.shape), device=DEV)
    blank = lambda *ts: [t.fill_(float("nan")) for t in ts]   # nothing an earlier product wrote may pass for this one's
    rel = lambda got, ref: float((got.double() - ref).norm() / ref.norm())
    tol = 1e-6 if dtype == dp.F32 else 2.0 ** -9
    dp.dipaco_k_set_gemm_tile(tile)
    try:
        blank(C)
        dp.dipaco_k_gemm(dtype, False, False, False, M, N, K, A, B, C, resid=R)
        assert rel(C, A.double() @ B.double() + R.double()) <= tol
        blank(C)
        dp.dipaco_k_gemm(dtype, False, True, False, M, N, K, A, Bt, C)
        assert rel(C, A.double() @ Bt.double().T) <= tol
        for splits in (1, 3):
            blank(W, P)
            dp.dipaco_k_gemm(dtype, True, False, True, W.shape[0], N, K + 5, X, Y, W, splits=splits, partial=P)
            assert rel(W, X.double().T @ Y.double()) <= 1e-6
    finally:
        dp.dipaco_k_set_gemm_tile(0)


@pytest.mark.parametrize("M,N,K", [(4097, 4096, 64), (4360, 4096, 32), (5700, 3584, 96), (1025, 16392, 64), (2800, 16384, 32)])
def test_bf16_products_whose_last_round_is_taken_in_fitted_tiles(M, N, K):
    """More than one round of 256 tiles of 256 x 256, the last one mostly empty: its rows are a second launch."""
    test_gemm_forward_layout_with_epilogues(dp.BF16, M, N, K, 0)
    test_gemm_input_gradient_layout(dp.BF16, M, N, K, 0)


@pytest.mark.parametrize("M,N,K,split", [(5700, 3584, 896, True), (5000, 3584, 3584, True), (5000, 5000, 4992, False), (32768, 2688, 896, False)])
def test_last_round_is_taken_in_fitted_tiles_only_where_that_is_ahead(M, N, K, split):
    """Told by the bits: forced, the direct-to-LDS kernel takes all rows."""
    A, B = torch.randn((M, K), device=DEV).to(torch.bfloat16), torch.randn((K, N), device=DEV).to(torch.bfloat16)
    C = {t: torch.empty((M, N), dtype=torch.bfloat16, device=DEV) for t in (0, 5)}
    try:
        for t in C:
            dp.dipaco_k_set_gemm_tile(t)
            dp.dipaco_k_gemm(dp.BF16, False, False, False, M, N, K, A, B, C[t])
    finally:
        dp.dipaco_k_set_gemm_tile(0)
    assert torch.equal(C[0], C[5]) != split


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)], ids=["A.B", "A.Bt", "At.B"])
@pytest.mark.parametrize("tile", [3, 4])
@pytest.mark.parametrize("M,N,K", [(128, 128, 32), (132, 136, 36), (256, 264, 500), (4, 8, 4), (260, 120, 2052)])
def test_fp32_products_from_bf16_parts(ta, tb, M, N, K, tile):
    """The 128 x 128 fp32 tile and the 64 x 128 one (four groups of waves along K) multiply three bf16 parts of every number.  The part products left out and the cut-off of a
    matrix-core step stay below 2^-22 of a step of 32, and the steps are added in fp32; numbers whose first part is not finite take
    the fp32 way."""
    dp.dipaco_k_set_gemm_tile(tile)
    try:
        A, Ar = _rand((K, M) if ta else (M, K), 21, dp.F32)
        B, Br = _rand((N, K) if tb else (K, N), 22, dp.F32)
        Br = Br.T if tb else Br
        C = torch.empty((M, N), dtype=torch.float32, device=DEV)
        run = lambda: dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, A, B, C)
        run()
        ref = (Ar.T if ta else Ar) @ Br
        assert rel_l2(host(C), ref) <= 2.0 ** -22 + 2.0 ** -25 * math.sqrt((K + 31) // 32)
        before = host(C).copy()
        row = lambda m: A[:, m] if ta else A[m]
        row(1)[K - 1] = math.inf
        row(2).zero_()
        row(2)[0] = 3.4e38                       # finite, but its first bf16 part is not
        B.mul_(0.125)
        run()
        got = host(C)
        with np.errstate(over="ignore"):
            assert np.array_equal(got[1], np.where(Br[K - 1] > 0, np.inf, -np.inf).astype(np.float32))
        assert np.allclose(got[2], 3.4e38 * 0.125 * Br[0], rtol=1e-6)
        assert np.array_equal(got[3:], before[3:] * np.float32(0.125)) and np.array_equal(got[0], before[0] * np.float32(0.125))
    finally:
        dp.dipaco_k_set_gemm_tile(0)


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)], ids=["A.B", "A.Bt", "At.B"])
@pytest.mark.parametrize("tile", [3, 4])
@pytest.mark.parametrize("M,N,K", [(132, 136, 36), (256, 264, 500), (260, 120, 2052)])
def test_fp32_products_from_bf16_parts_keep_the_bits_of_small_numbers(ta, tb, M, N, K, tile):
    """Below 2^-110 three bf16 parts hold fewer than 24 bits.  Sums that consist of such numbers alone are taken on the fp32 instruction: its
    error is a few 2^-24 of the terms and their partial sums; sums that normal numbers decide keep their bits."""
    dp.dipaco_k_set_gemm_tile(tile)
    try:
        A, Ar = _rand((K, M) if ta else (M, K), 31, dp.F32)
        B, Br = _rand((N, K) if tb else (K, N), 32, dp.F32)
        Br = Br.T if tb else Br
        C = torch.empty((M, N), dtype=torch.float32, device=DEV)
        run = lambda: dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, A, B, C)
        run()
        ref = (Ar.T if ta else Ar) @ Br
        before = host(C).copy()
        bound = 2.0 ** -24 * (4 + math.sqrt(K))
        row = lambda m: A[:, m] if ta else A[m]
        row(1).mul_(2.0 ** -120)
        row(2).zero_()
        row(3)[::2] = 0.0                        # zeros lack nothing
        run()
        got = host(C)
        assert rel_l2(got[1] * 2.0 ** 120, ref[1]) <= bound
        assert not got[2].any()
        assert np.array_equal(got[4:], before[4:]) and np.array_equal(got[0], before[0])
        A.copy_(torch.from_numpy((Ar * 2.0 ** -120).astype(np.float32)))
        B.mul_(2.0 ** 100)
        run()
        assert rel_l2(host(C) * 2.0 ** 20, ref) <= bound
        if ta:                                   # cut over K, ragged at the end
            C.zero_()
            dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, A, B, C, splits=3, partial=torch.empty((3, M, N), device=DEV))
            assert rel_l2(host(C) * 2.0 ** 20, ref) <= bound
            A[K - 1, 5] = math.inf
            dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, A, B, C, splits=3, partial=torch.empty((3, M, N), device=DEV))
            got = host(C)
            assert np.array_equal(got[5], np.where(Br[K - 1] > 0, np.inf, -np.inf).astype(np.float32))
            assert rel_l2(np.delete(got, 5, 0) * 2.0 ** 20, np.delete(ref, 5, 0)) <= bound
    finally:
        dp.dipaco_k_set_gemm_tile(0)


@pytest.mark.parametrize("M,N,K,ta,tb,tile", [
    (4036, 512, 264, False, False, 2), (4036, 512, 264, False, True, 2), (1920, 512, 264, True, False, 2), (768, 2048, 520, False, True, 2),
    (2564, 2056, 136, False, False, 2), (1476, 2048, 896, False, True, 2), (9540, 512, 136, True, False, 2), (5756, 1024, 264, False, True, 2),
    (4000, 512, 2048, False, False, 3), (768, 2048, 1024, True, False, 3), (4000, 8192, 512, False, True, 4), (4096, 2048, 1024, True, False, 4)])
def test_fp32_products_take_parts_only_where_they_are_ahead(M, N, K, ta, tb, tile):
    """64 x 128 tiles of the fp32 instruction (2) against 64 x 128 (3) and 128 x 128 (4) in bf16 parts, told by their bits: sizes where one of
    them measured at least 5 % ahead of the others."""
    A, B = torch.randn((K, M) if ta else (M, K), device=DEV), torch.randn((N, K) if tb else (K, N), device=DEV)
    C = {t: torch.empty((M, N), device=DEV) for t in (0, 2, 3, 4)}
    try:
        for t in C:
            dp.dipaco_k_set_gemm_tile(t)
            dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, A, B, C[t])
    finally:
        dp.dipaco_k_set_gemm_tile(0)
    assert [t for t in (2, 3, 4) if torch.equal(C[0], C[t])] == [tile]


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)], ids=["A.B", "A.Bt", "At.B"])
def test_fp32_products_of_mixed_magnitudes_err_no_more_in_bf16_parts(ta, tb):
    """Rows from 2^-130 to 2^60, and single numbers from 2^-125 to 2^-100: element by element, in units of the absolute products, against
    the tile of the fp32 instruction."""
    M, N, K = 520, 264, 1160
    g = torch.Generator().manual_seed(3)
    a, b = torch.randn((M, K), generator=g), torch.randn((K, N), generator=g)
    for scale, col in ((torch.randint(-130, 60, (M, 1), generator=g), 1.0), (torch.randint(-125, -100, (M, K), generator=g), 2.0 ** 40)):
        A, B = a * torch.exp2(scale.float()), b * col
        ref, mag = A.double() @ B.double(), A.double().abs() @ B.double().abs()
        A, B = (A.t() if ta else A).contiguous().to(DEV), (B.t() if tb else B).contiguous().to(DEV)
        seen = mag > 2.0 ** -120                 # below, the sums themselves are subnormal
        errors = []
        try:
            for tile in (2, 3, 4):
                dp.dipaco_k_set_gemm_tile(tile)
                C = torch.empty((M, N), device=DEV)
                dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, A, B, C)
                errors.append((((C.cpu().double() - ref).abs() / mag)[seen]).max().item())
        finally:
            dp.dipaco_k_set_gemm_tile(0)
        print("largest error, 2^-24 of the absolute products:", [round(e * 2 ** 24, 2) for e in errors], flush=True)
        assert max(errors[1:]) <= 1.05 * errors[0]


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)], ids=["A.B", "A.Bt", "At.B"])
@pytest.mark.parametrize("M,N,K", [(256, 192, 128), (520, 264, 112), (248, 200, 100), (200, 200, 80)])
def test_fp32_products_over_a_short_k_err_no_more_than_chains_of_sixteen(M, N, K, ta, tb):
    """Every 16 of K are a chain of their own; chains 64 apart are added first, then the four such sums.  The root mean square of the errors is
    that of the same sums taken here (over tens of thousands of elements it is known to about 0.5 %); one chain over both steps errs by more."""
    g = torch.Generator().manual_seed(K)
    a, b = torch.randn((M, K), generator=g), torch.randn((K, N), generator=g)
    ref = a.double() @ b.double()
    sums = np.zeros((4, M, N), np.float32)
    for k0 in range(0, K, 16):
        chain = np.zeros((M, N), np.float32)
        for k in range(k0, min(k0 + 16, K)):
            chain = fma32(a[:, k:k + 1].numpy(), b[k].numpy(), chain)
        sums[k0 // 16 % 4] += chain
    model = ((sums[0] + sums[1]) + sums[2]) + sums[3]
    A, B = (a.t() if ta else a).contiguous().to(DEV), (b.t() if tb else b).contiguous().to(DEV)
    C = torch.empty((M, N), device=DEV)
    dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, A, B, C)
    mine, theirs = ((x.double() - ref).square().mean().sqrt().item() for x in (C.cpu(), torch.from_numpy(model)))
    print(f"rms error {mine:.3e}, of chains of sixteen {theirs:.3e}", flush=True)
    assert mine <= 1.03 * theirs


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)], ids=["A.B", "A.Bt", "At.B"])
@pytest.mark.parametrize("M,N,K", [(256, 192, 256), (40, 72, 132), (264, 120, 200), (8, 8, 144), (512, 504, 248), (360, 104, 136)])
def test_fp32_products_of_few_tiles_over_up_to_256_are_chains_of_sixteen(M, N, K, ta, tb):
    """Eight waves of two chains of sixteen K each, 128 apart: sixteen roundings of the largest partial sum in a chain, and eight of what is
    added behind them, on every element; and an element of the result that is not finite stays alone with its row or column."""
    g = torch.Generator().manual_seed(K)
    a, b = torch.randn((M, K), generator=g), torch.randn((K, N), generator=g)
    ref, most = a.double() @ b.double(), a.double().abs() @ b.double().abs()
    C = torch.empty((M, N), device=DEV)
    dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, (a.t() if ta else a).contiguous().to(DEV), (b.t() if tb else b).contiguous().to(DEV), C)
    assert bool(((C.cpu().double() - ref).abs() <= 24 * 2.0 ** -24 * most).all())
    assert (C.cpu().double() - ref).norm() <= 2e-7 * ref.norm()   # 1.2e-7 in chains of sixteen
    a[M // 2, K - 1], b[K - 4, N - 1] = math.inf, math.nan
    dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, (a.t() if ta else a).contiguous().to(DEV), (b.t() if tb else b).contiguous().to(DEV), C)
    off = ~torch.isfinite(C.cpu())
    assert bool(off[M // 2].all()) and bool(off[:, N - 1].all()) and int(off.sum()) == M + N - 1


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)], ids=["A.B", "A.Bt", "At.B"])
@pytest.mark.parametrize("tile", [3, 4])
def test_fp32_products_from_bf16_parts_with_one_large_value_in_a_tile(ta, tb, tile):
    """An infinity, or a number whose first part is one, anywhere in an operand: each in a call of its own, so that the sums it reaches
    lie with a few lanes of a wave."""
    M, N, K = 256, 264, 160
    A0, Ar = _rand((K, M) if ta else (M, K), 41, dp.F32)
    B0, Br = _rand((N, K) if tb else (K, N), 42, dp.F32)
    Ar, Br = Ar.T if ta else Ar, Br.T if tb else Br
    plain = Ar @ Br
    C = torch.empty((M, N), dtype=torch.float32, device=DEV)
    dp.dipaco_k_set_gemm_tile(tile)
    try:
        for value in (math.inf, -math.inf, 3.4e38):
            for side, at in (("A", 5), ("A", 31), ("A", 78), ("A", 128 + 63), ("A", 255), ("B", 7), ("B", 61), ("B", 128 + 90), ("B", 263)):
                A, B = A0.clone(), B0.clone()
                k = (3 * at) % K
                x = (A if ta else A.T) if side == "A" else (B.T if tb else B)   # [K, M or N]
                x[k, at] = value
                dp.dipaco_k_gemm(dp.F32, ta, tb, ta, M, N, K, A, B, C)
                got, want = host(C).astype(np.float64), plain.copy()
                with np.errstate(over="ignore", invalid="ignore"):
                    if side == "A":
                        want[at] = (Ar[at] @ Br - Ar[at, k] * Br[k] + np.float64(np.float32(value)) * Br[k]).astype(np.float32)
                    else:
                        want[:, at] = (Ar @ Br[:, at] - Br[k, at] * Ar[:, k] + np.float64(np.float32(value)) * Ar[:, k]).astype(np.float32)
                assert np.array_equal(np.isfinite(got), np.isfinite(want)) and np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
                fin = np.isfinite(want)
                assert (np.abs(got[fin] - want[fin]) <= 1e-5 * np.maximum(np.abs(want[fin]), math.sqrt(K))).all(), (value, side, at)
    finally:
        dp.dipaco_k_set_gemm_tile(0)


@pytest.mark.parametrize("tile", [3, 4])
def test_fp32_products_of_values_that_are_not_finite_take_no_second_walk_per_sum(tile):
    """NaN operands: their sums are NaN already.  Numbers below 2^-110 that no sum depends on: they are.  Infinities: the tiles they reach
    are multiplied once more."""
    M, N, K = 2048, 2048, 2048
    A, B = torch.randn((M, K), device=DEV), torch.randn((K, N), device=DEV)
    C = torch.empty((M, N), device=DEV)
    dp.dipaco_k_set_gemm_tile(tile)
    try:
        run = lambda: dp.dipaco_k_gemm(dp.F32, False, False, False, M, N, K, A, B, C)
        finite = median_us(run)
        A[5, 7] = math.nan
        B[:, 11] = math.nan
        run()
        nan = torch.isnan(C)
        assert bool(nan[5].all()) and bool(nan[:, 11].all()) and int(nan.sum()) == M + N - 1
        A[:, 9] = math.nan
        times = [median_us(run)]
        assert bool(torch.isnan(C).all())
        A[:, 7:10], B[:, 11] = 1.0, 1.0
        A[:, 9] = 2.0 ** -120
        times.append(median_us(run))
        A[:, 9], B[:, 11] = math.inf, math.nan
        times.append(median_us(run))
        C[:, 11] = 0.0
        assert bool(torch.isinf(C).sum() == M * (N - 1))
        print(f"tile {tile}: us finite {finite:.0f} NaN {times[0]:.0f} small {times[1]:.0f} infinite {times[2]:.0f}", flush=True)
        assert max(times[:2]) <= 3 * finite and times[2] <= 10 * finite   # a walk for each sum: a hundred times and more
    finally:
        dp.dipaco_k_set_gemm_tile(0)


@pytest.mark.parametrize("B,S,H,dh", [(260, 33, 2, 32), (260, 33, 2, 64), (260, 100, 2, 128), (60, 300, 3, 32), (171, 129, 2, 64)])
def test_fp32_attention_above_512_blocks(B, S, H, dh):
    """More than 512 blocks of 128 rows run eight waves a workgroup, forward and backward."""
    assert B * H * -(-S // 128) > 512
    test_attention_forward_backward(dp.F32, B, S, H, dh, 1)


@pytest.mark.parametrize("B,S,H,dh", [(5, 257, 17, 32), (2, 300, 43, 64), (1, 385, 3, 128), (4, 200, 3, 64), (3, 129, 2, 32), (32, 128, 9, 64), (4, 512, 16, 64),
                                      (3, 600, 17, 128), (65, 513, 10, 32), (40, 641, 9, 32), (30, 1025, 5, 64)])
def test_bf16_attention_gradients_in_one_launch_and_in_two(B, S, H, dh):
    """One block of 128 positions to five; 255, 256 and 258 blocks, on the two sides of two groups a block; two launches for 3250 blocks, and
    for 2160 and 1350 of sequences of six and nine with narrow heads."""
    print(f"{B * H * -(-S // 128)} blocks", flush=True)
    test_attention_forward_backward(dp.BF16, B, S, H, dh, 1)


@pytest.mark.parametrize("B,S,H,dh", [(16, 130, 5, 64), (43, 100, 3, 32), (16, 200, 8, 32), (19, 330, 3, 64), (24, 450, 4, 64), (8, 257, 17, 32), (64, 200, 4, 32), (8, 320, 13, 128)])
def test_fp32_attention_of_blocks_that_are_resident_at_once(B, S, H, dh):
    """240 to 1024 workgroups of 64 positions: one round of the compute units, one more than one, two, a ragged third, four; each block is taken
    once, whatever its place."""
    blocks = B * H * -(-S // 64)
    print(f"{blocks} workgroups", flush=True)
    assert B * H * -(-S // 128) <= 512 and 240 <= blocks <= 1024
    test_attention_forward_backward(dp.F32, B, S, H, dh, 1)


@pytest.mark.parametrize("B,S,H,dh", [(3, 32, 3, 64), (5, 17, 1, 64), (2, 32, 3, 128), (1, 5, 1, 128), (5, 32, 1, 32), (1, 33, 1, 64)])
def test_attention_of_short_sequences(B, S, H, dh):
    """Up to 32 positions a wave owns a sequence and head: full and ragged workgroups of four, every head size; 33 is the first
    length of the tiled kernel."""
    test_attention_forward_backward(dp.BF16, B, S, H, dh, 1)


@pytest.mark.parametrize("dtype,trans_a,trans_b,M,N,K", [
    (dp.F32, False, False, 64, 8, 40_000_000),     # A: 31 rows of a 32-row tile are 4.96e9 bytes apart
    (dp.F32, False, True, 8, 64, 40_000_000),      # B^T: 63 rows of 160 MB
    (dp.BF16, True, False, 40_000_000, 8, 64),     # A: 63 K-rows of 80 MB
    (dp.F32, True, False, 8, 9_000_000, 304),      # B: 127 K-rows of 36 MB
])
def test_gemm_operand_tiles_that_span_more_than_4_gib(dtype, trans_a, trans_b, M, N, K):
    """Accepted sizes (fewer than 2^32 elements an operand, or 64 K-rows of it) whose byte offsets inside one tile pass 2^32.
    Operands of small whole numbers, zero but for a few K (or a few rows of the long side): every product is exact."""
    print(f"gemm far dtype={dtype} ta={trans_a} tb={trans_b} M={M} N={N} K={K}", flush=True)
    g = torch.Generator().manual_seed(5)
    A = torch.zeros((K, M) if trans_a else (M, K), dtype=TDT[dtype], device=DEV)
    B = torch.zeros((N, K) if trans_b else (K, N), dtype=TDT[dtype], device=DEV)
    pick = lambda n: torch.tensor(sorted({0, 1, n // 3, n // 2 + 1, n - 2, n - 1}) if n > 4096 else list(range(n)))
    km, kn, kk = pick(M), pick(N), pick(K)
    a = torch.randint(-3, 4, (len(km), len(kk)), generator=g).double()
    b = torch.randint(-3, 4, (len(kk), len(kn)), generator=g).double()
    put = lambda t, r, c, v: t.__setitem__((r.to(DEV)[:, None], c.to(DEV)[None, :]), v.to(TDT[dtype]).to(DEV))
    put(A, *((kk, km, a.T) if trans_a else (km, kk, a)))
    put(B, *((kn, kk, b.T) if trans_b else (kk, kn, b)))
    C = torch.full((M, N), float("nan"), dtype=torch.float32 if trans_a else TDT[dtype], device=DEV)
    dp.dipaco_k_gemm(dtype, trans_a, trans_b, trans_a, M, N, K, A, B, C)
    got = C[km.to(DEV)][:, kn.to(DEV)].double().cpu()
    assert torch.equal(got, a @ b)
    assert float(C.double().abs().sum()) == float((a @ b).abs().sum())   # and zero everywhere else


@pytest.mark.parametrize("dh", [32, 128])
@pytest.mark.parametrize("B,S,H", [(4, 17, 4), (3, 32, 4), (3, 33, 4), (2, 200, 3), (1, 1000, 2)])
def test_bf16_attention_is_as_exact_as_its_outputs_are_rounded(B, S, H, dh):
    """Head sizes 32 and 128 carry probabilities and dS with at least 16 bits into their products and sum rows in fp32: all that is
    left of the error is the rounding of the bf16 outputs, plus 2 % for operands (2^-17 against 2^-9) and single roundings that
    fall the other way; lse is fp32: 2^-24 of |lse| + |score| < 40 in a few roundings."""
    print(f"attention exact B={B} S={S} H={H} dh={dh}", flush=True)
    A, scale = H * dh, 1.0 / math.sqrt(dh)
    qkv, x = _rand((B * S, 3 * A), 31, dp.BF16)
    d_o, g = _rand((B * S, A), 32, dp.BF16)
    o, dqkv = torch.empty_like(d_o), torch.empty_like(qkv)
    lse = torch.empty((B, H, S), device=DEV)
    dp.dipaco_k_attention_fwd(dp.BF16, qkv, o, lse, B, S, H, dh)
    dsum = torch.empty(2 * B * H * ((S + 127) // 128 * 128), device=DEV)
    dp.dipaco_k_attention_bwd(dp.BF16, qkv, o, d_o, lse, dqkv, dsum, B, S, H, dh)
    q, k, v = np.moveaxis(x.reshape(B, S, 3, H, dh), (2, 3), (0, 2))            # [B, H, S, dh] each
    g, stored = (np.moveaxis(t.reshape(B, S, H, dh), 1, 2) for t in (g, host(o).astype(np.float64)))
    s = np.where(np.tril(np.ones((S, S), bool)), q @ np.swapaxes(k, -1, -2) * scale, -np.inf)
    top = s.max(-1, keepdims=True)
    L = top + np.log(np.exp(s - top).sum(-1, keepdims=True))
    P = np.exp(s - L)
    dS = P * (g @ np.swapaxes(v, -1, -2) - (stored * g).sum(-1, keepdims=True))
    got = np.moveaxis(host(dqkv).astype(np.float64).reshape(B, S, 3, H, dh), (2, 3), (0, 2))
    want = {"o": P @ v, "dq": dS @ k * scale, "dk": np.swapaxes(dS, -1, -2) @ q * scale, "dv": np.swapaxes(P, -1, -2) @ g}
    for name, have in zip(want, (stored, *got)):
        rounded = torch.from_numpy(want[name]).to(torch.bfloat16).double().numpy()
        assert rel_l2(have, want[name]) <= 1.02 * rel_l2(rounded, want[name]), name
    assert np.abs(host(lse) - L[..., 0]).max() <= 1e-5


def _attention_over_visible_pairs(q, k, v, g, o, scale):
    """One head in fp64, every sum over the pairs (query i, key j <= i) alone; o: the stored output, for D."""
    S, n = len(q), q.shape[1]
    lse, out, dq, dk, dv = np.zeros(S), np.zeros((S, n)), np.zeros((S, n)), np.zeros((S, n)), np.zeros((S, n))
    with np.errstate(all="ignore"):
        for i in range(S):
            s = k[:i + 1] @ q[i] * scale
            top = s.max()
            lse[i] = top + np.log(np.exp(s - top).sum())
            p = np.exp(s - lse[i])
            ds = p * (v[:i + 1] @ g[i] - o[i] @ g[i])
            out[i], dq[i] = p @ v[:i + 1], ds @ k[:i + 1] * scale
            dv[:i + 1] += p[:, None] * g[i]
            dk[:i + 1] += ds[:, None] * q[i] * scale
    return lse, out, dq, dk, dv


@pytest.mark.parametrize("dtype,dh", [(dp.F32, 32), (dp.F32, 64), (dp.F32, 128), (dp.BF16, 32), (dp.BF16, 128)])
@pytest.mark.parametrize("B,S,H,at", [(2, 9, 2, 4), (2, 100, 2, 70), (1, 100, 2, 99), (1, 300, 1, 131), (260, 130, 2, 129)])
@pytest.mark.parametrize("where,value", [("q", math.nan), ("k", math.nan), ("v", math.nan), ("v", math.inf), ("d_o", math.nan),
                                         ("d_o", -math.inf)])
def test_attention_keeps_non_finite_values_from_rows_that_do_not_see_them(dtype, dh, B, S, H, at, where, value):
    """One non-finite row: what is finite over the visible pairs is finite and right, what is not is not.  S - 1 is the row that
    rows past the end re-read; 260 x 2 heads of 130 positions run eight waves a workgroup in fp32."""
    print(f"attention non-finite dtype={dtype} dh={dh} B={B} S={S} H={H} {where}[{at}]={value}", flush=True)
    A = H * dh
    qkv, _ = _rand((B * S, 3 * A), 41, dtype)
    d_o, _ = _rand((B * S, A), 42, dtype)
    third = {"q": 0, "k": 1, "v": 2}
    if where == "d_o":
        d_o[at, :dh] = value
    else:
        qkv[at, third[where] * A:third[where] * A + dh] = value
    o, dqkv = torch.full_like(d_o, 7.0), torch.full_like(qkv, 7.0)
    lse = torch.empty((B, H, S), device=DEV)
    dp.dipaco_k_attention_fwd(dtype, qkv, o, lse, B, S, H, dh)
    dsum = torch.empty(2 * B * H * ((S + 127) // 128 * 128), device=DEV)
    dp.dipaco_k_attention_bwd(dtype, qkv, o, d_o, lse, dqkv, dsum, B, S, H, dh)
    head = lambda t, n: host(t[:S]).astype(np.float64)[:, n * A:n * A + dh]
    q, k, v = (head(qkv, n) for n in range(3))
    want = _attention_over_visible_pairs(q, k, v, head(d_o, 0), head(o, 0), 1.0 / math.sqrt(dh))
    have = (host(lse)[0, 0].astype(np.float64), head(o, 0), *(head(dqkv, n) for n in range(3)))
    tol = 2e-5 if dtype == dp.F32 else 6e-3
    for name, a, b in zip(("lse", "o", "dq", "dk", "dv"), have, want):
        ok = np.isfinite(b)
        assert np.array_equal(np.isfinite(a), ok), name
        assert rel_l2(a[ok], b[ok]) <= tol, name
    if B * H > 1:   # other heads and sequences
        assert bool(torch.isfinite(o[:, dh:]).all()) and bool(torch.isfinite(dqkv.view(B * S, 3, A)[:, :, dh:]).all())
        assert bool(torch.isfinite(o[S:]).all()) and bool(torch.isfinite(dqkv[S:]).all()) and bool(torch.isfinite(lse[1:]).all())


@pytest.mark.parametrize("dtype,S,B,H,dh", [(dp.F32, 1, 3_000_000, 3, 32), (dp.F32, 2, 9_000_000, 1, 32), (dp.BF16, 1, 17_000_000, 1, 32)])
def test_attention_of_more_heads_than_one_launch_holds(dtype, S, B, H, dh):
    """Sequences x heads x threads of a workgroup reach 2^32.  One position: o = v, dv = d_o and their column sums (dS = p (dO.v - dO.o)
    is a rounding difference of the two); two: the second row of the last sequence too."""
    print(f"attention many dtype={dtype} S={S} B={B} H={H} dh={dh}", flush=True)
    A, T = H * dh, B * S
    qkv, d_o = (torch.randn((T, w), dtype=TDT[dtype], device=DEV, generator=torch.Generator(DEV).manual_seed(w)) for w in (3 * A, A))
    o, dqkv = torch.full_like(d_o, 7.0), torch.full_like(qkv, 7.0)
    lse = torch.full((B, H, S), float("nan"), device=DEV)
    dp.dipaco_k_attention_fwd(dtype, qkv, o, lse, B, S, H, dh)
    first = torch.arange(0, T, S, device=DEV) if S > 1 else slice(None)
    assert torch.equal(o[first], qkv[first, 2 * A:]) and bool(torch.isfinite(o).all()) and bool(torch.isfinite(lse).all())
    dsum, cs = torch.empty(2 * B * H * 128, device=DEV), torch.zeros(3 * A, device=DEV)
    scratch = torch.full((B * 3 * A,), float("nan"), device=DEV)
    dp.dipaco_k_attention_bwd(dtype, qkv, o, d_o, lse, dqkv, dsum, B, S, H, dh, colsum_out=cs, colsum_scratch=scratch)
    assert bool(torch.isfinite(dqkv).all())
    want = dqkv[:, 2 * A:].double().sum(0)
    # stored bf16 values against the sums of the unrounded ones: 2^-9 of sqrt(T) values of about one each
    assert float((cs[2 * A:].double() - want).abs().max()) <= (2e-3 if dtype == dp.F32 else 2.0 ** -8) * math.sqrt(T)
    if S == 1:
        # p = exp(score - lse) = 1 within 2^-24 of |score| < 12, times |d_o| < 7; in bf16 rounding gives d_o back
        assert float((dqkv[:, 2 * A:] - d_o).abs().max()) <= (1e-5 if dtype == dp.F32 else 0.0)
    else:
        q, k, v = (t.double() for t in qkv[-2:].split(A, 1))
        w = torch.softmax(q[1] @ k.T / math.sqrt(dh), 0)
        assert rel_l2(host(o[-1]), (w @ v).cpu().numpy()) <= 1e-5
        assert rel_l2(host(dqkv[-1, 2 * A:]), (w[1] * d_o[-1].double()).cpu().numpy()) <= 1e-5
