"""GPU parity of the single operations (the kernels one by one) against the oracle's primitives,
at shapes that span several tiles plus ragged tails, through the C ABI."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import stage_oracle as O
from tests import harness as hz

pytestmark = pytest.mark.gpu


def _randn(role, shape, std=1.0, seed=0, dtype="bf16"):
    return si.round_to(si.normal(si.stream_key(seed, role, *shape), shape, std), dtype)


def _f32_dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


GEMM_SHAPES = [
    # (M, N, K)
    (256, 256, 128),       # one 256 tile / 4 tiles of 128
    (512, 768, 320),       # several tiles, K = 5 slices
    (2048, 2048, 512),     # 64 tiles of 256 -> 128 path; 256 tiles of 128
    (1024, 12288, 256),    # 192 tiles of 256
    (200, 264, 136),       # ragged everywhere (multiples of 8)
    (130, 72, 64),         # smaller than a tile
]


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
@pytest.mark.parametrize("form", ["fwd", "dgrad", "wgrad"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_gemm_forms(M, N, K, form, dtype):
    import torch
    import paper_2410_19367_amd as bp
    if dtype == "f32" and M * N * K > 512 * 768 * 320:
        pytest.skip("fp32 path is exercised on the small shapes")
    dt = bp.BP_BF16 if dtype == "bf16" else bp.BP_F32
    tol = hz.TOL[dtype] if dtype == "f32" else 1e-2
    if form == "fwd":            # Y[M,N] = X[M,K] W[K,N] + b + R
        X = _randn("gx", (M, K), dtype=dtype); W = _randn("gw", (K, N), 0.05, dtype=dtype)
        b = _randn("gb", (N,), 0.5, dtype="f32"); R = _randn("gr", (M, N), dtype=dtype)
        ref = O.linear_fwd(X.astype(np.float64), W.astype(np.float64), b.astype(np.float64), R.astype(np.float64))
        out = hz.empty_like_dev((M, N), dtype)
        bp.bp_op_gemm(dt, 0, 0, M, N, K, hz.to_dev(X, dtype), K, hz.to_dev(W, dtype), N, out, N,
                      bias=_f32_dev(b), residual=hz.to_dev(R, dtype))
        got = hz.to_host(out)
    elif form == "dgrad":        # dX[M,N] = dY[M,K] W[N,K]^T
        dY = _randn("gdy", (M, K), dtype=dtype); W = _randn("gw2", (N, K), 0.05, dtype=dtype)
        ref = O.linear_dgrad(dY.astype(np.float64), W.astype(np.float64))
        out = hz.empty_like_dev((M, N), dtype)
        bp.bp_op_gemm(dt, 0, 1, M, N, K, hz.to_dev(dY, dtype), K, hz.to_dev(W, dtype), K, out, N)
        got = hz.to_host(out)
    else:                        # dW[M,N] += X[K,M]^T dY[K,N]   (K = tokens)
        X = _randn("gx3", (K, M), dtype=dtype); dY = _randn("gdy3", (K, N), dtype=dtype)
        C0 = _randn("gc0", (M, N), 3.0, dtype="f32")
        dW, _ = O.linear_wgrad(X.astype(np.float64), dY.astype(np.float64))
        ref = C0.astype(np.float64) + dW
        out = _f32_dev(C0)
        bp.bp_op_gemm(dt, 1, 0, M, N, K, hz.to_dev(X, dtype), M, hz.to_dev(dY, dtype), N, out, N, accumulate=1)
        got = hz.to_host(out)
    torch.cuda.synchronize()
    err = hz.rel_err(got, ref)
    assert err <= tol, (form, M, N, K, err)


# Edge tiles of the direct-to-LDS kernel: one row / column / chunk, one past a tile, K (a token count in
# the weight-gradient form) that is no multiple of anything, each tile shape.  Tolerances as above: the
# same products with the same roundings.
@pytest.mark.parametrize("form,M,N,K", [
    ("dgrad", 1, 8, 8), ("dgrad", 129, 136, 72), ("dgrad", 255, 264, 200), ("dgrad", 1000, 9600, 72),
    ("dgrad", 4000, 3200, 136), ("fwd", 257, 136, 72), ("fwd", 1, 264, 64),
    ("wgrad", 8, 8, 1), ("wgrad", 136, 264, 77), ("wgrad", 520, 136, 333), ("wgrad", 4000, 3200, 97),
    ("wgrad", 1000, 9600, 65), ("wgrad", 264, 520, 1999),
])
def test_gemm_edge_tiles(form, M, N, K):
    test_gemm_forms(M, N, K, form, "bf16")


# Large forward-form tiles (256 x 256 and 256 x 192 wide), whose operands are requested half a slice apart
# into three and two LDS stages: fewer slices than stages, every phase of the 3 x 2 stage cycle at the end.
@pytest.mark.parametrize("M,N,K", [
    (1024, 12288, 64), (1024, 12288, 128), (1024, 12288, 192), (1024, 12288, 256), (1024, 12288, 448),
    (2048, 6144, 64), (2048, 6144, 320), (2048, 6144, 384), (4000, 3200, 8), (4000, 3200, 264), (1000, 9600, 328),
])
def test_gemm_large_tiles_few_slices(M, N, K):
    test_gemm_forms(M, N, K, "dgrad", "bf16")


# Small outputs: 64 x 64 tiles (slices of 128 along K), 128 x 64 and 128 x 128 tiles (slices of 64), each with one
# slice, fewer slices than LDS stages, and one more; the limits between the tiles; edges of 64.
@pytest.mark.parametrize("form,M,N,K", [
    ("dgrad", 384, 256, 128), ("dgrad", 384, 256, 256), ("dgrad", 384, 768, 384), ("dgrad", 1024, 1024, 512),
    ("dgrad", 1024, 1088, 64), ("dgrad", 1024, 2048, 128), ("dgrad", 1024, 2048, 192), ("dgrad", 1024, 2112, 128),
    ("dgrad", 1000, 4800, 136), ("dgrad", 63, 72, 136), ("dgrad", 65, 136, 264), ("dgrad", 1001, 1608, 72),
    ("wgrad", 256, 192, 384), ("wgrad", 72, 328, 129), ("wgrad", 1024, 1024, 250),
])
def test_gemm_small_tiles(form, M, N, K):
    test_gemm_forms(M, N, K, form, "bf16")


# 128 x 128 tiles of the forward form with two blocks per CU (more than 256 tiles on 256 CUs) and, at the limit, one: fewer
# slices than LDS stages, every phase of the 3 x 2 stage cycle at the end, edge tiles and K tails
@pytest.mark.parametrize("form,M,N,K", [
    ("dgrad", 2176, 2048, 64), ("dgrad", 2176, 2048, 128), ("dgrad", 2176, 2048, 192), ("dgrad", 2176, 2048, 448), ("dgrad", 2048, 2048, 128),
    ("dgrad", 2048, 4096, 320), ("dgrad", 2050, 4096, 72), ("dgrad", 1998, 2304, 8), ("dgrad", 1998, 2304, 200), ("dgrad", 1000, 4808, 264),
    ("fwd", 1998, 2304, 136),
])
def test_gemm_two_blocks_per_cu(form, M, N, K):
    test_gemm_forms(M, N, K, form, "bf16")


# fp32 kernel: both tile widths, one element past a tile, the shortest K, K tails of four, unaligned rows
# (the generic kernel); 1e-5 relative to the largest element bounds fp32 sums of this length
@pytest.mark.parametrize("form,M,N,K", [
    ("dgrad", 33, 32, 4), ("dgrad", 1, 36, 68), ("dgrad", 65, 132, 200), ("dgrad", 1030, 1100, 72), ("fwd", 31, 100, 132),
    ("fwd", 1030, 1100, 36), ("wgrad", 4, 4, 1), ("wgrad", 36, 132, 77), ("wgrad", 1028, 1100, 65), ("fwd", 50, 37, 64),
])
def test_gemm_f32_edge_tiles(form, M, N, K):
    test_gemm_forms(M, N, K, form, "f32")


@pytest.mark.parametrize("T,H", [(64, 128), (300, 1024), (260, 2048), (77, 5120), (33, 8192), (5, 8)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_layernorm_fwd_bwd(T, H, dtype):
    import torch
    import paper_2410_19367_amd as bp
    dt = bp.BP_BF16 if dtype == "bf16" else bp.BP_F32
    x = _randn("lx", (T, H), 2.0, dtype=dtype) + np.float32(0.5)
    x = si.round_to(x, dtype)
    g = _randn("lg", (H,), 0.3, dtype="f32") + 1.0
    b = _randn("lb", (H,), 0.3, dtype="f32")
    dout = _randn("ld", (T, H), dtype=dtype)
    res = _randn("lr", (T, H), dtype=dtype)
    eps = 1e-5
    x64 = x.astype(np.float64)
    ref, xhat, rstd = O.layer_norm_fwd(x64, g.astype(np.float64), b.astype(np.float64), eps)
    dx_ref, dg_ref, db_ref = O.layer_norm_bwd(dout.astype(np.float64), xhat, rstd, g.astype(np.float64))
    dx_ref = dx_ref + res
    xd, gd, bd = hz.to_dev(x, dtype), _f32_dev(g), _f32_dev(b)
    out = hz.empty_like_dev((T, H), dtype)
    mean = torch.empty(T, device="cuda"); rs = torch.empty(T, device="cuda")
    bp.bp_op_layernorm_fwd(dt, T, H, xd, gd, bd, eps, out, mean, rs)
    dx = hz.empty_like_dev((T, H), dtype)
    dg0 = _randn("ldg0", (H,), dtype="f32"); db0 = _randn("ldb0", (H,), dtype="f32")
    dgd, dbd = _f32_dev(dg0), _f32_dev(db0)
    ws = torch.empty(2 * bp.bp_op_colsum_workspace(T, H), device="cuda")
    bp.bp_op_layernorm_bwd(dt, T, H, hz.to_dev(dout, dtype), xd, mean, rs, gd, hz.to_dev(res, dtype),
                           dx, dgd, dbd, ws)
    torch.cuda.synchronize()
    tol = 1e-2 if dtype == "bf16" else 1e-5
    assert hz.rel_err(hz.to_host(out), ref) <= tol
    assert hz.rel_err(hz.to_host(mean), x64.mean(-1)) <= 1e-5
    assert hz.rel_err(hz.to_host(rs), rstd[:, 0]) <= 1e-5
    assert hz.rel_err(hz.to_host(dx), dx_ref) <= tol
    assert hz.rel_err(hz.to_host(dgd), dg0 + dg_ref) <= 1e-4
    assert hz.rel_err(hz.to_host(dbd), db0 + db_ref) <= 1e-4


@pytest.mark.parametrize("T,F", [(64, 512), (300, 4096), (100, 8192), (37, 520)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_bias_gelu_fwd_bwd(T, F, dtype):
    import torch
    import paper_2410_19367_amd as bp
    dt = bp.BP_BF16 if dtype == "bf16" else bp.BP_F32
    u = _randn("gu", (T, F), 2.0, dtype=dtype)
    b = _randn("gbias", (F,), 0.5, dtype="f32")
    dg = _randn("gdg", (T, F), dtype=dtype)
    h = u.astype(np.float64) + b
    g_ref = O.gelu(h)
    du_ref = dg * O.gelu_grad(h)
    db0 = _randn("gdb0", (F,), dtype="f32")
    ud, bd = hz.to_dev(u, dtype), _f32_dev(b)
    g = hz.empty_like_dev((T, F), dtype)
    bp.bp_op_bias_gelu_fwd(dt, T, F, ud, bd, g)
    du = hz.empty_like_dev((T, F), dtype)
    dbd = _f32_dev(db0)
    ws = torch.empty(bp.bp_op_colsum_workspace(T, F), device="cuda")
    bp.bp_op_bias_gelu_bwd(dt, T, F, hz.to_dev(dg, dtype), ud, bd, du, dbd, ws)
    torch.cuda.synchronize()
    tol = 1e-2 if dtype == "bf16" else 1e-5
    assert hz.rel_err(hz.to_host(g), g_ref) <= tol
    assert hz.rel_err(hz.to_host(du), du_ref) <= tol
    assert hz.rel_err(hz.to_host(dbd), db0 + du_ref.sum(0)) <= (2e-3 if dtype == "bf16" else 1e-5)


# Column sums over 1, 8, 9 chunks of 32 rows and around the rounds of 64 chunks, the last chunk whole and cut
@pytest.mark.parametrize("T,N", [(1, 8), (256, 8), (257, 16), (1920, 8), (1953, 8), (2043, 16), (2048, 8), (2049, 72), (4127, 24), (13082, 8)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_column_sums_many_chunks(T, N, dtype):
    test_layernorm_fwd_bwd(T, N, dtype)
    test_bias_gelu_fwd_bwd(T, N, dtype)


ATTN_CASES = [
    # B, S, heads, d, causal, lens
    (2, 64, 2, 64, True, None),
    (1, 200, 2, 128, True, None),
    (2, 384, 3, 64, True, None),
    (1, 512, 2, 128, True, None),
    (3, 160, 2, 64, False, [160, 41, 97]),
    (2, 256, 2, 128, False, [256, 130]),
    (2, 96, 2, 64, False, None),
    (1, 72, 1, 32, True, None),
    (3, 128, 2, 64, False, [128, 41, 97]),
    (2, 256, 2, 64, False, None),
    (1, 640, 2, 128, False, [333]),
    (2, 1024, 1, 128, True, None),
    (2, 192, 2, 64, True, None),
    (1, 320, 3, 128, False, [200]),
    (2, 64, 2, 128, True, None),
    # head widths below the tile width (padded inside the MFMA kernels): the paper's 40 and 96, and others
    (2, 128, 4, 40, False, [128, 77]),
    (1, 256, 2, 96, True, None),
    (2, 192, 2, 40, True, None),
    (1, 128, 3, 96, False, [100]),
    (1, 192, 2, 32, True, None),
    (1, 128, 2, 112, False, None),
    (1, 128, 2, 48, True, None),
    (1, 64, 2, 8, True, None),
    # long enough for the eight-wave forward (two tiles per step), padded widths
    (1, 512, 2, 112, True, None),
    (1, 512, 2, 40, False, [300]),
    # the eight-wave forward with an odd number of 64-key tiles, so that the last step holds one tile only
    (1, 576, 2, 64, True, None),
    (1, 704, 1, 96, True, None),
    (1, 576, 2, 128, False, [500]),
]


@pytest.mark.parametrize("B,S,heads,d,causal,lens", ATTN_CASES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention_fwd_bwd(B, S, heads, d, causal, lens, dtype):
    import torch
    import paper_2410_19367_amd as bp
    dt = bp.BP_BF16 if dtype == "bf16" else bp.BP_F32
    H = heads * d
    qkv = _randn("aqkv", (B, S, 3 * H), 1.0, dtype=dtype)
    dctx = _randn("adctx", (B, S, H), dtype=dtype)
    q64 = qkv.astype(np.float64)
    q = O._split_heads(q64[..., :H], heads); k = O._split_heads(q64[..., H:2 * H], heads)
    v = O._split_heads(q64[..., 2 * H:], heads)
    la = None if lens is None else np.array(lens)
    ctx_h, p = O.attention_fwd(q, k, v, causal, la)
    ctx_ref = O._merge_heads(ctx_h)
    dq, dk, dv = O.attention_bwd(O._split_heads(dctx.astype(np.float64), heads), q, k, v, p)
    dqkv_ref = np.concatenate([O._merge_heads(dq), O._merge_heads(dk), O._merge_heads(dv)], -1)
    # log-sum-exp of the scaled, masked scores, from the definition
    lse_ref = np.empty((B, heads, S))
    for b in range(B):
        ok = O.allowed_mask(S, causal, None if la is None else la[b])
        for h in range(heads):
            s = np.where(ok, q[b, h] @ k[b, h].T / np.sqrt(d), -np.inf)
            mx = s.max(-1)
            lse_ref[b, h] = mx + np.log(np.exp(s - mx[:, None]).sum(-1))
    qd = hz.to_dev(qkv, dtype)
    ctx = hz.empty_like_dev((B, S, H), dtype)
    lse = torch.empty((B, heads, S), device="cuda")
    lens_d = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    bp.bp_op_attention_fwd(dt, B, S, heads, d, causal, lens_d, qd, ctx, lse)
    dqkv = hz.empty_like_dev((B, S, 3 * H), dtype)
    delta = torch.empty((B, heads, S), device="cuda")
    # the backward consumes the oracle's ctx (rounded to the storage type), not the GPU's
    ctx_in = hz.to_dev(si.round_to(ctx_ref, dtype), dtype)
    bp.bp_op_attention_bwd(dt, B, S, heads, d, causal, lens_d, qd, ctx_in, lse, hz.to_dev(dctx, dtype), dqkv, delta)
    torch.cuda.synchronize()
    tol = 1e-2 if dtype == "bf16" else 2e-5
    assert hz.rel_err(hz.to_host(ctx), ctx_ref) <= tol
    assert np.max(np.abs(hz.to_host(lse) - lse_ref)) <= (1e-4 if dtype == "f32" else 2e-3)
    got = hz.to_host(dqkv)
    for name, sl in (("dq", slice(0, H)), ("dk", slice(H, 2 * H)), ("dv", slice(2 * H, 3 * H))):
        err = hz.rel_err(got[..., sl], dqkv_ref[..., sl])
        assert err <= (2e-2 if dtype == "bf16" else 5e-5), (name, err)


# Sequence lengths around the 64-row tiles and the 32-row halves, one and two tiles per forward step
@pytest.mark.parametrize("B,S,heads,d,causal,lens", [
    (2, 2, 2, 64, True, None), (2, 31, 2, 64, True, None), (1, 33, 3, 128, True, None), (2, 63, 2, 40, True, None),
    (3, 65, 2, 64, False, [65, 1, 64]), (1, 97, 2, 96, False, [33]), (2, 127, 2, 128, True, None),
    (1, 513, 2, 64, True, None), (1, 545, 2, 128, False, [544]), (1, 1000, 1, 64, True, None), (2, 333, 2, 64, False, [100, 333]),
])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention_ragged_lengths(B, S, heads, d, causal, lens, dtype):
    test_attention_fwd_bwd(B, S, heads, d, causal, lens, dtype)


# Launches with enough blocks for those of 128 rows (on 256 CUs): an odd number of 64-row tiles, valid lengths around
# the halves of a tile and of a block, every head width with a kernel of its own and one without; causal blocks in the three
# orders that wide launches have: folded up to 512 of them, heaviest first of all batch entries together up to 1024, one entry
# after the other above; forward alone (256 blocks), forward and dQ alone (causal beyond S 512)
@pytest.mark.parametrize("B,S,heads,d,causal,lens", [
    (16, 192, 16, 64, True, None), (16, 192, 16, 64, False, [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 191, 192]),
    (16, 192, 16, 40, False, [192, 96, 33, 64] * 4), (16, 128, 32, 128, True, None), (16, 192, 16, 96, True, None),
    (16, 192, 16, 128, False, [160, 161, 128, 1] * 4), (16, 64, 64, 64, True, None), (16, 192, 16, 80, True, None),
    (5, 320, 48, 24, True, None), (4, 512, 16, 128, False, [512, 479, 480, 200]), (8, 576, 16, 96, True, None),
    (24, 320, 16, 64, True, None), (18, 192, 32, 40, True, None), (17, 256, 32, 128, True, None), (13, 320, 28, 96, True, None),
    (8, 192, 48, 64, True, None),
])
def test_attention_blocks_of_128_rows(B, S, heads, d, causal, lens):
    test_attention_fwd_bwd(B, S, heads, d, causal, lens, "bf16")


# Backward: both sides of the limits up to which dQ and dK/dV share a launch (on 256 CUs: 384, 512 causal, 768 ragged
# blocks of each up to head width 64, 256 of 96, 128 of other wide heads; fp32 256), and every head width on either side
@pytest.mark.parametrize("B,S,heads,d,causal,lens,dtype", [
    (6, 256, 16, 64, False, [1, 63, 64, 65, 200, 256], "bf16"), (5, 320, 16, 64, False, None, "bf16"), (4, 512, 16, 64, True, None, "bf16"),
    (5, 448, 16, 64, True, None, "bf16"), (6, 100, 64, 64, False, [1, 33, 64, 65, 99, 100], "bf16"), (7, 100, 64, 40, False, None, "bf16"),
    (6, 70, 64, 64, True, None, "bf16"), (7, 70, 64, 24, True, None, "bf16"), (2, 512, 16, 96, True, None, "bf16"), (2, 576, 16, 96, True, None, "bf16"),
    (2, 256, 16, 128, True, None, "bf16"), (2, 320, 16, 128, True, None, "bf16"), (2, 200, 16, 112, False, [200, 129], "bf16"), (3, 200, 16, 112, True, None, "bf16"),
    (2, 512, 16, 64, True, None, "f32"), (3, 400, 16, 64, False, [400, 1, 70], "f32"), (2, 512, 16, 24, True, None, "f32"), (3, 400, 16, 24, True, None, "f32"),
    (2, 200, 16, 96, True, None, "f32"), (3, 200, 16, 128, False, None, "f32"),
    # and between those and the kernels of one row per block
    (1, 32, 8, 64, True, None, "f32"), (1, 33, 8, 64, True, None, "f32"), (1, 78, 2, 40, False, [70], "f32"), (1, 44, 2, 96, True, None, "f32"),
    (1, 45, 2, 96, True, None, "f32"), (1, 112, 2, 128, True, None, "f32"), (1, 113, 2, 128, False, None, "f32"), (2, 3, 2, 24, True, None, "f32"),
    (1, 2, 2, 64, True, None, "bf16"), (2, 3, 2, 96, False, [1, 3], "bf16"), (1, 40, 2, 128, True, None, "bf16"), (1, 41, 2, 128, True, None, "bf16"),
    (1, 52, 2, 80, True, None, "bf16"), (1, 53, 2, 80, True, None, "bf16"), (1, 80, 2, 80, True, None, "bf16"), (1, 81, 2, 80, False, [64], "bf16"),
])
def test_attention_bwd_one_launch(B, S, heads, d, causal, lens, dtype):
    test_attention_fwd_bwd(B, S, heads, d, causal, lens, dtype)


# Both sides of the limits between the kernels of one row per block and the matrix-core ones
@pytest.mark.parametrize("B,S,heads,d,causal,lens", [
    (2, 5, 2, 64, True, None), (8, 3, 32, 64, False, [1, 2, 3, 3, 1, 2, 3, 1]), (2, 12, 2, 128, True, None), (3, 13, 2, 128, False, None),
    (2, 16, 16, 64, True, None), (3, 16, 16, 64, True, None), (2, 17, 2, 64, False, [17, 9]), (1, 24, 4, 24, True, None), (1, 25, 4, 24, True, None),
    (2, 32, 16, 64, False, [30, 32]), (3, 37, 16, 40, True, None), (1, 244, 2, 128, False, [70]), (1, 245, 2, 128, True, None), (1, 200, 2, 64, True, None), (1, 201, 2, 64, True, None), (2, 70, 2, 80, True, None), (3, 67, 4, 80, False, [67, 1, 40]),
    (1, 90, 4, 128, True, None), (1, 127, 2, 128, False, None),
])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention_short_sequences(B, S, heads, d, causal, lens, dtype):
    test_attention_fwd_bwd(B, S, heads, d, causal, lens, dtype)


@pytest.mark.parametrize("S,heads,d", [(77, 2, 64), (333, 1, 128), (333, 2, 40), (577, 1, 96), (545, 1, 128), (130, 2, 24), (100, 1, 112)])
def test_attention_ragged_lengths_keep_probabilities_in_fp32(S, heads, d):
    """bf16 storage, a length that is no multiple of 64: P and dS stay in fp32.  Keys, values, queries and output
    gradients come in pairs whose contributions nearly cancel (v, -v under almost equal weights, ...; keys far
    from the origin, so that dQ = sum dS k is what is left of sum dS = 0).  Rounding P and dS to bf16 then costs
    1.1e-2 and more in the 2-norm of every result (emulated in 64 bits); kept in fp32 what remains is the
    rounding of the stored result, at most 2^-9, and as much again for the fp32 sums and scores."""
    import torch
    import paper_2410_19367_amd as bp
    B, H, n = 1, heads * d, (S + 1) // 2
    half = lambda role: si.round_to(si.normal(si.stream_key(0, role, S, heads, d), (heads, n, d)), "bf16").astype(np.float64)
    q, k, v, g = half("pq"), half("pk"), half("pv"), half("pg")
    step = 0.125 * np.sign(np.round(half("ps")))
    def pairs(a, b):
        o = np.empty((heads, 2 * n, d))
        o[:, 0::2], o[:, 1::2] = a, b
        return si.round_to(o[:, :S], "bf16").astype(np.float64)
    q, k, v, g = pairs(q, q * (1 + 2.0 ** -5)), pairs(k + 8, k + 8 + step), pairs(v, -v), pairs(g, -g)
    merge = lambda t: np.swapaxes(t, 0, 1).reshape(B, S, H)
    qd = hz.to_dev(np.concatenate([merge(q), merge(k), merge(v)], -1), "bf16")
    dd = hz.to_dev(merge(g), "bf16")
    ctx, dqkv = hz.empty_like_dev((B, S, H), "bf16"), hz.empty_like_dev((B, S, 3 * H), "bf16")
    lse, delta = torch.empty((B, heads, S), device="cuda"), torch.empty((B, heads, S), device="cuda")
    bp.bp_op_attention_fwd(bp.BP_BF16, B, S, heads, d, False, None, qd, ctx, lse)
    bp.bp_op_attention_bwd(bp.BP_BF16, B, S, heads, d, False, None, qd, ctx, lse, dd, dqkv, delta)
    torch.cuda.synchronize()
    s = q @ np.swapaxes(k, 1, 2) / np.sqrt(d)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    got_ctx = hz.to_host(ctx)
    o = np.swapaxes(got_ctx.reshape(S, heads, d), 0, 1)         # the backward starts from the stored ctx
    ds = p * (g @ np.swapaxes(v, 1, 2) - (g * o).sum(-1, keepdims=True))
    got, t = hz.to_host(dqkv), lambda a: np.swapaxes(a, 1, 2)
    for name, a, ref in (("ctx", got_ctx, p @ v), ("dq", got[..., :H], ds @ k / np.sqrt(d)),
                         ("dk", got[..., H:2 * H], t(ds) @ q / np.sqrt(d)), ("dv", got[..., 2 * H:], t(p) @ g)):
        ref = merge(ref)
        err = np.linalg.norm(a - ref) / np.linalg.norm(ref)
        print(f"  S {S} d {d} {name} {err:.2e}", flush=True)
        assert err <= 2.0 ** -8, (name, err)


@pytest.mark.parametrize("S,heads,d,lens,dtype", [
    (77, 2, 64, [50, 77], "bf16"), (333, 1, 128, [100, 333], "bf16"), (577, 2, 40, [1, 560], "bf16"), (70, 1, 24, [65, 3], "bf16"),
    (64, 2, 64, [50, 64], "f32"), (77, 2, 96, [64, 33], "f32"), (333, 1, 128, [100, 1], "f32"), (128, 2, 24, [127, 96], "f32"),
])
def test_attention_padding_may_hold_anything(S, heads, d, lens, dtype):
    """Keys and values beyond a sequence's valid length take no part: NaN and infinities there leave every bit
    of the outputs as zeros there do, and their own gradients are zeros."""
    import torch
    import paper_2410_19367_amd as bp
    dt = bp.BP_BF16 if dtype == "bf16" else bp.BP_F32
    B, H = len(lens), heads * d
    qkv = _randn("nqkv", (B, S, 3 * H), 1.0, dtype=dtype)
    dd = hz.to_dev(_randn("ndctx", (B, S, H), dtype=dtype), dtype)
    lens_d = torch.tensor(lens, dtype=torch.int32, device="cuda")
    results = []
    for fill in (0.0, float("nan"), float("inf")):
        qd = hz.to_dev(qkv, dtype)
        for b, n in enumerate(lens):
            qd[b, n:, H:] = fill
        ctx, dqkv = hz.empty_like_dev((B, S, H), dtype), hz.empty_like_dev((B, S, 3 * H), dtype)
        lse, delta = torch.empty((B, heads, S), device="cuda"), torch.empty((B, heads, S), device="cuda")
        bp.bp_op_attention_fwd(dt, B, S, heads, d, False, lens_d, qd, ctx, lse)
        bp.bp_op_attention_bwd(dt, B, S, heads, d, False, lens_d, qd, ctx, lse, dd, dqkv, delta)
        torch.cuda.synchronize()
        results.append([hz.to_host(t) for t in (ctx, lse, delta, dqkv)])
    for r in results:
        for b, n in enumerate(lens):
            assert not np.any(r[3][b, n:, H:])
        for a, ref in zip(r, results[0]):
            assert np.all(np.isfinite(a)) and np.array_equal(a, ref)


@pytest.mark.parametrize("S,heads,d,t,dtype", [
    (100, 2, 64, 40, "bf16"), (333, 1, 128, 331, "bf16"), (545, 1, 40, 100, "bf16"), (70, 2, 96, 65, "bf16"), (3001, 1, 64, 1500, "bf16"),
    (64, 2, 64, 1, "f32"), (100, 2, 96, 40, "f32"), (333, 1, 128, 331, "f32"), (128, 1, 24, 70, "f32"),
])
@pytest.mark.parametrize("where", ["q", "k", "v", "dctx"])
def test_attention_causal_token_that_is_not_finite(S, heads, d, t, dtype, where):
    """A causal mask keeps token t from those before it, whatever it holds: what does not depend on it stays as
    it is without it (to the rounding of either path), in fp32 and at lengths that are no multiple of 64."""
    import torch
    import paper_2410_19367_amd as bp
    dt = bp.BP_BF16 if dtype == "bf16" else bp.BP_F32
    H = heads * d
    runs = []
    for fill in (None, float("nan"), float("inf")):
        qd = hz.to_dev(_randn("cqkv", (1, S, 3 * H), 1.0, dtype=dtype), dtype)
        dd = hz.to_dev(_randn("cdctx", (1, S, H), dtype=dtype), dtype)
        if fill is not None:
            if where == "dctx":
                dd[0, t] = fill
            else:
                k = "qkv".index(where)
                qd[0, t, k * H:(k + 1) * H] = fill
        ctx, dqkv = hz.empty_like_dev((1, S, H), dtype), hz.empty_like_dev((1, S, 3 * H), dtype)
        lse, delta = torch.empty((1, heads, S), device="cuda"), torch.empty((1, heads, S), device="cuda")
        bp.bp_op_attention_fwd(dt, 1, S, heads, d, True, None, qd, ctx, lse)
        bp.bp_op_attention_bwd(dt, 1, S, heads, d, True, None, qd, ctx, lse, dd, dqkv, delta)
        torch.cuda.synchronize()
        g = hz.to_host(dqkv)[0]
        runs.append({"ctx": hz.to_host(ctx)[0], "dq": g[:, :H], "dk": g[:, H:2 * H], "dv": g[:, 2 * H:]})
    rows = np.arange(S)
    before, others, after, every, none = rows < t, rows != t, rows > t, rows >= 0, rows < 0
    clean = {"q": {"ctx": others, "dq": others, "dk": after, "dv": after},
             "k": {"ctx": before, "dq": before, "dk": none, "dv": none},
             "v": {"ctx": before, "dq": before, "dk": none, "dv": every},
             "dctx": {"ctx": every, "dq": others, "dk": after, "dv": after}}[where]
    for r in runs[1:]:
        for name, ok in clean.items():
            ref, got = runs[0][name], r[name][ok]
            assert np.all(np.isfinite(got)), (name, rows[ok][~np.all(np.isfinite(got), axis=-1)])
            if got.size:
                err = np.max(np.abs(got - ref[ok])) / np.max(np.abs(ref))
                assert err <= (1e-2 if dtype == "bf16" else 5e-5), (name, err)


@pytest.mark.parametrize("S,heads", [(600, 4), (64, 16), (333, 8)])
def test_attention_f32_large_scores(S, heads):
    """fp32, one valid key per sequence, scores of about +-200 (d = 64: the scale is a power of two): every
    probability is exactly one whatever the score, so ctx is v to an ulp and dv = sum dctx with the rounding of a
    sum of S terms (2^-24 sqrt(S) of their norm; twice that allowed)."""
    import torch
    import paper_2410_19367_amd as bp
    B, d = 2, 64
    H = heads * d
    qkv = _randn("sqkv", (B, S, 3 * H), dtype="f32")
    qkv[..., :2 * H] *= 14
    dctx = _randn("sdctx", (B, S, H), dtype="f32")
    lens = torch.ones(B, dtype=torch.int32, device="cuda")
    qd, dd = hz.to_dev(qkv, "f32"), hz.to_dev(dctx, "f32")
    ctx, dqkv = hz.empty_like_dev((B, S, H), "f32"), hz.empty_like_dev((B, S, 3 * H), "f32")
    lse, delta = torch.empty((B, heads, S), device="cuda"), torch.empty((B, heads, S), device="cuda")
    bp.bp_op_attention_fwd(bp.BP_F32, B, S, heads, d, False, lens, qd, ctx, lse)
    bp.bp_op_attention_bwd(bp.BP_F32, B, S, heads, d, False, lens, qd, ctx, lse, dd, dqkv, delta)
    torch.cuda.synchronize()
    v0 = qkv[:, :1, 2 * H:].astype(np.float64)
    assert np.allclose(hz.to_host(ctx), np.broadcast_to(v0, (B, S, H)), rtol=2.0 ** -22, atol=0)
    ref = dctx.astype(np.float64).sum(1)
    err = np.linalg.norm(hz.to_host(dqkv)[:, 0, 2 * H:] - ref) / np.linalg.norm(ref)
    print(f"  S {S}: dv {err:.2e}", flush=True)
    assert err <= 2 * 2.0 ** -24 * np.sqrt(S), err


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention_one_token(dtype):
    """S = 1: probability one, so ctx = v and dv = dctx exactly, and dq, dk vanish up to the rounding of
    dP - delta, two equal sums of d = 64 products of about unit size: below 64 * 64 * 2^-24 * 16 * max|k|/8 < 1e-2."""
    import torch
    import paper_2410_19367_amd as bp
    B, heads, d = 3, 2, 64
    H, dt = heads * d, bp.BP_BF16 if dtype == "bf16" else bp.BP_F32
    qkv, dctx = _randn("oqkv", (B, 1, 3 * H), dtype=dtype), _randn("odctx", (B, 1, H), dtype=dtype)
    qd, dd = hz.to_dev(qkv, dtype), hz.to_dev(dctx, dtype)
    ctx, dqkv = hz.empty_like_dev((B, 1, H), dtype), hz.empty_like_dev((B, 1, 3 * H), dtype)
    lse, delta = torch.empty((B, heads, 1), device="cuda"), torch.empty((B, heads, 1), device="cuda")
    bp.bp_op_attention_fwd(dt, B, 1, heads, d, True, None, qd, ctx, lse)
    bp.bp_op_attention_bwd(dt, B, 1, heads, d, True, None, qd, ctx, lse, dd, dqkv, delta)
    torch.cuda.synchronize()
    assert np.allclose(hz.to_host(ctx), qkv[..., 2 * H:], rtol=1e-5)
    got = hz.to_host(dqkv)
    assert np.allclose(got[..., 2 * H:], dctx, rtol=1e-5 if dtype == "f32" else 2 ** -8)
    assert np.max(np.abs(got[..., :2 * H])) < 1e-2


@pytest.mark.parametrize("B,S,heads,d,causal", [(1, 512, 2, 128, True), (2, 256, 2, 64, False), (1, 1024, 1, 128, True)])
def test_attention_wide_score_range(B, S, heads, d, causal):
    """Scores whose magnitude grows along the key axis (std up to ~16, maxima tens of binary orders
    apart between tiles): the running softmax reference has to move many times, by large and by
    small amounts, and the result must still match the definition."""
    import torch
    import paper_2410_19367_amd as bp
    H = heads * d
    qkv = _randn("wqkv", (B, S, 3 * H), 1.0, dtype="f32").astype(np.float64)
    ramp = 1.0 + 7.0 * np.arange(S) / S
    qkv[..., :H] *= 2.0
    qkv[..., H:2 * H] *= ramp[None, :, None]
    qkv = si.round_to(qkv, "bf16")
    dctx = _randn("wdctx", (B, S, H), dtype="bf16")
    q64 = qkv.astype(np.float64)
    q = O._split_heads(q64[..., :H], heads); k = O._split_heads(q64[..., H:2 * H], heads)
    v = O._split_heads(q64[..., 2 * H:], heads)
    ctx_h, p = O.attention_fwd(q, k, v, causal, None)
    ctx_ref = O._merge_heads(ctx_h)
    dq, dk, dv = O.attention_bwd(O._split_heads(dctx.astype(np.float64), heads), q, k, v, p)
    dqkv_ref = np.concatenate([O._merge_heads(dq), O._merge_heads(dk), O._merge_heads(dv)], -1)
    qd = hz.to_dev(qkv, "bf16")
    ctx = hz.empty_like_dev((B, S, H), "bf16")
    lse = torch.empty((B, heads, S), device="cuda")
    bp.bp_op_attention_fwd(bp.BP_BF16, B, S, heads, d, causal, None, qd, ctx, lse)
    dqkv = hz.empty_like_dev((B, S, 3 * H), "bf16")
    delta = torch.empty((B, heads, S), device="cuda")
    ctx_in = hz.to_dev(si.round_to(ctx_ref, "bf16"), "bf16")
    bp.bp_op_attention_bwd(bp.BP_BF16, B, S, heads, d, causal, None, qd, ctx_in, lse, hz.to_dev(dctx, "bf16"), dqkv,
                           delta)
    torch.cuda.synchronize()
    assert np.all(np.isfinite(hz.to_host(ctx)))
    assert hz.rel_err(hz.to_host(ctx), ctx_ref) <= 1e-2
    got = hz.to_host(dqkv)
    for name, sl in (("dq", slice(0, H)), ("dk", slice(H, 2 * H)), ("dv", slice(2 * H, 3 * H))):
        err = hz.rel_err(got[..., sl], dqkv_ref[..., sl])
        assert err <= 2e-2, (name, err)


@pytest.mark.parametrize("M,N,T,n", [
    (512, 768, 256, 2),        # 128-tile direct-to-LDS kernel, segment change between slices
    (2048, 6144, 192, 3),      # 256x192 tiles
    (4096, 4096, 128, 4),      # 256x256 tiles, four segments of two slices
    (256, 256, 64, 4),         # one slice per segment
    (256, 256, 64, 8),         # the most segments
    (2048, 2048, 128, 8),      # 256x256 tiles, eight segments of two slices
    (200, 264, 136, 3),        # ragged: one launch per segment
    (512, 768, 256, 1),
    (2048, 2048, 1024, 4),     # with a workspace: 64 tiles x 4 token slices, one per segment
    (2048, 2048, 2048, 2),     # with a workspace: 4 token slices, two per segment
    (2048, 2048, 1536, 2),     # with a workspace: 3072 tokens -> 3 slices, boundaries inside segments
    (4096, 5120, 2048, 2),     # with a workspace: 320 tiles, the last 64 cut into 4 token slices
    (512, 768, 1024, 2),       # with a workspace: 24 tiles of 128 x 128, two token slices, K steps of 128
    (512, 768, 1088, 2),       # the same with K steps of 64 (1088 = 17 * 64)
    (2048, 2560, 1664, 2),     # with a workspace: 80 tiles x 3 token slices of 18, 17, 17 steps
    (512, 768, 1600, 2),       # with a workspace: 24 small tiles x 3 token slices of 17, 17, 16 steps
    (2048, 1152, 2048, 2),     # with a workspace, N a multiple of 128 and 192 but not of 256
    (264, 520, 77, 3),         # ragged everywhere, segments of an odd number of tokens
    (264, 520, 1025, 3),       # the same with a workspace: token slices that end inside segments
    (4000, 3200, 33, 2),       # 256x256 tiles with edges, segments shorter than a slice
])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("overwrite", [0, 1])
def test_wgrad_group(M, N, T, n, dtype, overwrite):
    """dW (+)= sum_i X_i^T dY_i over a group of micro-batches in one call."""
    import torch
    import paper_2410_19367_amd as bp
    if dtype == "f32" and M * N > 2 ** 21:
        pytest.skip("fp32 path is exercised on the small shapes")
    dt = bp.BP_BF16 if dtype == "bf16" else bp.BP_F32
    xs = [_randn(f"gx{i}", (T, M), dtype=dtype) for i in range(n)]
    ys = [_randn(f"gy{i}", (T, N), dtype=dtype) for i in range(n)]
    w0 = _randn("gw0", (M, N), dtype="f32")
    ref = sum(x.astype(np.float64).T @ y.astype(np.float64) for x, y in zip(xs, ys))
    if not overwrite:
        ref = ref + w0
    xd = [hz.to_dev(x, dtype) for x in xs]
    yd = [hz.to_dev(y, dtype) for y in ys]
    wd = _f32_dev(w0)
    ws = torch.empty(4 * M * N, device="cuda") if T >= 1024 else None
    bp.bp_op_wgrad_group(dt, M, N, T, xd, yd, wd, overwrite, ws, 0 if ws is None else ws.numel())
    torch.cuda.synchronize()
    err = hz.rel_err(wd.cpu().numpy().astype(np.float64), ref)
    assert err <= (2e-3 if dtype == "bf16" else 1e-5), err


@pytest.mark.parametrize("M,N,T", [(8192, 8, 370001), (8192, 128, 371200), (32768, 8, 80000)])
def test_wgrad_operand_beyond_4_gib(M, N, T):
    """X of 5 to 6 GB: K slices (and, in the last case, one walk over all tokens) that reach offsets no 32-bit
    number holds; a wrapped offset reads other tokens, an error of the size of the result.  fp32 sums of T products
    of about unit size in another order: below 1e-4 of the largest element."""
    import torch
    import paper_2410_19367_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.randn(T, M, device="cuda", generator=g, dtype=torch.bfloat16)
    y = torch.randn(T, N, device="cuda", generator=g, dtype=torch.bfloat16)
    assert x.numel() * 2 > 2 ** 32
    ref = torch.zeros(M, N, device="cuda", dtype=torch.float64)
    for t in range(0, T, 8192):
        ref += (x[t:t + 8192].float().t().contiguous() @ y[t:t + 8192].float()).double()
    w = torch.empty(M, N, device="cuda")
    ws = torch.empty(4 * M * max(N, 128), device="cuda")         # whole 128 x 128 tiles
    bp.bp_op_wgrad_group(bp.BP_BF16, M, N, T, [x], [y], w, 1, ws, ws.numel())
    torch.cuda.synchronize()
    err = float((w.double() - ref).abs().max() / ref.abs().max())
    assert err <= 1e-4, err


@pytest.mark.parametrize("M,N,T,n", [(1024, 1024, 700, 4), (512, 512, 2000, 8)])
def test_wgrad_group_f32_rounds_like_one_micro_batch(M, N, T, n):
    """fp32: the sum over a group is no less accurate than micro-batch after micro-batch.  A chain of T additions of
    random terms is off by 0.31 2^-24 sqrt(T) in the 2-norm (rounding errors of 0.43 2^-24 of the partial sum, rms,
    partial sums growing like sqrt(k)); n such chains added up are too; a single one of n T is off by sqrt(n)
    times that."""
    import torch
    import paper_2410_19367_amd as bp
    xs = [_randn(f"rx{i}", (T, M), dtype="f32") for i in range(n)]
    ys = [_randn(f"ry{i}", (T, N), dtype="f32") for i in range(n)]
    ref = sum(x.astype(np.float64).T @ y.astype(np.float64) for x, y in zip(xs, ys))
    w = torch.empty(M, N, device="cuda")
    bp.bp_op_wgrad_group(bp.BP_F32, M, N, T, [_f32_dev(x) for x in xs], [_f32_dev(y) for y in ys], w, 1, None, 0)
    torch.cuda.synchronize()
    err = np.linalg.norm(w.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
    print(f"  {M} x {N}, {n} x {T}: {err:.2e}", flush=True)
    assert err <= 1.3 * 0.31 * 2.0 ** -24 * np.sqrt(T), err
