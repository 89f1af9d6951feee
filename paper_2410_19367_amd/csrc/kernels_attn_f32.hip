// Fused fp32 attention on the gfx950 matrix cores (v_mfma_f32_32x32x2_f32), the fp32 counterpart of the
// bf16 kernels: forward with online softmax and the backward in two deterministic parts (dQ; dK and
// dV; one launch each or both in one), for any sequence length and head widths that are multiples of 8 up to 128.
//
// Bound: the fp32 matrix rate (an eighth of the bf16 one), so the kernels are kept simple: four waves,
// 32 queries (keys in dK/dV) x one half of every 64-row tile each, tiles through two LDS stages.
// Scores keep the orientation that leaves the softmax row of a query (column of a key) in one lane:
//   forward, dQ :  S^T[key][q] = K Q^T      lane <-> query, registers <-> keys
//   dK, dV      :  S  [q][key] = Q K^T      lane <-> key,   registers <-> queries
// Register v of the accumulator then is, as it stands, the B operand of the two-deep MFMA that
// contracts over rows {v, lower half} and {v, upper half}; its A operand (V^T, K^T, dO^T, Q^T) is one
// float per lane of the same row-major tile.
// Measured (forward / backward): B 2, S 512, 12 heads of 64, causal 26 / 68 us against 163 / 814 us for the
// one-row-per-block kernels; without the mask 62 / 39 TFLOP/s.  Heads wider than 64 leave one wave per SIMD (dK/dV
// at 128 spills 18 registers): S 300, 16 heads of 128, without the mask 34.5 / 61 us (rows 135 / 740 us), of 96
// 27.7 / 44 us (107 and 80 us in two launches).
#include <atomic>

#include "bp_kernels.h"
#include "bp_device.h"
#include "bp_attn_rows.h"
#include "bp_tile.h"

namespace bp {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// tile [64][D] floats: 16-byte chunk c of row r sits at c ^ (r & 15)
template <int D> __device__ __forceinline__ int f32_tile_off(int row, int chunk) {
    return row * (D * 4) + ((chunk ^ (row & 15)) << 4);
}

// Direct global->LDS copy of the first `rows` rows of a [64][D] tile by four waves (keys: up to the valid
// length, since what padding holds must not reach the products: zero times NaN); the other rows and
// the columns at and beyond the head width dr lie outside the buffer descriptor's range: zeros.
template <int D>
struct F32Tile {
    static constexpr int CPR = D / 4, NI = 64 * CPR / 64 / 4;
    uint32_t off[NI];
    __device__ __forceinline__ void init(int wave, int lane, int ld, int dr) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int P = (wave + 4 * i) * 64 + lane, row = P / CPR, c = (P % CPR) ^ (row & 15);
            off[i] = c * 4 < dr ? 4u * (uint32_t)(row * ld + c * 4) : kOutside;
        }
    }
    __device__ __forceinline__ void issue(const float* base, int ld, int dr, int rows, char* lds, int wave) const {
        const rsrc_t src = make_rsrc(base, 4u * (uint32_t)((min(rows, 64) - 1) * ld + dr));
#pragma unroll
        for (int i = 0; i < NI; ++i) dma16(src, off[i], 0, lds + (wave + 4 * i) * 1024);
    }
};

// chunk pair j (columns 8j .. 8j+7, this lane's half of them) of row row0 + lane % 32
template <int D>
__device__ __forceinline__ f32x4 rows4(const char* lds, int row0, int j, int lane) {
    return *reinterpret_cast<const f32x4*>(lds + f32_tile_off<D>(row0 + (lane & 31), 2 * j + (lane >> 5)));
}
// element (row, col0 + lane % 32)
template <int D>
__device__ __forceinline__ float col1(const char* lds, int row, int col0, int lane) {
    const int col = col0 + (lane & 31);
    return *reinterpret_cast<const float*>(lds + f32_tile_off<D>(row, col >> 2) + (col & 3) * 4);
}
// load(i + 1) is issued before use(i), and nothing moves across the end of a step: one step's LDS reads are
// in flight while the previous one's MFMAs run, and the compiler does not pull all the reads of a tile
// to its front (which spilled registers in the backward kernels)
template <int N, typename L, typename U>
__device__ __forceinline__ void pipelined(L load, U use) {
    load(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (i + 1 < N) load(i + 1);
        use(i);
        __builtin_amdgcn_sched_barrier(0);
    }
}
__device__ __forceinline__ f32x4 row_piece(const float* row, int col, int dr) {
    return col < dr ? *reinterpret_cast<const f32x4*>(row + col) : f32x4{0.f, 0.f, 0.f, 0.f};
}
__device__ __forceinline__ int f32_acc_row(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }
// out^T (D x 32) += tile[row0 .. row0 + 31][.]^T x, x as a score accumulator holds it
template <int D, int DC>
__device__ __forceinline__ void contract(const char* tile, int row0, int lane, const f32x16& x, f32x16 (&out)[DC / 32]) {
    constexpr int DT = DC / 32;
    float av[2][4][DT];
    pipelined<4>([&](int g) {
#pragma unroll
                     for (int e = 0; e < 4; ++e)
#pragma unroll
                         for (int t = 0; t < DT; ++t)
                             av[g & 1][e][t] = col1<D>(tile, row0 + f32_acc_row(4 * g + e, lane >> 5), 32 * t, lane);
                 },
                 [&](int g) {
#pragma unroll
                     for (int e = 0; e < 4; ++e)
#pragma unroll
                         for (int t = 0; t < DT; ++t)
                             out[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[g & 1][e][t], x[4 * g + e], out[t], 0, 0, 0);
                 });
}
// s += A b^T and p += C d^T over the head width: 32 rows of the tiles A and C, b and d in registers
template <int D, int DC>
__device__ __forceinline__ void scores(const char* tile_a, const char* tile_c, int row0, int lane,
                                       const f32x4 (&b)[DC / 8], const f32x4 (&d)[DC / 8], f32x16& s, f32x16& p) {
    f32x4 fa[2], fc[2];
    pipelined<DC / 8>([&](int j) {
                         fa[j & 1] = rows4<D>(tile_a, row0, j, lane);
                         fc[j & 1] = rows4<D>(tile_c, row0, j, lane);
                     },
                     [&](int j) {
#pragma unroll
                         for (int e = 0; e < 4; ++e) {
                             s = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[j & 1][e], b[j][e], s, 0, 0, 0);
                             p = __builtin_amdgcn_mfma_f32_32x32x2f32(fc[j & 1][e], d[j][e], p, 0, 0, 0);
                         }
                     });
}
// no NaN and no infinity in rows row0 .. row0 + 31 of a tile (the same answer in every lane)
template <int D, int DC>
__device__ __forceinline__ bool rows_finite(const char* tile, int row0, int lane) {
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < DC / 8; ++j) {
        const f32x4 f = rows4<D>(tile, row0, j, lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) z = __builtin_fmaf(0.f, f[e], z);
    }
    return __builtin_amdgcn_ballot_w64(z != 0.f) == 0;
}
// exp(s scale - m).  The difference is taken before the change of base: scores are then rounded relative to what is left
// of them and not to themselves (with log2 e folded into the scale, a score of 200 that is its row's only one
// had the probability 1 +- 1e-5).
__device__ __forceinline__ float exp_diff(float s, float scale, float m) {
    return __builtin_amdgcn_exp2f(__builtin_fmaf(s, scale, -m) * kLog2e);
}
__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
    return z;
}
// Query (key) block of this thread block: the most expensive causal blocks start first
__device__ __forceinline__ void f32_block(const AttnArgs& a, int bid, bool last_is_heavy, int& blk, int& head, int& b) {
    const int nblk = (a.S + 63) / 64, per = nblk * a.heads, lin = bid % per;
    b = bid / per;
    head = lin % a.heads;
    blk = a.causal && last_is_heavy ? nblk - 1 - lin / a.heads : lin / a.heads;
}

template <int D, int DC>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_fwd_f32_kernel(AttnArgs a, float scale) {
    attn_args_now(a, scale);
    constexpr int KS = DC / 8, DT = DC / 32, TILE = 64 * D * 4, STAGE = 2 * TILE;    // K then V
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qg = wave >> 1, kh = wave & 1;
    int qblk, head, b;
    f32_block(a, blockIdx.x, true, qblk, head, b);
    const int dr = a.d, H = a.heads * dr, ld = 3 * H, S = a.S;
    const float* qkv = (const float*)a.qkv + (size_t)b * S * ld + head * dr;
    const int q_wave = qblk * 64 + qg * 32, q_lane = q_wave + (lane & 31);
    const int klen = a.causal ? S : (a.lens ? a.lens[b] : S);
    const int nt = ((a.causal ? min(qblk * 64 + 64, S) : klen) + 63) / 64;

    f32x4 qf[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) qf[j] = row_piece(qkv + (size_t)min(q_lane, S - 1) * ld, 8 * j + 4 * h, dr);
    f32x16 ot[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) ot[t] = zero16();
    float m = -INFINITY, lsum = 0.f;
    bool by_rows = false;       // a value on the diagonal is not finite: see bp_attn_rows.h

    F32Tile<D> plan;
    plan.init(wave, lane, ld, dr);
    auto request = [&](int t) {
        char* st = smem + (t & 1) * STAGE;
        plan.issue(qkv + H + (size_t)t * 64 * ld, ld, dr, klen - t * 64, st, wave);
        plan.issue(qkv + 2 * H + (size_t)t * 64 * ld, ld, dr, klen - t * 64, st + TILE, wave);
    };
    if (nt > 0) request(0);
    for (int t = 0; t < nt; ++t) {
        BP_WAIT_VMCNT(0);
        __syncthreads();
        if (t + 1 < nt) request(t + 1);
        const int kw = t * 64 + 32 * kh;
        if ((a.causal && kw > q_wave + 31) || kw >= klen) continue;
        const char* sk = smem + (t & 1) * STAGE;
        const char* sv = sk + TILE;
        f32x16 st2 = zero16();
        f32x4 kf[2];
        pipelined<KS>([&](int j) { kf[j & 1] = rows4<D>(sk, 32 * kh, j, lane); },
                      [&](int j) {
 #pragma unroll
                          for (int e = 0; e < 4; ++e)
                              st2 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j & 1][e], qf[j][e], st2, 0, 0, 0);
                      });
        const bool need_mask = (a.causal && kw + 31 > q_wave) || kw + 32 > klen;
        float mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = kw + f32_acc_row(v, h);
            if (need_mask && ((a.causal && key > q_lane) || key >= klen)) st2[v] = -INFINITY;
            mx = fmaxf(mx, st2[v]);
        }
        mx = halves_max(mx) * scale;
        // the running reference point moves only when a score is more than 8 binary orders above it
        if (__builtin_amdgcn_ballot_w64(mx > m + 8.f * kLn2) != 0) {
            const float m_new = fmaxf(m, mx);
            const float alpha = m == -INFINITY ? 0.f : exp_diff(m, 1.f, m_new);
            m = m_new;
            lsum *= alpha;
#pragma unroll
            for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
                for (int v = 0; v < 16; ++v) ot[t2][v] *= alpha;
        }
        const float m_use = m == -INFINITY ? 0.f : m;   // every key masked so far: no inf - inf
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            st2[v] = exp_diff(st2[v], scale, m_use);
            lsum += st2[v];
        }
        if (a.causal && kw + 31 > q_wave && !rows_finite<D, DC>(sv, 32 * kh, lane)) by_rows = true;
        contract<D, DC>(sv, 32 * kh, lane, st2, ot);
    }
    if (a.causal && any_wave(by_rows, smem)) {
        for (int q = qblk * 64; q < min(qblk * 64 + 64, S); ++q) attn_fwd_row<float>(a, scale, q, head, b, (float*)smem);
        return;
    }

    // merge the two key halves through LDS; half 0 has seen key 0, so its m is finite
    const float l = halves_sum(lsum);
    __syncthreads();
    float* xo = (float*)smem + qg * (DT * 16 * 64 + 128);
    if (kh == 1) {
#pragma unroll
        for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
            for (int v = 0; v < 16; ++v) xo[(t2 * 16 + v) * 64 + lane] = ot[t2][v];
        xo[DT * 16 * 64 + lane] = m;
        xo[DT * 16 * 64 + 64 + lane] = l;
    }
    __syncthreads();
    if (kh == 1 || q_lane >= S) return;
    const float m1 = xo[DT * 16 * 64 + lane], mm = fmaxf(m, m1);
    const float a0 = exp_diff(m, 1.f, mm), a1 = exp_diff(m1, 1.f, mm);
    const float ls = l * a0 + xo[DT * 16 * 64 + 64 + lane] * a1;
    const float inv = 1.f / ls;
    float* out = (float*)a.ctx + ((size_t)b * S + q_lane) * H + head * dr;
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = t2 * 32 + 8 * g + 4 * h;
            if (col >= dr) continue;
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o[e] = (ot[t2][4 * g + e] * a0 + xo[(t2 * 16 + 4 * g + e) * 64 + lane] * a1) * inv;
            *reinterpret_cast<f32x4*>(out + col) = o;
        }
    if (h == 0) a.lse[((size_t)b * a.heads + head) * S + q_lane] = mm + log2f(ls) * kLn2;
}

// dQ, and delta[q] = sum_d dO[q][d] O[q][d] for the dK/dV kernel
template <int D, int DC>
__device__ __forceinline__ void attn_bwd_dq_f32_block(const AttnArgs& a, float scale, int bid, char* smem) {
    constexpr int KS = DC / 8, DT = DC / 32, TILE = 64 * D * 4, STAGE = 2 * TILE;
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qg = wave >> 1, kh = wave & 1;
    int qblk, head, b;
    f32_block(a, bid, true, qblk, head, b);
    const int dr = a.d, H = a.heads * dr, ld = 3 * H, S = a.S;
    const float* qkv = (const float*)a.qkv + (size_t)b * S * ld + head * dr;
    const int q_wave = qblk * 64 + qg * 32, q_lane = q_wave + (lane & 31), q_src = min(q_lane, S - 1);
    const int klen = a.causal ? S : (a.lens ? a.lens[b] : S);
    const int nt = ((a.causal ? min(qblk * 64 + 64, S) : klen) + 63) / 64;

    const size_t orow = ((size_t)b * S + q_src) * H + head * dr;
    f32x4 qf[KS], dof[KS];
    float delta = 0.f;
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        qf[j] = row_piece(qkv + (size_t)q_src * ld, 8 * j + 4 * h, dr);
        dof[j] = row_piece((const float*)a.dctx + orow, 8 * j + 4 * h, dr);
        const f32x4 of = row_piece((const float*)a.ctx + orow, 8 * j + 4 * h, dr);
#pragma unroll
        for (int e = 0; e < 4; ++e) delta += of[e] * dof[j][e];
    }
    delta = halves_sum(delta);
    const size_t li = ((size_t)b * a.heads + head) * S + q_src;
    if (kh == 0 && h == 0 && q_lane < S) a.delta[li] = delta;
    const float lse = a.lse[li];

    f32x16 dq[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) dq[t] = zero16();
    bool by_rows = false;       // a key or value on the diagonal is not finite
    F32Tile<D> plan;
    plan.init(wave, lane, ld, dr);
    auto request = [&](int t) {
        char* st = smem + (t & 1) * STAGE;
        plan.issue(qkv + H + (size_t)t * 64 * ld, ld, dr, klen - t * 64, st, wave);
        plan.issue(qkv + 2 * H + (size_t)t * 64 * ld, ld, dr, klen - t * 64, st + TILE, wave);
    };
    if (nt > 0) request(0);
    for (int t = 0; t < nt; ++t) {
        BP_WAIT_VMCNT(0);
        __syncthreads();
        if (t + 1 < nt) request(t + 1);
        const int kw = t * 64 + 32 * kh;
        if ((a.causal && kw > q_wave + 31) || kw >= klen) continue;
        const char* sk = smem + (t & 1) * STAGE;
        const char* sv = sk + TILE;
        // (a value that is not finite makes dP of the queries that do not attend it NaN)
        if (a.causal && kw + 31 > q_wave && (!rows_finite<D, DC>(sk, 32 * kh, lane) || !rows_finite<D, DC>(sv, 32 * kh, lane)))
            by_rows = true;
        f32x16 sacc = zero16(), dp = zero16();
        scores<D, DC>(sk, sv, 32 * kh, lane, qf, dof, sacc, dp);
        const bool need_mask = (a.causal && kw + 31 > q_wave) || kw + 32 > klen;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            float p = exp_diff(sacc[v], scale, lse);
            const int key = kw + f32_acc_row(v, h);
            if (need_mask && ((a.causal && key > q_lane) || key >= klen)) p = 0.f;
            dp[v] = p * (dp[v] - delta);                // dS^T
        }
        contract<D, DC>(sk, 32 * kh, lane, dp, dq);
    }
    if (a.causal && any_wave(by_rows, smem)) {
        for (int q = qblk * 64; q < min(qblk * 64 + 64, S); ++q) attn_bwd_dq_row<float>(a, scale, q, head, b, (float*)smem);
        return;
    }
    __syncthreads();
    float* xo = (float*)smem + qg * (DT * 16 * 64);
    if (kh == 1) {
#pragma unroll
        for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
            for (int v = 0; v < 16; ++v) xo[(t2 * 16 + v) * 64 + lane] = dq[t2][v];
    }
    __syncthreads();
    if (kh == 1 || q_lane >= S) return;
    float* out = (float*)a.dqkv + ((size_t)b * S + q_lane) * ld + head * dr;
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = t2 * 32 + 8 * g + 4 * h;
            if (col >= dr) continue;
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (dq[t2][4 * g + e] + xo[(t2 * 16 + 4 * g + e) * 64 + lane]) * scale;
            *reinterpret_cast<f32x4*>(out + col) = o;
        }
}

// dK and dV: 32 keys per wave, one half of every 64-query tile of Q and dO that streams by
template <int D, int DC, bool ALONE>
__device__ __forceinline__ void attn_bwd_dkv_f32_block(const AttnArgs& a, float scale, int bid, char* smem) {
    constexpr int KS = DC / 8, DT = DC / 32, TILE = 64 * D * 4, STAGE = 2 * TILE + 512;   // Q, dO, lse[64], delta[64]
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave >> 1, qh = wave & 1;
    int kblk, head, b;
    f32_block(a, bid, false, kblk, head, b);
    const int dr = a.d, H = a.heads * dr, ld = 3 * H, S = a.S;
    const float* qkv = (const float*)a.qkv + (size_t)b * S * ld + head * dr;
    const float* dobase = (const float*)a.dctx + (size_t)b * S * H + head * dr;
    const int k_wave = kblk * 64 + kg * 32, k_lane = k_wave + (lane & 31);
    const int klen = a.causal ? S : (a.lens ? a.lens[b] : S);
    const int k_src = max(min(k_lane, klen - 1), 0);     // row this lane reads (its own, unless it is padding)
    float* dk_out = (float*)a.dqkv + ((size_t)b * S + k_lane) * ld + H + head * dr;
    float* dv_out = dk_out + H;
    const float* lse = a.lse + ((size_t)b * a.heads + head) * S;
    const float* dlt = a.delta + ((size_t)b * a.heads + head) * S;

    f32x4 kf[KS], vf[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        kf[j] = row_piece(qkv + H + (size_t)k_src * ld, 8 * j + 4 * h, dr);
        vf[j] = row_piece(qkv + 2 * H + (size_t)k_src * ld, 8 * j + 4 * h, dr);
    }
    f32x16 dk[DT], dv[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) { dk[t] = zero16(); dv[t] = zero16(); }
    bool by_rows = false;       // a query on the diagonal is not finite
    // a block of padding keys that no query attends skips the loop and stores zeros
    const int t0 = a.causal ? kblk : 0, nt = kblk * 64 >= klen ? t0 : (S + 63) / 64;

    F32Tile<D> plan_q, plan_do;
    plan_q.init(wave, lane, ld, dr);
    plan_do.init(wave, lane, H, dr);
    auto request = [&](int t) {
        char* st = smem + (t & 1) * STAGE;
        plan_q.issue(qkv + (size_t)t * 64 * ld, ld, dr, S - t * 64, st, wave);
        plan_do.issue(dobase + (size_t)t * 64 * H, H, dr, S - t * 64, st + TILE, wave);
        const int q = min(t * 64 + lane, S - 1);
        if (wave == 0)
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(lse + q),
                                             (void __attribute__((address_space(3)))*)(st + 2 * TILE), 4, 0, 0);
        else if (ALONE && wave == 1)
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(dlt + q),
                                             (void __attribute__((address_space(3)))*)(st + 2 * TILE + 256), 4, 0, 0);
    };
    // Beside the dQ blocks, which leave delta in memory too late for this launch, a block takes delta of a tile's rows
    // from O and dO itself, four lanes to a row, in two halves that arrive under the products of the tile before.
    constexpr int NO = DC / 32;
    f32x4 o_row[ALONE ? 1 : NO], do_row[ALONE ? 1 : NO];
    float delta_part = 0.f;
    auto fetch_delta = [&](int t, int half) {
        if constexpr (!ALONE) {
            const size_t row = ((size_t)b * S + min(t * 64 + (int)(threadIdx.x >> 2), S - 1)) * H + head * dr;
#pragma unroll
            for (int j = 0; j < NO; ++j) {
                const int col = 16 * (half * NO + j) + 4 * (threadIdx.x & 3);
                o_row[j] = row_piece((const float*)a.ctx + row, col, dr);
                do_row[j] = row_piece((const float*)a.dctx + row, col, dr);
            }
        }
    };
    auto fold_delta = [&]() {
        if constexpr (!ALONE) {
#pragma unroll
            for (int j = 0; j < NO; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) delta_part += o_row[j][e] * do_row[j][e];
        }
    };
    // (rows past the end of the last tile, and the tile past the last one, repeat the last row)
    auto first_half = [&](int t) { fold_delta(); fetch_delta(t, 1); };
    auto second_half = [&](int t) {
        if constexpr (!ALONE) {
            fold_delta();
            delta_part += __shfl_xor(delta_part, 1, 64);
            delta_part += __shfl_xor(delta_part, 2, 64);
            if ((threadIdx.x & 3) == 0) ((float*)(smem + (t & 1) * STAGE + 2 * TILE))[64 + (threadIdx.x >> 2)] = delta_part;
            delta_part = 0.f;
        }
    };
    if (t0 < nt) {
        request(t0);
        fetch_delta(t0, 0);
        first_half(t0);
        second_half(t0);
    }
    for (int t = t0; t < nt; ++t) {
        BP_WAIT_VMCNT(0);
        __syncthreads();
        if (t + 1 < nt) request(t + 1);
        fetch_delta(t + 1, 0);
        const int qw = t * 64 + 32 * qh;
        if ((a.causal && qw + 31 < k_wave) || qw >= S) {
            first_half(t + 1);
            second_half(t + 1);
            continue;
        }
        const char* sq = smem + (t & 1) * STAGE;
        const char* sdo = sq + TILE;
        const float* s_lse = (const float*)(sq + 2 * TILE) + 32 * qh;
        const float* s_dlt = s_lse + 64;
        if (a.causal && qw < k_wave + 31 && (!rows_finite<D, DC>(sq, 32 * qh, lane) || !rows_finite<D, DC>(sdo, 32 * qh, lane) ||
                                             !stats_finite(s_lse, s_dlt, lane)))
            by_rows = true;
        f32x16 sacc = zero16(), dp = zero16();
        scores<D, DC>(sq, sdo, 32 * qh, lane, kf, vf, sacc, dp);
        const bool need_mask = (a.causal && qw < k_wave + 31) || qw + 32 > S || k_wave + 32 > klen;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int qi = f32_acc_row(v, h), q = qw + qi;
            float p = exp_diff(sacc[v], scale, s_lse[qi]);
            if (need_mask && ((a.causal && k_lane > q) || q >= S || k_lane >= klen)) p = 0.f;
            sacc[v] = p;
            dp[v] = p * (dp[v] - s_dlt[qi]);            // dS
        }
        first_half(t + 1);
        contract<D, DC>(sdo, 32 * qh, lane, sacc, dv);
        contract<D, DC>(sq, 32 * qh, lane, dp, dk);
        second_half(t + 1);
    }
    if (a.causal && any_wave(by_rows, smem)) {
        for (int k = kblk * 64; k < min(kblk * 64 + 64, S); ++k) attn_bwd_dkv_row<float, !ALONE>(a, scale, k, head, b, (float*)smem);
        return;
    }
    __syncthreads();
    float* xo = (float*)smem + kg * (2 * DT * 16 * 64);
    if (qh == 1) {
#pragma unroll
        for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                xo[(t2 * 16 + v) * 64 + lane] = dk[t2][v];
                xo[((DT + t2) * 16 + v) * 64 + lane] = dv[t2][v];
            }
    }
    __syncthreads();
    if (qh == 1 || k_lane >= S) return;
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = t2 * 32 + 8 * g + 4 * h;
            if (col >= dr) continue;
            f32x4 k4, v4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                k4[e] = (dk[t2][4 * g + e] + xo[(t2 * 16 + 4 * g + e) * 64 + lane]) * scale;
                v4[e] = dv[t2][4 * g + e] + xo[((DT + t2) * 16 + 4 * g + e) * 64 + lane];
            }
            *reinterpret_cast<f32x4*>(dk_out + col) = k4;
            *reinterpret_cast<f32x4*>(dv_out + col) = v4;
        }
}

template <int D, int DC>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_bwd_dq_f32_kernel(AttnArgs a, float scale) {
    attn_args_now(a, scale);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    attn_bwd_dq_f32_block<D, DC>(a, scale, blockIdx.x, smem);
}
template <int D, int DC>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_bwd_dkv_f32_kernel(AttnArgs a, float scale) {
    attn_args_now(a, scale);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    attn_bwd_dkv_f32_block<D, DC, true>(a, scale, blockIdx.x, smem);
}
// Both in one launch (attn_bwd_f32_one_launch): the first half of the blocks, which have more to do, dK and dV, the others dQ.
template <int D, int DC>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_bwd_f32_kernel(AttnArgs a, float scale) {
    attn_args_now(a, scale);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int n = gridDim.x / 2, bid = blockIdx.x;
    if (bid < n) attn_bwd_dkv_f32_block<D, DC, false>(a, scale, bid, smem);
    else attn_bwd_dq_f32_block<D, DC>(a, scale, bid - n, smem);
}

bool attn_f32_supported(const AttnArgs& a) {
    auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
    // (a tile's rows are addressed with 32-bit byte offsets)
    if (a.d % 8 || a.d < 8 || a.d > 128 || a.S < 1 || (long)a.heads * a.d > 1 << 20) return false;
    return al16(a.qkv) && al16(a.ctx) && (!a.dctx || al16(a.dctx)) && (!a.dqkv || al16(a.dqkv));
}

// dQ and dK/dV side by side in one launch while the blocks of both find room at once, two per CU (one for heads wider than
// 64).  n blocks of each on 256 CUs, two launches / one, us: d 64 n 40 52.6 / 36.0, 96 78.8 / 55.5, 192 79.4 / 68.4, 220
// 104 / 110, 256 79.2 / 80.1; d 40 192 76.8 / 70.1; d 24 64 28.0 / 16.2; d 96 128 120 / 67; d 128 64 151 / 90, 128 152 / 91.
bool attn_bwd_f32_one_launch(const AttnArgs& a) {
    const long n = (long)((a.S + 63) / 64) * a.heads * a.B, cu = cu_count();
    return a.d <= 64 ? 4 * n <= 3 * cu : 2 * n <= cu;
}

template <int D, int DC>
static hipError_t launch_f32_attn(const AttnArgs& a, bool bwd, hipStream_t s) {
    const float scale = 1.f / sqrtf((float)a.d);
    const dim3 grid(((a.S + 63) / 64) * a.heads * a.B), block(256);
    // two stages; the merges fit in them (forward: (D/32*1024 + 128) floats twice, dK/dV: D/32*4096 floats)
    // (more than the rows by themselves take: 60000 bytes at most)
    const int smem = 2 * 2 * 64 * D * 4, smem2 = smem + 1024;
    static std::atomic<bool> set{false};
    if (!set.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute((const void*)(attn_fwd_f32_kernel<D, DC>), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void*)(attn_bwd_dq_f32_kernel<D, DC>), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void*)(attn_bwd_dkv_f32_kernel<D, DC>), hipFuncAttributeMaxDynamicSharedMemorySize, smem2);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void*)(attn_bwd_f32_kernel<D, DC>), hipFuncAttributeMaxDynamicSharedMemorySize, smem2);
        if (e != hipSuccess) return e;
        set.store(true, std::memory_order_release);
    }
    if (bwd && attn_bwd_f32_one_launch(a)) {
        hipLaunchKernelGGL((attn_bwd_f32_kernel<D, DC>), dim3(2 * grid.x), block, smem2, s, a, scale);
    } else if (bwd) {
        hipLaunchKernelGGL((attn_bwd_dq_f32_kernel<D, DC>), grid, block, smem, s, a, scale);
        hipLaunchKernelGGL((attn_bwd_dkv_f32_kernel<D, DC>), grid, block, smem2, s, a, scale);
    } else {
        hipLaunchKernelGGL((attn_fwd_f32_kernel<D, DC>), grid, block, smem, s, a, scale);
    }
    return hipGetLastError();
}

// tile width D, computed width DC: the next multiple of 32 above the head width (the columns between
// are zeros; products, unlike loads and stores, have no guards)
static hipError_t launch_attn_f32(const AttnArgs& a, bool bwd, hipStream_t s) {
    if (a.d > 96) return launch_f32_attn<128, 128>(a, bwd, s);
    if (a.d > 64) return launch_f32_attn<128, 96>(a, bwd, s);
    return a.d > 32 ? launch_f32_attn<64, 64>(a, bwd, s) : launch_f32_attn<64, 32>(a, bwd, s);
}
hipError_t launch_attn_fwd_f32(const AttnArgs& a, hipStream_t s) { return launch_attn_f32(a, false, s); }
hipError_t launch_attn_bwd_f32(const AttnArgs& a, hipStream_t s) { return launch_attn_f32(a, true, s); }

}  // namespace bp
