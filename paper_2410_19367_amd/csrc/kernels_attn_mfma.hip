// Fused attention on the gfx950 matrix cores (bf16 inputs, fp32 softmax and accumulation; P and dS enter their
// second product in bf16 where the sequence length is a multiple of 64, else in fp32):
// forward with online softmax, and the backward in two deterministic parts (dQ; dK and dV), one launch each or both in one.
//
// All three kernels stream [64 rows][D] tiles of the packed qkv / dctx tensors through LDS with
// direct global->LDS loads and never materialise an S x S matrix.  Scores are produced
// transposed where that keeps the softmax row of a query inside one lane:
//   forward, dQ :  S^T[key][q] = K Q^T      lane <-> query, registers <-> keys
//   dK, dV      :  S  [q][key] = Q K^T      lane <-> key,   registers <-> queries
// In both cases the probabilities leave the MFMA accumulators as the B operand of the next
// product (the contraction index is the accumulator's row index), so P never goes through LDS.
// The accumulator rows a lane holds come in groups of four consecutive indices, which is exactly
// what the LDS transpose read (ds_read_b64_tr_b16) returns, so the A operands of those second
// products (V^T, K^T, dO^T, Q^T) are read straight from the row-major tiles.
//
// One swizzle serves plain 16-byte fragment reads and transpose reads of the same tile:
// chunk c of row r is stored at c ^ f(r), f chosen so that 16 consecutive rows (plain reads) and
// 4 consecutive rows x 64 bytes (transpose reads) both cover all banks.
#include <algorithm>
#include <atomic>

#include "bp_kernels.h"
#include "bp_device.h"
#include "bp_attn_rows.h"
#include "bp_tile.h"

namespace bp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// bare v_exp_f32: arguments here are <= 8 and anything below -126 may flush to zero
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Head dimensions below the tile width D (any multiple of 8: 40 -> 64, 96 -> 128): the tile columns
// at and beyond the real width dr are filled from this chunk of zeros and the register fragments
// get zeros there, so the padded part contributes nothing; products that only touch padded columns
// are skipped, and padded output columns are never stored.
__device__ __attribute__((aligned(16))) unsigned int g_zero_chunk[4] = {0u, 0u, 0u, 0u};

// An empty asm that keeps a wave-uniform condition a branch: left alone the compiler turns masking loops into one
// branch per element (forward, dQ) or into a compare and a select per element of every tile (dK/dV).  With the
// statistics of a dK/dV tile scaled once per row: forward, S 6144, 16 heads of 64, causal 122 -> 110 us, backward
// 345 -> 312 us; S 2048, 16 heads of 128 36 -> 34, 118 -> 109 us.
__device__ __forceinline__ void stay_a_branch() { asm volatile(""); }

// 8 consecutive elements of a row starting at column `col`, zeros at and beyond column dr
__device__ __forceinline__ bf16x8 load_frag(const bf16_t* row, int col, int dr) {
    bf16x8 z;
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = (bf16_t)0.f;
    return col < dr ? *reinterpret_cast<const bf16x8*>(row + col) : z;
}

// ---- tile layout: [rows][D] bf16, 16-byte chunks XOR-swizzled by row
template <int D> __device__ __forceinline__ int swz(int row) {
    return D == 128 ? (((row & 3) << 2) | ((row >> 2) & 3))
                    : ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));
}
template <int D> __device__ __forceinline__ int tile_off(int row, int chunk) {
    return row * (D * 2) + ((chunk ^ swz<D>(row)) << 4);
}

// Direct global->LDS copy of a [64][D] tile by NW waves.  Which 16-byte chunk a lane fetches
// depends only on its position, so the per-lane source offsets are computed once per kernel and a
// step only adds the tile's base address.  dr is the real row width; with PAD, chunks beyond it come
// from zeros.  A tile that reaches past the last row of its sequence is requested with issue_rows,
// which takes the rows beyond the valid ones from the same zeros.
template <int D, int NW, bool PAD>
struct TilePlan {
    static constexpr int CPR = D / 8;              // chunks per row
    static constexpr int NI = 64 * CPR / 64 / NW;  // wave instructions per wave
    static constexpr int ROWSTEP = NW * 64 / CPR;  // rows between a lane's consecutive chunks: a multiple
                                                   // of 16, the period of the swizzle, so the column stays
    int off0;                                      // element offset of the first chunk; < 0: padded column
    int ld;                                        // row pitch in elements (wave-uniform)
    int row0;                                      // row of the first chunk
    __device__ __forceinline__ void init(int wave, int lane, int ld_, int dr) {
        const int P = wave * 64 + lane;
        const int row = P / CPR;
        const int c = (P % CPR) ^ swz<D>(row);
        ld = ld_;
        row0 = row;
        off0 = (!PAD || c * 8 < dr) ? row * ld + c * 8 : -1;
    }
    // gbase points at (row 0, col 0) of the tile
    __device__ __forceinline__ void issue(const bf16_t* gbase, char* lds, int wave) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const bf16_t* src = (!PAD || off0 >= 0) ? gbase + (size_t)i * ROWSTEP * ld + off0
                                                    : (const bf16_t*)g_zero_chunk;
            __builtin_amdgcn_global_load_lds(
                (const void __attribute__((address_space(1)))*)src,
                (void __attribute__((address_space(3)))*)(lds + (wave + NW * i) * 1024), 16, 0, 0);
        }
    }
    // the same with only the first `rows` rows of the tile inside the tensor
    __device__ __forceinline__ void issue_rows(const bf16_t* gbase, char* lds, int wave, int rows) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const bool ok = (!PAD || off0 >= 0) && row0 + i * ROWSTEP < rows;
            const bf16_t* src = ok ? gbase + (size_t)i * ROWSTEP * ld + off0 : (const bf16_t*)g_zero_chunk;
            __builtin_amdgcn_global_load_lds(
                (const void __attribute__((address_space(1)))*)src,
                (void __attribute__((address_space(3)))*)(lds + (wave + NW * i) * 1024), 16, 0, 0);
        }
    }
};

// plain fragment: 8 consecutive columns (k16 step s, half h) of row (row0 + lane%32)
template <int D>
__device__ __forceinline__ bf16x8 frag_rows(const char* lds, int row0, int s, int lane) {
    return *reinterpret_cast<const bf16x8*>(lds + tile_off<D>(row0 + (lane & 31), 2 * s + (lane >> 5)));
}
// transposed fragment for a product whose contraction runs over the tile's rows: lane gets, for
// column (col0 + lane%32), the rows {r0 + 4h .. +3} and {r0 + 8 + 4h .. +3} (h = lane/32): the
// row order in which a 32x32 accumulator hands its 16 rows to the next MFMA.
template <int D>
__device__ __forceinline__ bf16x8 frag_cols(const char* lds, int r0, int col0, int lane) {
    const int i = lane & 15, g2 = (lane >> 4) & 1, h = lane >> 5;
    const int col = col0 + 16 * g2 + 4 * (i & 3);
    const int chunk = col >> 3, byte = (col & 7) * 2;
    const int ra = r0 + 4 * h + (i >> 2);
    s16x4 lo = lds_read_tr((const lds_s16x4*)(lds + tile_off<D>(ra, chunk) + byte));
    s16x4 hi = lds_read_tr((const lds_s16x4*)(lds + tile_off<D>(ra + 8, chunk) + byte));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// accumulator registers 8*half .. 8*half+7 of a 32x32 tile as a bf16 B operand
__device__ __forceinline__ bf16x8 acc_to_b(const f32x16& a, int half) {
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (bf16_t)a[8 * half + e];
    return r;
}

// The same registers as three bf16 operands whose sum they are: 24 significant bits cut into 8 + 8 + 8.
struct Split8 { bf16x8 part[3]; };
__device__ __forceinline__ Split8 acc_to_b3(const f32x16& a, int half) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    float r[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = a[8 * half + e];
    Split8 o;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        u32x4 w;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const uint32_t u0 = __builtin_bit_cast(uint32_t, r[e]), u1 = __builtin_bit_cast(uint32_t, r[e + 1]);
            w[e / 2] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);      // the upper halves of both
            r[e] -= __builtin_bit_cast(float, u0 & 0xffff0000u);        // exact
            r[e + 1] -= __builtin_bit_cast(float, u1 & 0xffff0000u);
        }
        o.part[i] = __builtin_bit_cast(bf16x8, w);
    }
    return o;
}

// out^T (D x 32) += tile[row0 .. row0 + 31]^T x, x as a score accumulator holds it (P or dS).  EXACT keeps x in
// fp32: three products with its bf16 parts, the smallest first, in place of one with its rounded value.
template <int D, int DT, bool EXACT>
__device__ __forceinline__ void contract(const char* tile, int row0, int lane, int dr, const f32x16& x, f32x16 (&out)[DT]) {
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
        if constexpr (EXACT) {
            const Split8 xb = acc_to_b3(x, s2);
#pragma unroll
            for (int t2 = 0; t2 < DT; ++t2) {
                if (32 * t2 >= dr) continue;
                const bf16x8 f = frag_cols<D>(tile, row0 + 16 * s2, t2 * 32, lane);
#pragma unroll
                for (int i = 2; i >= 0; --i)
                    out[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, xb.part[i], out[t2], 0, 0, 0);
            }
        } else {
            const bf16x8 xb = acc_to_b(x, s2);
#pragma unroll
            for (int t2 = 0; t2 < DT; ++t2)
                if (32 * t2 < dr)
                    out[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        frag_cols<D>(tile, row0 + 16 * s2, t2 * 32, lane), xb, out[t2], 0, 0, 0);
        }
    }
}

// row index inside a 32-row accumulator tile held in register v by a lane of half h
__device__ __forceinline__ int acc_row(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }

// no NaN and no infinity in rows row0 .. row0 + 31 of a tile (the same answer in every lane)
template <int D>
__device__ __forceinline__ bool rows_finite(const char* tile, int row0, int lane, int dr) {
    typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
    u16x8 top = (u16x8)(unsigned short)0;
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
        if (16 * s < dr)
            top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x8, frag_rows<D>(tile, row0, s, lane)) &
                                                     (u16x8)(unsigned short)0x7fff);
    bool ok = true;
#pragma unroll
    for (int e = 0; e < 8; ++e) ok = ok && top[e] < 0x7f80;
    return __builtin_amdgcn_ballot_w64(!ok) == 0;
}

// Which block of rows (queries or keys) of which head a launched block takes.  Under a causal mask the blocks of a
// head differ in work, and the position of a block in the launch counts:
//   ORDER_FOLDED: the first half of the positions walks from the most expensive block down, the second half from the
//     cheapest up, so that two blocks that share a CU add up to the same everywhere; else heaviest first, which lets
//     the hardware hand the light blocks to whichever CU finishes first;
//   ORDER_ALL: positions run over all batch entries together, else over one entry after the other, which keeps fewer
//     heads' keys and values in the L2s at a time but pairs heavy blocks of one entry with heavy ones of another.
enum { ORDER_FOLDED = 1, ORDER_ALL = 2 };
__device__ __forceinline__ void block_coords(int bid, int nblk, int heads, int batch, bool causal, bool heavy_is_last_index,
                                            int order, int& blk, int& head, int& b) {
    const int per = nblk * heads;             // blocks per batch entry
    int i;                                    // position in the work-sorted order
    if (causal && (order & ORDER_ALL)) {
        i = bid / (heads * batch);
        const int r = bid - i * (heads * batch);
        b = r / heads;
        head = r - b * heads;
    } else {
        const int lin = bid % per;
        b = bid / per;
        i = lin / heads;
        head = lin % heads;
    }
    if (causal) {
        const int half = (nblk + 1) / 2;
        const int rank = !(order & ORDER_FOLDED) ? i : i < half ? i : nblk - 1 - (i - half);      // 0 = heaviest
        blk = heavy_is_last_index ? nblk - 1 - rank : rank;
    } else {
        blk = i;
    }
}

// =====================================================================================
// Forward.  Block = 64 queries = 2 groups of 32 queries x (2 NT) sub-ranges of 32 keys: a step
// covers NT tiles of 64 keys and every wave takes one half of one tile, keeping its own
// online-softmax state; the sub-ranges are merged through LDS at the end.  NT = 1: 4 waves, 64 KB
// (D = 128) of LDS, two blocks per CU.  NT = 2: 8 waves, 128 KB, one block per CU: the heaviest
// causal block then needs half as many steps, and because blocks are dealt out heaviest first
// as CUs become free the tail of the launch stays short.
// WIDE: block = 128 queries, a wave takes 32 of them and both halves of every tile, so nothing is merged and a tile
// is loaded for twice as many products: for launches with enough blocks (wide_rows).
// =====================================================================================
// RAG: the sequence length is not a multiple of 64.  The last query block and the last key tile are
// then partly filled: tile rows of keys past the end, or past the sequence's valid length, are zeros
// (what padding holds must not reach the products: zero times NaN), such keys are masked, queries past
// the end repeat the last one and are not stored.  (The guards cost a branch per
// tile, so multiples of 64 keep kernels without them.  Before, such lengths went to the kernels of
// one row per block: 8 micro-batches of 2 layers with H = 1600, S = 1000, B = 1: 46.7 ms, now 16.0 ms.
// Those kernels kept P and dS in fp32, and these lengths still do: each goes into the second product as three
// bf16 parts that add up to it exactly.  Against one product with the rounded value: forward B 3, S 2550,
// 12 heads of 64, causal 55 -> 79 us, backward B 2, S 1058, 32 heads of 128 237 -> 340 us, 5 - 20 % below S 300;
// the kernels of one row per block take ten times as long.)
template <int D, int DR, int NT, bool RAG, bool WIDE = false>
__global__ __launch_bounds__(256 * NT, NT == 1 ? 2 : 1) void attn_fwd_mfma_kernel(AttnArgs a, float scale, int order) {
    static_assert(!WIDE || (NT == 1 && !RAG), "128 queries: one tile a step, whole tiles");
    attn_args_now(a, scale, order);
    constexpr int NW = 4 * NT, NSUB = WIDE ? 1 : 2 * NT, KS = D / 16, DT = D / 32;
    constexpr int QB = WIDE ? 128 : 64, NH = WIDE ? 2 : 1;      // queries of a block; halves of a tile that a wave takes
    constexpr int TILE = 64 * D * 2, STAGE = NT * 2 * TILE;   // per tile: K then V
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qg = wave / NSUB, sub = wave % NSUB;      // query group; (tile of the step, half of the tile)
    const int tj = sub >> 1, kh = sub & 1;
    const int h = lane >> 5;
    int qblk, head, b;
    block_coords(blockIdx.x, (a.S + QB - 1) / QB, a.heads, a.B, a.causal != 0, true, order, qblk, head, b);
    // real head dimension: the tile width (no padding, every guard below folds away), a fixed narrower
    // width (the guards fold to constants), or with DR = 0 whatever the call says
    constexpr bool PAD = DR != D;
    const int dr = DR ? DR : a.d;
    const int H = a.heads * dr, ld = 3 * H;
    const bf16_t* qkv = (const bf16_t*)a.qkv + (size_t)b * a.S * ld + head * dr;
    const bf16_t* kbase = qkv + H;
    const bf16_t* vbase = qkv + 2 * H;
    const int q_wave = qblk * QB + qg * 32;
    const int q_lane = q_wave + (lane & 31);
    const int klen = a.causal ? a.S : (a.lens ? a.lens[b] : a.S);
    const int kend = a.causal ? (RAG || WIDE ? min(qblk * QB + QB, a.S) : qblk * QB + QB) : klen;   // keys [0, kend) matter to this block
    const int nt = (kend + 63) / 64;                        // tiles
    const int nsteps = (nt + NT - 1) / NT;
    const float c = scale * kLog2e;

    bf16x8 qf[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
        qf[s] = load_frag(qkv + (size_t)(RAG || WIDE ? min(q_lane, a.S - 1) : q_lane) * ld, 16 * s + 8 * h, dr);

    f32x16 ot[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) ot[t][v] = 0.f;
    float m = -INFINITY, lsum = 0.f;
    bool by_rows = false;       // a value on the diagonal is not finite: see bp_attn_rows.h

    TilePlan<D, NW, PAD> plan;
    plan.init(wave, lane, ld, dr);
    auto request = [&](int step, char* st) {             // the NT tiles of a step (those that exist)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int k0 = (step * NT + j) * 64;
            if (step * NT + j < nt) {
                if (RAG && k0 + 64 > klen) {
                    plan.issue_rows(kbase + (size_t)k0 * ld, st + j * 2 * TILE, wave, klen - k0);
                    plan.issue_rows(vbase + (size_t)k0 * ld, st + j * 2 * TILE + TILE, wave, klen - k0);
                    continue;
                }
                plan.issue(kbase + (size_t)k0 * ld, st + j * 2 * TILE, wave);
                plan.issue(vbase + (size_t)k0 * ld, st + j * 2 * TILE + TILE, wave);
            }
        }
    };
    request(0, smem);

    for (int t = 0; t < nsteps; ++t) {
        BP_WAIT_VMCNT(0);
        __syncthreads();
        if (t + 1 < nsteps) request(t + 1, smem + ((t + 1) & 1) * STAGE);
        const int tile = t * NT + tj;
        const int kw = tile * 64 + 32 * kh;             // first key of this wave's sub-range
        if (tile >= nt || (a.causal && kw > q_wave + 31) || kw >= klen) continue;   // nothing unmasked for this wave
        if (WIDE && q_wave >= a.S) continue;                        // the second half of the last block: no queries
        const char* sk = smem + (t & 1) * STAGE + tj * 2 * TILE;
        const char* sv = sk + TILE;

        // S^T (32 keys x 32 queries), of both halves of the tile in a wide block
        f32x16 st2[NH];
#pragma unroll
        for (int u = 0; u < NH; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) st2[u][v] = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            if (16 * s < dr)
#pragma unroll
                for (int u = 0; u < NH; ++u)
                    st2[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<D>(sk, 32 * (kh + u), s, lane), qf[s], st2[u], 0, 0, 0);
        if ((a.causal && kw + 32 * NH - 1 > q_wave) || kw + 32 * NH > klen) {     // the diagonal, or padded keys
            stay_a_branch();
            const int last = a.causal ? min(q_lane, klen - 1) : klen - 1;     // last key this query attends
#pragma unroll
            for (int u = 0; u < NH; ++u)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (kw + 32 * u + acc_row(v, h) > last) st2[u][v] = -INFINITY;
        }
        float mx = st2[0][0];
#pragma unroll
        for (int u = 0; u < NH; ++u)
#pragma unroll
            for (int v = u == 0; v < 16; ++v) mx = fmaxf(mx, st2[u][v]);
        mx = halves_max(mx) * c;     // c > 0: the maximum commutes with the scaling
        // The reference point m of the running softmax only has to stay within a bounded distance of
        // the true maximum: it moves (and O, l are rescaled) only when some query of the wave sees a
        // score more than 8 binary orders above it, so p <= 2^8 and most tiles skip the rescaling.
        if (__builtin_amdgcn_ballot_w64(mx > m + 8.f) != 0) {
            const float m_new = fmaxf(m, mx);
            const float alpha = m == -INFINITY ? 0.f : fast_exp2(m - m_new);
            m = m_new;
            lsum *= alpha;
#pragma unroll
            for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
                for (int v = 0; v < 16; ++v) ot[t2][v] *= alpha;
        }
        // a row whose keys are all masked so far keeps m = -inf; avoid inf - inf
        const float m_use = m == -INFINITY ? 0.f : m;
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            float ps = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float p = fast_exp2(__builtin_fmaf(st2[u][v], c, -m_use));
                st2[u][v] = p;
                ps += p;
            }
            lsum += ps;
        }
        // O^T (D x 32 queries) += V^T P^T over this wave's keys
        if (RAG && a.causal && kw + 31 > q_wave && !rows_finite<D>(sv, 32 * kh, lane, dr)) by_rows = true;
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            // (a half that is masked throughout contributes nothing, whatever its values are)
            if (u && ((a.causal && kw + 32 > q_wave + 31) || kw + 32 >= klen)) break;
            contract<D, DT, RAG>(sv, 32 * (kh + u), lane, dr, st2[u], ot);
        }
    }
    if (RAG && a.causal && any_wave(by_rows, smem)) {
        for (int q = qblk * 64; q < min(qblk * 64 + 64, a.S); ++q) attn_fwd_row<bf16_t>(a, scale, q, head, b, (float*)smem);
        return;
    }

    // merge the key sub-ranges: waves 1 .. NSUB-1 of a query group hand (m, l, O^T) to wave 0 through LDS
    float l = halves_sum(lsum), mm = m;
    if constexpr (!WIDE) {
        __syncthreads();                                    // all tile reads are over; LDS is free
        constexpr int XO = DT * 16 * 64 + 128;              // [DT*16][64 lanes] + m[64] + l[64]
        float* xo = (float*)smem + (size_t)qg * (NSUB - 1) * XO;
        if (sub != 0) {
            float* mine = xo + (size_t)(sub - 1) * XO;
#pragma unroll
            for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
                for (int v = 0; v < 16; ++v) mine[(t2 * 16 + v) * 64 + lane] = ot[t2][v];
            mine[DT * 16 * 64 + lane] = m;
            mine[DT * 16 * 64 + 64 + lane] = l;
        }
        __syncthreads();
        if (sub != 0) return;
        // (m is finite: key 0 lies in this wave's sub-range)
#pragma unroll
        for (int j = 0; j < NSUB - 1; ++j) mm = fmaxf(mm, xo[(size_t)j * XO + DT * 16 * 64 + lane]);
        const float a0 = fast_exp2(m - mm);
        l *= a0;
#pragma unroll
        for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
            for (int v = 0; v < 16; ++v) ot[t2][v] *= a0;
#pragma unroll
        for (int j = 0; j < NSUB - 1; ++j) {
            const float* other = xo + (size_t)j * XO;
            const float aj = fast_exp2(other[DT * 16 * 64 + lane] - mm);
            l += other[DT * 16 * 64 + 64 + lane] * aj;
#pragma unroll
            for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
                for (int v = 0; v < 16; ++v) ot[t2][v] += other[(t2 * 16 + v) * 64 + lane] * aj;
        }
    }
    if ((RAG || WIDE) && q_lane >= a.S) return;
    const float inv = 1.f / l;
    bf16_t* out = (bf16_t*)a.ctx + ((size_t)b * a.S + q_lane) * H + head * dr;
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint2 pk;
            pk.x = pack_bf16x2(ot[t2][4 * g] * inv, ot[t2][4 * g + 1] * inv);
            pk.y = pack_bf16x2(ot[t2][4 * g + 2] * inv, ot[t2][4 * g + 3] * inv);
            if (t2 * 32 + 8 * g + 4 * h < dr) *reinterpret_cast<uint2*>(out + t2 * 32 + 8 * g + 4 * h) = pk;
        }
    if (h == 0) a.lse[((size_t)b * a.heads + head) * a.S + q_lane] = (mm + log2f(l)) * kLn2;
}

// =====================================================================================
// Backward, part 1: dQ (and delta[q] = sum_d dO[q][d] O[q][d], kept for part 2).  Same decomposition as the forward (lane <-> query, two key halves):
//   S^T = K Q^T, P^T = exp(S^T - lse), dP^T = V dO^T, dS^T = P^T (dP^T - delta),
//   dQ^T (D x 32) += K^T dS^T         (K tile read plainly for S^T and transposed for dQ^T)
// The two halves' partial dQ^T are added through LDS at the end.
// =====================================================================================
template <int D, int DR, bool RAG, bool WIDE>
__device__ __forceinline__ void attn_bwd_dq_block(const AttnArgs& a, float scale, int order, int bid, char* smem) {
    static_assert(!WIDE || !RAG, "128 queries: whole tiles");
    constexpr int QB = WIDE ? 128 : 64;                 // queries of a block
    constexpr int NW = 4, KS = D / 16, DT = D / 32;
    constexpr int TILE = 64 * D * 2, STAGE = 2 * TILE;
    // dP - delta: -delta is what the accumulators of dP start from, where 16 registers are left for it
    constexpr bool DELTA_FIRST = !(RAG && D == 128);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qg = WIDE ? wave : wave >> 1, kh0 = WIDE ? 0 : wave & 1;
    const int h = lane >> 5;
    int qblk, head, b;
    block_coords(bid, (a.S + QB - 1) / QB, a.heads, a.B, a.causal != 0, true, order, qblk, head, b);
    // real head dimension: the tile width (no padding, every guard below folds away), a fixed narrower
    // width (the guards fold to constants), or with DR = 0 whatever the call says
    constexpr bool PAD = DR != D;
    const int dr = DR ? DR : a.d;
    const int H = a.heads * dr, ld = 3 * H;
    const bf16_t* qkv = (const bf16_t*)a.qkv + (size_t)b * a.S * ld + head * dr;
    const bf16_t* kbase = qkv + H;
    const bf16_t* vbase = qkv + 2 * H;
    const int q_wave = qblk * QB + qg * 32;
    const int q_lane = q_wave + (lane & 31);
    const int klen = a.causal ? a.S : (a.lens ? a.lens[b] : a.S);
    const int kend = a.causal ? (RAG || WIDE ? min(qblk * QB + QB, a.S) : qblk * QB + QB) : klen;
    const int nt = (kend + 63) / 64;
    const float c = scale * kLog2e;

    const int q_src = RAG || WIDE ? min(q_lane, a.S - 1) : q_lane;     // row this lane reads
    const bf16_t* dob = (const bf16_t*)a.dctx + ((size_t)b * a.S + q_src) * H + head * dr;
    bf16x8 qf[KS], dof[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        qf[s] = load_frag(qkv + (size_t)q_src * ld, 16 * s + 8 * h, dr);
        dof[s] = load_frag(dob, 16 * s + 8 * h, dr);
    }
    const size_t li = ((size_t)b * a.heads + head) * a.S + q_src;
    const float lse2 = a.lse[li] * kLog2e;
    // delta[q] = sum_d dO[q][d] O[q][d]: each lane holds half of its query's dO row already; the
    // value is also left in a.delta for the dK/dV kernel, which runs after this one
    float delta = 0.f;
    {
        const bf16_t* ob = (const bf16_t*)a.ctx + ((size_t)b * a.S + q_src) * H + head * dr;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const bf16x8 of = load_frag(ob, 16 * s + 8 * h, dr);
#pragma unroll
            for (int e = 0; e < 8; ++e) delta += (float)of[e] * (float)dof[s][e];
        }
        delta = halves_sum(delta);
        if (kh0 == 0 && h == 0 && (!(RAG || WIDE) || q_lane < a.S)) a.delta[li] = delta;
    }

    f32x16 dq[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) dq[t][v] = 0.f;
    bool by_rows = false;       // a key or value on the diagonal is not finite

    TilePlan<D, NW, PAD> plan;
    plan.init(wave, lane, ld, dr);
    auto request = [&](int k0, char* st) {
        if (RAG && k0 + 64 > klen) {
            plan.issue_rows(kbase + (size_t)k0 * ld, st, wave, klen - k0);
            plan.issue_rows(vbase + (size_t)k0 * ld, st + TILE, wave, klen - k0);
            return;
        }
        plan.issue(kbase + (size_t)k0 * ld, st, wave);
        plan.issue(vbase + (size_t)k0 * ld, st + TILE, wave);
    };
    if (nt > 0) request(0, smem);

    for (int t = 0; t < nt; ++t) {
        const int k0 = t * 64;
        BP_WAIT_VMCNT(0);
        __syncthreads();
        if (t + 1 < nt) request(k0 + 64, smem + ((t + 1) & 1) * STAGE);
        if (WIDE && q_wave >= a.S) continue;            // the second half of the last block: no queries
        const char* sk = smem + (t & 1) * STAGE;
        const char* sv = sk + TILE;
#pragma unroll
        for (int kh = kh0; kh < (WIDE ? 2 : kh0 + 1); ++kh) {
            const int kw = k0 + 32 * kh;
            if ((a.causal && kw > q_wave + 31) || kw >= klen) break;
            // (a value that is not finite makes dP of the queries that do not attend it NaN)
            if (RAG && a.causal && kw + 31 > q_wave &&
                (!rows_finite<D>(sk, 32 * kh, lane, dr) || !rows_finite<D>(sv, 32 * kh, lane, dr))) by_rows = true;
            f32x16 sacc, dp;
#pragma unroll
            for (int v = 0; v < 16; ++v) { sacc[v] = 0.f; dp[v] = DELTA_FIRST ? -delta : 0.f; }
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (16 * s >= dr) continue;
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<D>(sk, 32 * kh, s, lane), qf[s], sacc, 0, 0, 0);
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<D>(sv, 32 * kh, s, lane), dof[s], dp, 0, 0, 0);
            }
            if ((a.causal && kw + 31 > q_wave) || kw + 32 > klen) {     // the diagonal, or padded keys: p = 0
                stay_a_branch();
                const int last = a.causal ? min(q_lane, klen - 1) : klen - 1;     // last key this query attends
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (kw + acc_row(v, h) > last) sacc[v] = -INFINITY;
            }
#pragma unroll
            for (int v = 0; v < 16; ++v)
                dp[v] = fast_exp2(__builtin_fmaf(sacc[v], c, -lse2)) * (DELTA_FIRST ? dp[v] : dp[v] - delta);   // dS^T
            contract<D, DT, RAG>(sk, 32 * kh, lane, dr, dp, dq);
        }
    }
    if (RAG && a.causal && any_wave(by_rows, smem)) {
        for (int q = qblk * 64; q < min(qblk * 64 + 64, a.S); ++q) attn_bwd_dq_row<bf16_t>(a, scale, q, head, b, (float*)smem);
        return;
    }
    if (WIDE && q_lane >= a.S) return;
    float* xo = (float*)smem + (WIDE ? 0 : qg * (DT * 16 * 64));
    if constexpr (!WIDE) {
        __syncthreads();
        if (kh0 == 1) {
#pragma unroll
            for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
                for (int v = 0; v < 16; ++v) xo[(t2 * 16 + v) * 64 + lane] = dq[t2][v];
        }
        __syncthreads();
        if (kh0 == 1 || (RAG && q_lane >= a.S)) return;
    }
    bf16_t* out = (bf16_t*)a.dqkv + ((size_t)b * a.S + q_lane) * ld + head * dr;
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            float o4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o4[e] = (WIDE ? dq[t2][4 * g + e] : dq[t2][4 * g + e] + xo[(t2 * 16 + 4 * g + e) * 64 + lane]) * scale;
            uint2 pk;
            pk.x = pack_bf16x2(o4[0], o4[1]);
            pk.y = pack_bf16x2(o4[2], o4[3]);
            if (t2 * 32 + 8 * g + 4 * h < dr) *reinterpret_cast<uint2*>(out + t2 * 32 + 8 * g + 4 * h) = pk;
        }
}

// =====================================================================================
// Backward, part 2: dK and dV.  Block = 4 waves = 2 groups of 32 keys x 2 halves of every
// 64-query tile of Q / dO that streams by.
//   S = Q K^T (lane <-> key), P = exp(S - lse[q]), dP = dO V^T, dS = P (dP - delta[q]),
//   dV^T (D x 32 keys) += dO^T P,   dK^T (D x 32 keys) += Q^T dS
// The two query halves' partial sums are added through LDS at the end.
// =====================================================================================
template <int D, int DR, bool RAG, bool WIDE, bool ALONE>
__device__ __forceinline__ void attn_bwd_dkv_block(const AttnArgs& a, float scale, int order, int bid, char* smem) {
    static_assert(!WIDE || (!RAG && ALONE), "128 keys: whole tiles, a launch of their own");
    constexpr int KB = WIDE ? 128 : 64;                 // keys of a block
    constexpr int NW = 4, KS = D / 16, DT = D / 32;
    constexpr int TILE = 64 * D * 2, STAGE = 2 * TILE + 512;   // Q, dO, then lse[64], delta[64]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = WIDE ? wave : wave >> 1, qh0 = WIDE ? 0 : wave & 1;
    const int h = lane >> 5;
    int kblk, head, b;
    block_coords(bid, (a.S + KB - 1) / KB, a.heads, a.B, a.causal != 0, false, order, kblk, head, b);   // key block 0 is the heaviest
    // real head dimension: the tile width (no padding, every guard below folds away), a fixed narrower
    // width (the guards fold to constants), or with DR = 0 whatever the call says
    constexpr bool PAD = DR != D;
    const int dr = DR ? DR : a.d;
    const int H = a.heads * dr, ld = 3 * H;
    const bf16_t* qkv = (const bf16_t*)a.qkv + (size_t)b * a.S * ld + head * dr;
    const bf16_t* dobase = (const bf16_t*)a.dctx + (size_t)b * a.S * H + head * dr;
    const int k_wave = kblk * KB + kg * 32;
    const int k_lane = k_wave + (lane & 31);
    const int klen = a.causal ? a.S : (a.lens ? a.lens[b] : a.S);
    bf16_t* dk_out = (bf16_t*)a.dqkv + ((size_t)b * a.S + k_lane) * ld + H + head * dr;
    bf16_t* dv_out = dk_out + H;
    if (kblk * KB >= klen) {      // the whole block of keys is padding: no query attends it
        if (qh0 == 0 && (!(RAG || WIDE) || k_lane < a.S)) {
            const uint2 z = make_uint2(0u, 0u);
#pragma unroll
            for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    if (t2 * 32 + 8 * g + 4 * h >= dr) continue;
                    *reinterpret_cast<uint2*>(dk_out + t2 * 32 + 8 * g + 4 * h) = z;
                    *reinterpret_cast<uint2*>(dv_out + t2 * 32 + 8 * g + 4 * h) = z;
                }
        }
        return;
    }
    const float c = scale * kLog2e;
    const float* lse = a.lse + ((size_t)b * a.heads + head) * a.S;
    const float* dlt = a.delta + ((size_t)b * a.heads + head) * a.S;

    const int k_src = RAG || WIDE ? min(k_lane, RAG ? klen - 1 : a.S - 1) : k_lane;     // row this lane reads (its own, unless it is padding)
    bf16x8 kf[KS], vf[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        kf[s] = load_frag(qkv + H + (size_t)k_src * ld, 16 * s + 8 * h, dr);
        vf[s] = load_frag(qkv + 2 * H + (size_t)k_src * ld, 16 * s + 8 * h, dr);
    }
    f32x16 dk[DT], dv[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) { dk[t][v] = 0.f; dv[t][v] = 0.f; }

    bool by_rows = false;       // a query on the diagonal is not finite
    const bool some_padded = (WIDE ? k_wave + 32 : kblk * 64 + 64) > klen;   // some of this wave's (block's) keys are padding
    const int t0 = a.causal ? kblk * (KB / 64) : 0;        // first 64-query tile that can see this block's keys
    const int nt = (a.S + 63) / 64;

    TilePlan<D, NW, PAD> plan_q, plan_do;
    plan_q.init(wave, lane, ld, dr);
    plan_do.init(wave, lane, H, dr);
    auto load_stage = [&](int t, char* st) {
        const int q0 = t * 64;
        if (RAG && q0 + 64 > a.S) {
            plan_q.issue_rows(qkv + (size_t)q0 * ld, st, wave, a.S - q0);
            plan_do.issue_rows(dobase + (size_t)q0 * H, st + TILE, wave, a.S - q0);
        } else {
            plan_q.issue(qkv + (size_t)q0 * ld, st, wave);
            plan_do.issue(dobase + (size_t)q0 * H, st + TILE, wave);
        }
    };
    // The 64 log-sum-exp values (wave 0) and 64 deltas (wave 1) of a tile go through registers, where they get the
    // sign and the base that the exponential and the accumulators want: once per row instead of once per element.
    // They are fetched two tiles ahead, so that nothing waits for them but the wait at the top of a step.
    const float* stat = wave == 0 ? lse : dlt;
    const float stat_factor = wave == 0 ? -kLog2e : -1.f;
    const int stats = ALONE ? 2 : 1;                     // waves with statistics to fetch
    auto fetch_stat = [&](int t) { return wave < stats && t < nt ? stat[RAG ? min(t * 64 + lane, a.S - 1) : t * 64 + lane] : 0.f; };
    auto put_stat = [&](float v, char* st) {
        if (wave < stats) ((float*)(st + 2 * TILE))[wave * 64 + lane] = v * stat_factor;
    };
    // Beside the dQ blocks, which leave delta in memory too late for this launch, a block takes delta of a tile's rows
    // from O and dO itself, four lanes to a row; the loads are made when the tile is requested and used a step later.
    constexpr int NO = D / 32;
    bf16x8 o_row[ALONE ? 1 : NO], do_row[ALONE ? 1 : NO];
    auto fetch_delta = [&](int t) {
        if constexpr (!ALONE) {
            if (t >= nt) return;
            const size_t row = (size_t)b * a.S + (RAG ? min(t * 64 + (int)(threadIdx.x >> 2), a.S - 1) : t * 64 + (int)(threadIdx.x >> 2));
            const bf16_t* ob = (const bf16_t*)a.ctx + row * H + head * dr;
            const bf16_t* gb = (const bf16_t*)a.dctx + row * H + head * dr;
#pragma unroll
            for (int j = 0; j < NO; ++j) {
                o_row[j] = load_frag(ob, 32 * j + 8 * (threadIdx.x & 3), dr);
                do_row[j] = load_frag(gb, 32 * j + 8 * (threadIdx.x & 3), dr);
            }
        }
    };
    auto put_delta = [&](int t, char* st) {
        if constexpr (!ALONE) {
            if (t >= nt) return;
            float d = 0.f;
#pragma unroll
            for (int j = 0; j < NO; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) d += (float)o_row[j][e] * (float)do_row[j][e];
            d += __shfl_xor(d, 1, 64);
            d += __shfl_xor(d, 2, 64);
            if ((threadIdx.x & 3) == 0) ((float*)(st + 2 * TILE))[64 + (threadIdx.x >> 2)] = -d;
        }
    };
    fetch_delta(t0);
    const float stat_first = fetch_stat(t0);
    float stat_next = fetch_stat(t0 + 1);
    load_stage(t0, smem + (t0 & 1) * STAGE);
    put_stat(stat_first, smem + (t0 & 1) * STAGE);
    put_delta(t0, smem + (t0 & 1) * STAGE);

    for (int t = t0; t < nt; ++t) {
        const int q0 = t * 64;
        BP_WAIT_VMCNT(0);
        __syncthreads();
        if (t + 1 < nt) {
            put_stat(stat_next, smem + ((t + 1) & 1) * STAGE);
            load_stage(t + 1, smem + ((t + 1) & 1) * STAGE);
            stat_next = fetch_stat(t + 2);
            fetch_delta(t + 1);
        }
        if (WIDE && k_wave >= klen) continue;            // none of this wave's keys exists, or is attended
        const char* sq = smem + (t & 1) * STAGE;
        const char* sdo = sq + TILE;
#pragma unroll
        for (int qh = qh0; qh < (WIDE ? 2 : qh0 + 1); ++qh) {
            const int qw = q0 + 32 * qh;                     // first query of this wave's half
            if (a.causal && qw + 31 < k_wave) continue;      // no query of this half reaches this wave's keys
            const float* s_nlse = (const float*)(sq + 2 * TILE) + 32 * qh;
            const float* s_ndlt = (const float*)(sq + 2 * TILE) + 64 + 32 * qh;
            const bool need_mask = a.causal && qw < k_wave + 31;
            if (RAG && need_mask && (!rows_finite<D>(sq, 32 * qh, lane, dr) || !rows_finite<D>(sdo, 32 * qh, lane, dr) ||
                                     !stats_finite(s_nlse, s_ndlt, lane))) by_rows = true;
            f32x16 sacc, dp;
#pragma unroll
            for (int v = 0; v < 16; ++v) { sacc[v] = 0.f; dp[v] = s_ndlt[acc_row(v, h)]; }
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (16 * s >= dr) continue;
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<D>(sq, 32 * qh, s, lane), kf[s], sacc, 0, 0, 0);
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<D>(sdo, 32 * qh, s, lane), vf[s], dp, 0, 0, 0);
            }
            // masked scores become -inf before the exponential (p = 0, dS = 0); both conditions are
            // wave-uniform branches, taken only on the diagonal tile and in a block with padded keys
            if (need_mask) {
                stay_a_branch();
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (k_lane > qw + acc_row(v, h)) sacc[v] = -INFINITY;
            }
            if (RAG && q0 + 64 > a.S) {                      // queries past the end: p = 0
                stay_a_branch();
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (qw + acc_row(v, h) >= a.S) sacc[v] = -INFINITY;
            }
            if (some_padded) {
                stay_a_branch();
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (k_lane >= klen) sacc[v] = -INFINITY;
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                sacc[v] = fast_exp2(__builtin_fmaf(sacc[v], c, s_nlse[acc_row(v, h)]));      // P
                dp[v] *= sacc[v];                                                            // dS = P (dP - delta)
            }
            if constexpr (RAG) {
                contract<D, DT, true>(sdo, 32 * qh, lane, dr, sacc, dv);
                contract<D, DT, true>(sq, 32 * qh, lane, dr, dp, dk);
            } else {
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    const bf16x8 pb = acc_to_b(sacc, s2);
                    const bf16x8 db = acc_to_b(dp, s2);
#pragma unroll
                    for (int t2 = 0; t2 < DT; ++t2) {
                        if (32 * t2 >= dr) continue;
                        dv[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            frag_cols<D>(sdo, 32 * qh + 16 * s2, t2 * 32, lane), pb, dv[t2], 0, 0, 0);
                        dk[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            frag_cols<D>(sq, 32 * qh + 16 * s2, t2 * 32, lane), db, dk[t2], 0, 0, 0);
                    }
                }
            }
        }
        put_delta(t + 1, smem + ((t + 1) & 1) * STAGE);
    }
    if (RAG && a.causal && any_wave(by_rows, smem)) {
        for (int k = kblk * 64; k < min(kblk * 64 + 64, a.S); ++k) attn_bwd_dkv_row<bf16_t, !ALONE>(a, scale, k, head, b, (float*)smem);
        return;
    }
    if (WIDE && k_lane >= a.S) return;
    float* xo = (float*)smem + (WIDE ? 0 : kg * (2 * DT * 16 * 64));
    if constexpr (!WIDE) {
        __syncthreads();
        if (qh0 == 1) {
#pragma unroll
            for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    xo[(t2 * 16 + v) * 64 + lane] = dk[t2][v];
                    xo[((DT + t2) * 16 + v) * 64 + lane] = dv[t2][v];
                }
        }
        __syncthreads();
        if (qh0 == 1 || (RAG && k_lane >= a.S)) return;
    }
#pragma unroll
    for (int t2 = 0; t2 < DT; ++t2)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            float k4[4], v4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                k4[e] = (WIDE ? dk[t2][4 * g + e] : dk[t2][4 * g + e] + xo[(t2 * 16 + 4 * g + e) * 64 + lane]) * scale;
                v4[e] = WIDE ? dv[t2][4 * g + e] : dv[t2][4 * g + e] + xo[((DT + t2) * 16 + 4 * g + e) * 64 + lane];
            }
            if (t2 * 32 + 8 * g + 4 * h >= dr) continue;
            uint2 pk;
            pk.x = pack_bf16x2(k4[0], k4[1]);
            pk.y = pack_bf16x2(k4[2], k4[3]);
            *reinterpret_cast<uint2*>(dk_out + t2 * 32 + 8 * g + 4 * h) = pk;
            pk.x = pack_bf16x2(v4[0], v4[1]);
            pk.y = pack_bf16x2(v4[2], v4[3]);
            *reinterpret_cast<uint2*>(dv_out + t2 * 32 + 8 * g + 4 * h) = pk;
        }
}

template <int D, int DR, bool RAG, bool WIDE = false>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_mfma_kernel(AttnArgs a, float scale, int order) {
    attn_args_now(a, scale, order);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    attn_bwd_dq_block<D, DR, RAG, WIDE>(a, scale, order, blockIdx.x, smem);
}
template <int D, int DR, bool RAG, bool WIDE = false>
__global__ __launch_bounds__(256, 2) void attn_bwd_dkv_mfma_kernel(AttnArgs a, float scale, int order) {
    attn_args_now(a, scale, order);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    attn_bwd_dkv_block<D, DR, RAG, WIDE, true>(a, scale, order, blockIdx.x, smem);
}

// Both parts in one launch (attn_bwd_mfma_one_launch): the first half of the blocks, which have more to do, dK and dV, the others dQ.
template <int D, int DR, bool RAG>
__global__ __launch_bounds__(256, 2) void attn_bwd_mfma_kernel(AttnArgs a, float scale, int order) {
    attn_args_now(a, scale, order);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int n = gridDim.x / 2, bid = blockIdx.x;
    if (bid < n) attn_bwd_dkv_block<D, DR, RAG, false, false>(a, scale, order, bid, smem);
    else attn_bwd_dq_block<D, DR, RAG, false>(a, scale, order, bid - n, smem);
}

// ---- host side
bool attn_mfma_supported(const AttnArgs& a) {
    auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
    if (a.d % 8 || a.d < 8 || a.d > 128) return false;      // tile width 64 or 128, narrower heads are padded
    if (a.S < 1) return false;
    return al16(a.qkv) && al16(a.ctx) && (!a.dctx || al16(a.dctx)) && (!a.dqkv || al16(a.dqkv));
}

template <typename K>
static hipError_t set_smem(K kern, size_t smem) {
    if (smem <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
}

// Tiles of 64 keys per forward step.  Two (8 waves, one block per CU) halve the step count of the
// heaviest causal block, which is what bounds a launch with only a couple of blocks per CU; with
// many blocks per CU the 4-wave form with two co-resident blocks is faster.
static int tiles_per_step(const AttnArgs& a) {
    const long blocks = (long)((a.S + 63) / 64) * a.heads * a.B;
    return (a.S >= 512 && blocks <= 2L * cu_count()) ? 2 : 1;
}

// Blocks of 128 rows whose four waves take 32 rows and all 64 columns of a tile each, in place of blocks of 64 rows
// whose waves share the tile's halves: half the loads and barriers per product, nothing to merge, but half as many
// blocks.  Whole tiles only.  Narrow / wide, us, on 256 CUs:
//   forward, no mask: 16 heads, S 512, B 8 (512 wide blocks), d 64 15.7 / 14.7, d 128 24.5 / 19.8; 256 blocks, d 64
//     0.95, d 128 1.21 of the speed; B 8, S 2048, 16 heads of 128, causal 194 / 164, B 2, S 2048, 40 heads of 128 129 / 104;
//   forward, causal, d 64 and less: loses at S 2048 and 4096 with 512 blocks (0.82 - 0.93: narrow ones balance better),
//     wins at S 512 (1.08) and from 768 on (1.07 - 1.3); d 96 and 128: 1.05 - 1.4 from 512 on;
//   dQ: 1.03 - 1.15 of the whole backward from 512 on, 0.92 - 0.95 causal with long sequences below 768;
//   dK/dV, whose registers allow two blocks per CU: 1.02 - 1.14 without a mask where rounds of two blocks per CU are
//     full (0.95 - 0.97 at 768), causal only at S 512 and less (1.05 - 1.15; else 0.85 - 1.0).
enum Which { FWD, DQ, DKV };
static bool wide_rows(const AttnArgs& a, Which k) {
    if (a.S % 64) return false;
    const long cu = cu_count(), n = (long)((a.S + 127) / 128) * a.heads * a.B, rounds = (n + 2 * cu - 1) / (2 * cu);
    if (n < (k == FWD && !a.causal && a.d > 64 ? cu : 2 * cu)) return false;
    if (!a.causal) {
        if (k != FWD && a.S % 128 && a.S < 384) return false;       // an idle half block counts (S 192 0.97 - 0.99 of the backward)
        return k != DKV || n * 100 >= 85 * rounds * 2 * cu;
    }
    if (a.S <= 512) return true;
    return k == FWD ? a.d > 64 || n >= 3 * cu : k == DQ && (a.S <= 1024 || n >= 3 * cu);
}

// Folded for two resident blocks per CU (narrow kernels, wide ones up to two blocks per CU; 768 wide blocks of d 128,
// forward: heaviest first 1.38, folded 1.16 of the narrow speed).  All batch entries together while about four blocks per CU
// hold the launch (16 heads of 64, S 1024, B 4, forward, narrow 1.37, backward 1.07; at 2048 blocks 0.9), one fewer for wide
// heads, whose keys and values fill the L2s (backward, d 128, 1024 blocks 0.95 - 0.98).
static int block_order(const AttnArgs& a, long blocks, bool wide, bool one_per_cu) {
    const long cu = cu_count();
    const bool folded = !one_per_cu && (!wide || blocks <= 2 * cu);
    const bool all = a.d > 64 ? blocks < 4 * cu : blocks <= 4 * cu;
    return (folded ? ORDER_FOLDED : 0) | (all ? ORDER_ALL : 0);
}

template <int D, int DR, int NT, bool RAG, bool WIDE = false>
static hipError_t launch_fwd_nt(const AttnArgs& a, hipStream_t s) {
    const float scale = 1.f / sqrtf((float)a.d);
    constexpr int QB = WIDE ? 128 : 64;
    const dim3 grid(((a.S + QB - 1) / QB) * a.heads * a.B), block(256 * NT);
    const size_t stages = (size_t)2 * NT * 2 * 64 * D * 2;
    const size_t merge = WIDE ? 0 : (size_t)2 * (2 * NT - 1) * ((D / 32) * 16 * 64 + 128) * sizeof(float);
    const size_t smem = std::max(std::max(stages, merge), RAG && a.causal ? attn_row_lds_fwd(a) : 0);
    static std::atomic<bool> set{false};   // several host threads may launch at once
    if (!set.load(std::memory_order_acquire)) {
        hipError_t e = set_smem(attn_fwd_mfma_kernel<D, DR, NT, RAG, WIDE>, std::max(std::max(stages, merge), kMaxAttnRowLds));
        if (e != hipSuccess) return e;
        set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, DR, NT, RAG, WIDE>), grid, block, smem, s, a, scale,
                       block_order(a, grid.x, WIDE, NT == 2));
    return hipGetLastError();
}
template <int D, int DR>
static hipError_t launch_fwd_t(const AttnArgs& a, hipStream_t s) {
    if (a.S % 64)
        return tiles_per_step(a) == 2 ? launch_fwd_nt<D, DR, 2, true>(a, s) : launch_fwd_nt<D, DR, 1, true>(a, s);
    if (wide_rows(a, FWD)) return launch_fwd_nt<D, DR, 1, false, true>(a, s);
    return tiles_per_step(a) == 2 ? launch_fwd_nt<D, DR, 2, false>(a, s) : launch_fwd_nt<D, DR, 1, false>(a, s);
}

hipError_t launch_attn_fwd_mfma(const AttnArgs& a, hipStream_t s) {
    if (a.d == 128) return launch_fwd_t<128, 128>(a, s);
    if (a.d == 64) return launch_fwd_t<64, 64>(a, s);
    // the head widths of the paper's own models (Table 3) get kernels with the width built in
    if (a.d == 96) return launch_fwd_t<128, 96>(a, s);
    if (a.d == 40) return launch_fwd_t<64, 40>(a, s);
    return a.d > 64 ? launch_fwd_t<128, 0>(a, s) : launch_fwd_t<64, 0>(a, s);
}

template <int D, int DR, bool RAG, bool WIDE>
static hipError_t launch_dq(const AttnArgs& a, hipStream_t s) {
    const float scale = 1.f / sqrtf((float)a.d);
    constexpr int QB = WIDE ? 128 : 64;
    const dim3 grid(((a.S + QB - 1) / QB) * a.heads * a.B), block(256);
    constexpr size_t stages = 2 * 2 * 64 * D * 2;
    const size_t smem = std::max(stages, RAG && a.causal ? attn_row_lds_dq(a) : 0);
    static std::atomic<bool> set{false};   // several host threads may launch at once
    if (!set.load(std::memory_order_acquire)) {
        hipError_t e = set_smem(attn_bwd_dq_mfma_kernel<D, DR, RAG, WIDE>, std::max(stages, kMaxAttnRowLds));
        if (e != hipSuccess) return e;
        set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((attn_bwd_dq_mfma_kernel<D, DR, RAG, WIDE>), grid, block, smem, s, a, scale,
                       block_order(a, grid.x, WIDE, false));
    return hipGetLastError();
}
template <int D, int DR, bool RAG, bool WIDE>
static hipError_t launch_dkv(const AttnArgs& a, hipStream_t s) {
    const float scale = 1.f / sqrtf((float)a.d);
    constexpr int KB = WIDE ? 128 : 64;
    const dim3 grid(((a.S + KB - 1) / KB) * a.heads * a.B), block(256);
    constexpr size_t stages = 2 * (2 * 64 * D * 2 + 512);
    const size_t smem = std::max(stages, RAG && a.causal ? attn_row_lds_dkv(a) : 0);
    static std::atomic<bool> set{false};
    if (!set.load(std::memory_order_acquire)) {
        hipError_t e = set_smem(attn_bwd_dkv_mfma_kernel<D, DR, RAG, WIDE>, std::max(stages, kMaxAttnRowLds));
        if (e != hipSuccess) return e;
        set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((attn_bwd_dkv_mfma_kernel<D, DR, RAG, WIDE>), grid, block, smem, s, a, scale,
                       block_order(a, grid.x, WIDE, false));
    return hipGetLastError();
}

template <int D, int DR, bool RAG>
static hipError_t launch_bwd_both(const AttnArgs& a, hipStream_t s) {
    const float scale = 1.f / sqrtf((float)a.d);
    const dim3 grid(2 * ((a.S + 63) / 64) * a.heads * a.B), block(256);
    constexpr size_t stages = 2 * (2 * 64 * D * 2 + 512);
    const size_t smem = std::max(stages, RAG && a.causal ? std::max(attn_row_lds_dq(a), attn_row_lds_dkv(a)) : 0);
    static std::atomic<bool> set{false};   // several host threads may launch at once
    if (!set.load(std::memory_order_acquire)) {
        hipError_t e = set_smem(attn_bwd_mfma_kernel<D, DR, RAG>, std::max(stages, kMaxAttnRowLds));
        if (e != hipSuccess) return e;
        set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((attn_bwd_mfma_kernel<D, DR, RAG>), grid, block, smem, s, a, scale,
                       block_order(a, grid.x / 2, false, false));
    return hipGetLastError();
}

// dQ and dK/dV side by side in one launch: while neither fills the chip by itself, they take the time of the longer one and
// one launch is saved; delta is then computed twice, and the registers of both (198 - 234 at width 64) allow two blocks
// per CU, where three of the split kernels' fit at lengths that are multiples of 64 (two at others).  n blocks of each on
// 256 CUs, two launches / one, us:
//   d up to 64: n 24 13.3 / 8.0, 128 20.6 / 14.0, 256 32.6 / 25.7 (causal), 384 27.2 / 24.8, 46.5 / 37.1 (causal), 512 76.3 / 79.7,
//     causal 58.9 / 51.9, 35.4 / 33.2, 18.2 / 16.9, d 40 23.8 / 24.8, 1024 48.2 / 58.2, causal 58.1 / 60.7;
//     other lengths: 72 22.7 / 15.1, 400 49.2 / 40.7, 504 32.8 / 32.0, 512 66.3 / 66.7, 576 44.6 / 36.4, 720 46.7 / 45.2;
//   d 96: 256 28.3 / 23.0, 60.3 / 56.2 (S 1000), 512 49.7 / 50.6;
//   other wide heads, which spill registers: d 128 96 47.2 / 44.5, 128 36.9 / 33.0, 192 44.8 / 54.7 (S 333), 256 59.2 / 68.0;
//     d 112 96 47.3 / 39.3 (S 333).
bool attn_bwd_mfma_one_launch(const AttnArgs& a) {
    const long cu = cu_count(), n = (long)((a.S + 63) / 64) * a.heads * a.B;
    if (a.d == 96) return n <= cu;
    if (a.d > 64) return 2 * n <= cu;
    return 2 * n <= 3 * cu || (a.S % 64 ? n <= 3 * cu : a.causal && a.d > 40 && n <= 2 * cu);
}

template <int D, int DR>
static hipError_t launch_bwd_t(const AttnArgs& a, hipStream_t s) {
    if (attn_bwd_mfma_one_launch(a)) return a.S % 64 ? launch_bwd_both<D, DR, true>(a, s) : launch_bwd_both<D, DR, false>(a, s);
    hipError_t e = a.S % 64 ? launch_dq<D, DR, true, false>(a, s) :
                   wide_rows(a, DQ) ? launch_dq<D, DR, false, true>(a, s) : launch_dq<D, DR, false, false>(a, s);
    if (e != hipSuccess) return e;
    return a.S % 64 ? launch_dkv<D, DR, true, false>(a, s) :
           wide_rows(a, DKV) ? launch_dkv<D, DR, false, true>(a, s) : launch_dkv<D, DR, false, false>(a, s);
}

hipError_t launch_attn_bwd_mfma(const AttnArgs& a, hipStream_t s) {
    if (a.d == 128) return launch_bwd_t<128, 128>(a, s);
    if (a.d == 64) return launch_bwd_t<64, 64>(a, s);
    if (a.d == 96) return launch_bwd_t<128, 96>(a, s);
    if (a.d == 40) return launch_bwd_t<64, 40>(a, s);
    return a.d > 64 ? launch_bwd_t<128, 0>(a, s) : launch_bwd_t<64, 0>(a, s);
}

}  // namespace bp
