// fp32 GEMM on the gfx950 matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands and accumulation) for the
// three shapes of a linear layer in the fp32 storage path.
//
// A block computes a BM x BN tile of C, stepping over K in slices of BK.  Slices go straight from
// global memory into NS LDS stages; the buffer descriptors end with their operand, so whatever lies
// past its edge arrives as zeros.  Bound: the fp32 matrix rate, 256 flop/clk per CU (157 TFLOP/s),
// an eighth of the bf16 one, so operand traffic is never the limit and the tiles can be small:
//   * an operand whose contraction index is contiguous in memory is kept as [row][BK], 16-byte chunks
//     swizzled; one ds_read_b128 gives a lane four k of its row, i.e. its part of four MFMAs (the
//     two halves of a wave take alternate chunks: the order of k inside a slice is free as long as
//     both operands use the same one);
//   * an operand whose row index is contiguous is kept as [k][rows] and read 4 bytes per lane.
// WK > 1: the waves of a block also share out the k of every slice and add their partial tiles
// through LDS in a fixed order at the end.
#include <atomic>

#include "bp_kernels.h"
#include "bp_device.h"
#include "bp_tile.h"

namespace bp {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Loads of one operand slice: R rows x BK k of floats by NW waves, 16 bytes per lane and instruction.
template <int R, int BK, int NW, bool RMAJOR>
struct F32Plan {
    static constexpr int NI = R * BK / 256 / NW;    // wave instructions per wave per slice
    static_assert(NI >= 1 && R * BK == NI * 256 * NW, "the waves share a slice evenly");
    uint32_t boff[NI], tail[NI];                    // byte offset from the slice's start; in a segment's last slice
    __device__ __forceinline__ void init(int wave, int lane, int ld, int k_tail) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int P = (wave + NW * i) * 64 + lane;          // 16-byte position in the tile
            if (RMAJOR) {
                boff[i] = tail[i] = 4u * (uint32_t)((P / (R / 4)) * ld + (P % (R / 4)) * 4);
            } else {
                const int row = P / (BK / 4), c = (P % (BK / 4)) ^ kmaj_swz<2 * BK>(row);
                boff[i] = 4u * (uint32_t)(row * ld + c * 4);
                tail[i] = c * 4 < k_tail ? boff[i] : kOutside;
            }
        }
    }
    __device__ __forceinline__ void issue(rsrc_t src, bool last, char* lds, int wave) const {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            dma16(src, !RMAJOR && last ? tail[i] : boff[i], 0, lds + (wave + NW * i) * 1024);
    }
};

// the eight k (chunk pair j: 8j .. 8j+7) of row row0 + lane % 32 that this lane's half feeds to four MFMAs
template <int R, int BK, bool RMAJOR>
__device__ __forceinline__ f32x4 f32_frag(const char* lds, int row0, int j, int lane) {
    const int h = lane >> 5, row = row0 + (lane & 31);
    if (!RMAJOR) return *reinterpret_cast<const f32x4*>(lds + kmaj_off<2 * BK>(row, 2 * j + h));
    const float* p = reinterpret_cast<const float*>(lds) + (8 * j + 4 * h) * R + row;
    return f32x4{p[0], p[R], p[2 * R], p[3 * R]};
}

// GROUP: several contraction segments (grouped weight gradients)
template <int BM, int BN, int WM, int WN, int WK, int BK, int NS, bool A_RMAJOR, bool B_RMAJOR, bool GROUP>
__global__ __launch_bounds__(WM* WN* WK * 64) void gemm_f32_kernel(GemmArgs g, int tiles_m, int tiles_n) {
    constexpr int NW = WM * WN * WK;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int A_BYTES = BM * BK * 4, STAGE = (BM + BN) * BK * 4;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const void *A0 = g.A, *B0 = g.B;        // every argument in one round trip
    asm volatile("" : "+s"(A0), "+s"(B0)
                 : "s"(g.M), "s"(g.N), "s"(g.K), "s"(g.lda), "s"(g.ldb), "s"(g.ldc), "s"(g.nseg), "s"(g.C),
                   "s"(g.bias), "s"(g.residual), "s"(g.accumulate), "s"(g.epi), "s"(g.C2), "s"(g.U), "s"(g.colpart),
                   "s"(tiles_m), "s"(tiles_n));
    int tm, tn;
    tile_coords(blockIdx.x, tiles_m, tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;

    // the contraction: g.nseg operand pairs of g.K each, one after the other, in slices of BK
    const int nk_seg = (g.K + BK - 1) / BK;
    const long a_step = 4L * (A_RMAJOR ? BK * (long)g.lda : BK), b_step = 4L * (B_RMAJOR ? BK * (long)g.ldb : BK);
    F32Plan<BM, BK, NW, A_RMAJOR> pa;
    F32Plan<BN, BK, NW, B_RMAJOR> pb;
    pa.init(wave, lane, g.lda, g.K - (nk_seg - 1) * BK);
    pb.init(wave, lane, g.ldb, g.K - (nk_seg - 1) * BK);
    constexpr int LPT = decltype(pa)::NI + decltype(pb)::NI;    // loads per slice per wave
    static_assert((NS - 2) * LPT < 64, "outstanding loads must fit the vmcnt field");
    const char *a_at, *b_at;                // where the next slice to request starts
    long a_left, b_left;                    // bytes from there to the operand's end
    int seg = 0, kl = 0;
    auto origin = [&]() {
        const void *A = A0, *B = B0;
        if (seg > 0) { A = g.A_more[seg - 1]; B = g.B_more[seg - 1]; }
        a_at = (const char*)((const float*)A + (A_RMAJOR ? m0 : (size_t)m0 * g.lda));
        b_at = (const char*)((const float*)B + (B_RMAJOR ? n0 : (size_t)n0 * g.ldb));
        a_left = 4L * (A_RMAJOR ? (g.K - 1) * (long)g.lda + g.M - m0 : (g.M - m0 - 1) * (long)g.lda + g.K);
        b_left = 4L * (B_RMAJOR ? (g.K - 1) * (long)g.ldb + g.N - n0 : (g.N - n0 - 1) * (long)g.ldb + g.K);
    };
    origin();
    auto clip = [](long left) { return left <= 0 ? 0u : left < (long)kOutside ? (uint32_t)left : kOutside; };
    // request the next slice; past the last one the descriptors are empty and nothing but zeros arrives
    auto request = [&](char* st) {
        pa.issue(make_rsrc(a_at, clip(a_left)), kl == nk_seg - 1, st, wave);
        pb.issue(make_rsrc(b_at, clip(b_left)), kl == nk_seg - 1, st + A_BYTES, wave);
        a_at += a_step; a_left -= a_step;
        b_at += b_step; b_left -= b_step;
        if (++kl == nk_seg) {
            if (++seg < g.nseg) { kl = 0; origin(); }
            else { a_left = b_left = 0; }
        }
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    // sums of the segments before: one chain of additions over all of them would round more than a launch per
    // micro-batch does (1024 x 4096 over 4 x 2100 tokens: 1.6e-6 against 8.2e-7 in the 2-norm); up to 5 % of a launch
    // over many short segments (472 x 708 over 8 x 328 tokens 39 -> 41 us)
    f32x16 done[GROUP ? TM : 1][GROUP ? TN : 1];
    if constexpr (GROUP) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) done[i][j][v] = 0.f;
    }

#pragma unroll
    for (int s = 0; s < NS - 1; ++s) request(smem + s * STAGE);
    int cur = 0;
    for (int sgm = 0; sgm < (GROUP ? g.nseg : 1); ++sgm) {
    for (int kt = 0; kt < nk_seg; ++kt) {
        BP_WAIT_VMCNT((NS - 2) * LPT);                  // this wave's part of slice kt has landed
        __builtin_amdgcn_s_waitcnt(0xC07F);             // lgkmcnt(0): its reads of slice kt - 1 are over
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        request(smem + (cur == 0 ? NS - 1 : cur - 1) * STAGE);      // into the stage of slice kt - 1
        const char* sa = smem + cur * STAGE;
        const char* sb = sa + A_BYTES;
#pragma unroll
        for (int jj = 0; jj < BK / 8 / WK; ++jj) {
            const int j = wk * (BK / 8 / WK) + jj;
            f32x4 fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = f32_frag<BM, BK, A_RMAJOR>(sa, wm * (BM / WM) + i * 32, j, lane);
#pragma unroll
            for (int i = 0; i < TN; ++i) fb[i] = f32_frag<BN, BK, B_RMAJOR>(sb, wn * (BN / WN) + i * 32, j, lane);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int i2 = 0; i2 < TN; ++i2)
                        acc[i][i2] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[i2][e], acc[i][i2], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        cur = cur + 1 == NS ? 0 : cur + 1;
    }
    if constexpr (GROUP) {
        const bool last = sgm + 1 == g.nseg;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    done[i][j][v] += acc[i][j][v];
                    acc[i][j][v] = last ? done[i][j][v] : 0.f;
                }
    }
    }
    BP_WAIT_VMCNT(0);

    if constexpr (WK > 1) {     // waves 1 .. WK-1 hand their partial tiles to wave 0 through LDS
        __syncthreads();
        float* part = (float*)smem + (size_t)(wm * WN + wn) * (WK - 1) * (TM * TN * 16 * 64);
        if (wk > 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        part[(size_t)(wk - 1) * (TM * TN * 16 * 64) + ((i * TN + j) * 16 + v) * 64 + lane] = acc[i][j][v];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int w = 0; w < WK - 1; ++w)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        acc[i][j][v] += part[(size_t)w * (TM * TN * 16 * 64) + ((i * TN + j) * 16 + v) * 64 + lane];
    }

    // Accumulator v of lane l holds C[8*(v/4) + 4*(l/32) + v%4][l%32]: a store writes two row pieces of
    // 128 contiguous bytes.
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 + wn * (BN / WN) + j * 32 + (lane & 31);
        const bool in_n = n < g.N;
        const float bias = g.bias && in_n ? g.bias[n] : 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m_base = m0 + wm * (BM / WM) + i * 32;
            float csum = 0.f;                           // EPI_GELU_BWD: column sums of these 32 rows
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m_base + 8 * (v >> 2) + 4 * h + (v & 3);
                if (!in_n || m >= g.M) continue;
                const size_t o = (size_t)m * g.ldc + n;
                float* c = (float*)g.C + o;
                const float r = acc[i][j][v];
                if (g.accumulate) {
                    *c = g.accumulate == 2 ? r : *c + r;
                } else if (g.epi == EPI_GELU_FWD) {
                    *c = r;
                    ((float*)g.C2)[o] = gelu_value(r + bias);
                } else if (g.epi == EPI_GELU_BWD) {
                    const float du = r * gelu_slope(((const float*)g.U)[o] + bias);
                    *c = du;
                    csum += du;
                } else {
                    *c = r + bias + (g.residual ? ((const float*)g.residual)[o] : 0.f);
                }
            }
            if (g.epi == EPI_GELU_BWD) {
                csum = halves_sum(csum);
                if (h == 0 && in_n && m_base < g.M) g.colpart[(size_t)(m_base >> 5) * g.N + n] = csum;
            }
        }
    }
}

// 16-byte loads: rows of both operands (and their k, where that is the contiguous index) in pieces of four
bool gemm_f32_supported(const GemmArgs& g) {
    auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
    if (g.lda % 4 || g.ldb % 4 || ((!g.a_t || g.b_t) && g.K % 4)) return false;
    if ((g.a_t && g.M % 4) || (!g.b_t && g.N % 4)) return false;
    if (!al16(g.A) || !al16(g.B)) return false;
    for (int i = 0; i + 1 < g.nseg; ++i)
        if (!al16(g.A_more[i]) || !al16(g.B_more[i])) return false;
    return true;
}

template <int BM, int BN, int WM, int WN, int WK, int BK, int NS>
static hipError_t launch_f32(const GemmArgs& g, hipStream_t s) {
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    const size_t stages = (size_t)NS * (BM + BN) * BK * 4;
    const size_t merge = (size_t)(WK - 1) * BM * BN * 4;
    const size_t smem = stages > merge ? stages : merge;
#define BP_GEMM_LAUNCH(AR, BR, GROUP)                                                            \
    do {                                                                                         \
        auto kern = gemm_f32_kernel<BM, BN, WM, WN, WK, BK, NS, AR, BR, GROUP>;                  \
        static std::atomic<bool> attr_set{false};   /* once per instantiation; host threads may race */ \
        if (smem > 64 * 1024 && !attr_set.load(std::memory_order_acquire)) {                     \
            hipError_t e = hipFuncSetAttribute((const void*)kern,                                \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem); \
            if (e != hipSuccess) return e;                                                       \
            attr_set.store(true, std::memory_order_release);                                     \
        }                                                                                        \
        hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(WM * WN * WK * 64), smem, s, g, tiles_m, tiles_n); \
    } while (0)
    if (g.nseg > 1) BP_GEMM_LAUNCH(true, true, true);
    else if (!g.a_t && !g.b_t) BP_GEMM_LAUNCH(false, true, false);
    else if (!g.a_t && g.b_t) BP_GEMM_LAUNCH(false, false, false);
    else if (g.a_t && !g.b_t) BP_GEMM_LAUNCH(true, true, false);
    else BP_GEMM_LAUNCH(true, false, false);
#undef BP_GEMM_LAUNCH
    return hipGetLastError();
}

// Tiles of 64 x 64 (four waves side by side, three blocks per CU) when they fill the CUs evenly, else
// tiles of 32 x 32 whose four waves share out k: the smaller tiles do 0.8 of the larger ones' rate at
// equal fill but four times as many share the chip more evenly and a short launch ends sooner
// (64 / 32 wide, us: 1024 x 3072 x 768, 768 tiles of 64: 52 / 68; 1024 x 768 x 768, 192 tiles: 23 / 20;
// 1024 x 768 x 3072: 71 / 56; weight gradient 768 x 3072 x 4096, 576 tiles: 208 / 186; 128 x 128 x 512:
// 16 / 9).  Larger tiles (128 x 64, 128 x 128) gain 2 % from 2048 x 4096 x 1024 on and lose below.
// The generic kernel these replace: 1024 x 768..3072 products 290 us on average, 128 x 128 x 512 41 us.
hipError_t launch_gemm_f32(const GemmArgs& g, hipStream_t s) {
    if (g.nseg > 1 && !(g.a_t && !g.b_t)) return launch_gemm_per_segment(g, s, launch_gemm_f32);    // (groups are weight gradients)
    const int ncu = cu_count();
    auto fill = [&](int b) {
        const long t = (long)((g.M + b - 1) / b) * ((g.N + b - 1) / b);
        return (double)t / (double)((t + ncu - 1) / ncu * ncu);
    };
    if (fill(64) >= 0.8 * fill(32)) return launch_f32<64, 64, 2, 2, 1, 32, 3>(g, s);
    return launch_f32<32, 32, 1, 1, 4, 64, 3>(g, s);
}

}  // namespace bp
