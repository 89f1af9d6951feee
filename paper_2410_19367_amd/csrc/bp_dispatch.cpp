// Kernel selection: which implementation serves a given GEMM / attention shape.
#include "bp_kernels.h"

#include <atomic>

namespace bp {

int cu_count() {
    static std::atomic<int> cached{0};
    int n = cached.load(std::memory_order_relaxed);
    if (!n) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cached.store(n, std::memory_order_relaxed);
    }
    return n;
}

// one launch per contraction segment, for kernels that take a single operand pair
hipError_t launch_gemm_per_segment(const GemmArgs& g, hipStream_t stream,
                                   hipError_t (*one)(const GemmArgs&, hipStream_t)) {
    GemmArgs h = g;
    h.nseg = 1;
    for (int sgm = 0; sgm < g.nseg; ++sgm) {
        if (sgm > 0) {
            h.A = g.A_more[sgm - 1];
            h.B = g.B_more[sgm - 1];
            h.accumulate = 1;
        }
        hipError_t e = one(h, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_gemm(int dtype, const GemmArgs& g, hipStream_t stream) {
    if (g.nseg < 1 || g.nseg > kMaxGemmSegments || (g.nseg > 1 && !g.accumulate)) return hipErrorInvalidValue;
    if (g.epi != EPI_NONE && !gemm_can_fuse_epilogue(dtype, g)) return hipErrorInvalidValue;
    if (dtype == BF16 && gemm_mfma_supported(g)) return launch_gemm_mfma(g, stream);
    if (dtype == F32 && gemm_f32_supported(g)) return launch_gemm_f32(g, stream);
    if (g.nseg == 1) return launch_gemm_generic(dtype, g, stream);
    if (dtype == BF16)
        return launch_gemm_per_segment(g, stream, [](const GemmArgs& h, hipStream_t s) {
            return launch_gemm_generic(BF16, h, s);
        });
    return launch_gemm_per_segment(g, stream, [](const GemmArgs& h, hipStream_t s) {
        return launch_gemm_generic(F32, h, s);
    });
}

// Short sequences: the kernels of one row per block beat the matrix-core ones, whose tiles of 64 rows are then mostly
// padding and whose time is one chain of latencies whatever the length.  What decides is the work of all rows, heads
// times S^2, and how soon the rows are more than the chip holds at once (rows / matrix cores, us):
//   fp32, heads wider than 64: 16 of 96, backward, S 63 (63504) 28.4 / 27.7, 256 of 96, S 12 (36864) 21.5 / 24.2, S 16
//     34.7 / 24.3; 4 of 104, backward, S 128 (512 rows, 65536) 31.0 / 49.9;
//   33 to 64 wide: 64 of 64, backward, S 24 (36864) 14.6 / 17.0, S 32 20.1 / 17.2; 16, forward, S 48 6.1 / 6.5, S 63 7.4 / 6.7;
//   narrower: 16 of 24, backward, S 32 10.2 / 11.4, S 48 13.7 / 11.8; 2 of 24, forward, S 24 4.3 / 4.5, S 32 4.6 / 4.1;
//   bf16 backward: 16 of 64, S 16 9.0 / 9.2, 64 of 64 10.4 / 9.3; 2 of 128, S 48 15.6 / 16.8; widths above 64 without a kernel
//     of their own spill registers: 1 of 80, S 76 16.6 / 24.5;
//   backward where dQ and dK/dV share a launch:
//     fp32, d 24 always (S 16 7.5 / 6.5, S 48 13.8 / 7.0); d 64 8 heads, S 32 (8192) 9.8 / 10.7, 4 heads, S 48 (9216) 12.6 / 11.1,
//       2 of 40, S 77 (11858) 15.8 / 16.4, 2 of 64, S 150 (45000) 31.5 / 23.8; d 96 4 heads, S 32 11.0 / 14.7, 16 heads, S 63 22.6 /
//       16.1; d 128 4 heads, S 90 26.2 / 33.4, d 104 S 128 32.7 / 31.9;
//     bf16, d 64 16 heads, S 16 8.8 / 6.2, 4 heads, S 4 7.6 / 5.9; d 96 S 12 9.6 / 8.6; d 128 S 40 13.4 / 13.4, S 16 11.2 / 12.9;
//       d 112 S 30 12.2 / 16.1, S 60 18.0 / 16.8; d 80 S 76 16.4 / 18.0, S 100 25.8 / 16.8;
//   bf16 forward: 16 of 64, S 4 4.2 / 4.1 (causal 4.2 / 4.6); 16 of 128, S 12 5.4 / 5.5 (causal 5.4 / 6.1).
// (bf16 at multiples of 64 has always been on the matrix cores.)
static bool rows_are_faster(int dtype, const AttnArgs& a, bool bwd) {
    const long rows = (long)a.B * a.heads * a.S, work = rows * a.S;
    if (dtype == F32 && bwd && attn_bwd_f32_one_launch(a)) {
        if (a.d <= 32) return false;
        if (a.d <= 64) return work <= (a.S <= 64 ? 8192 : 12000);
        return a.d <= 96 ? a.S <= 44 && work <= 40000 : a.S <= 112 && work <= 60000;
    }
    if (dtype == F32) {
        if (a.d > 32 && rows > 3072) return work <= 40000;
        if (a.d > 32 && rows <= 512) return work <= (a.d > 64 ? 120000 : 80000);
        if (a.d > 32) return work <= (a.d > 64 ? 64000 : bwd ? 50000 : 40000);
        return a.S <= (bwd ? 48 : 24) && work <= 20000;
    }
    if (a.S % 64 == 0) return false;
    if (bwd && attn_bwd_mfma_one_launch(a)) {
        if (a.d <= 64 || a.d == 96) return false;
        return a.d == 128 ? a.S <= 40 && work <= 16384 : (a.S <= 52 || (a.S > 64 && a.S <= 80)) && work <= 40000;
    }
    if (bwd && a.d > 64 && a.d != 96) return a.d == 128 ? a.S <= 48 && work <= 16384 : work <= 40000;
    if (bwd) return a.S <= (a.d == 96 ? 24 : 16) && work <= 8192;
    return a.d > 32 && a.d <= 64 ? a.S <= 4 && work <= 2048 : a.S <= 12 && work <= 4096;
}

hipError_t launch_attn_fwd(int dtype, const AttnArgs& a, hipStream_t stream) {
    const bool rows = rows_are_faster(dtype, a, false);
    if (dtype == BF16 && !rows && attn_mfma_supported(a)) return launch_attn_fwd_mfma(a, stream);
    if (dtype == F32 && !rows && attn_f32_supported(a)) return launch_attn_fwd_f32(a, stream);
    return launch_attn_fwd_generic(dtype, a, stream);
}

hipError_t launch_attn_bwd(int dtype, const AttnArgs& a, hipStream_t stream) {
    const bool rows = rows_are_faster(dtype, a, true);
    if (dtype == BF16 && !rows && attn_mfma_supported(a)) return launch_attn_bwd_mfma(a, stream);
    if (dtype == F32 && !rows && attn_f32_supported(a)) return launch_attn_bwd_f32(a, stream);
    return launch_attn_bwd_generic(dtype, a, stream);
}

}  // namespace bp
