// Shape-generic kernels: a tiled GEMM with fp32 accumulation and a row-at-a-time attention
// forward/backward.  They serve any shape or alignment the matrix-core kernels do not cover, and short
// sequences; correctness first, no tuning.
#include "bp_kernels.h"
#include "bp_device.h"
#include "bp_attn_rows.h"

namespace bp {

// ------------------------------------------------------------------ GEMM 64x64x16, 4x4 per thread
template <typename T>
__global__ __launch_bounds__(256) void gemm_generic_kernel(GemmArgs g) {
    __shared__ float As[16][65];
    __shared__ float Bs[16][65];
    const T* A = (const T*)g.A;
    const T* B = (const T*)g.B;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < g.K; k0 += 16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = threadIdx.x + i * 256;
            int m, k;
            if (g.a_t) { k = e >> 6; m = e & 63; } else { m = e >> 4; k = e & 15; }
            const int gm = m0 + m, gk = k0 + k;
            float v = 0.f;
            if (gm < g.M && gk < g.K)
                v = to_float<T>(g.a_t ? A[(size_t)gk * g.lda + gm] : A[(size_t)gm * g.lda + gk]);
            As[k][m] = v;
            int n;
            if (g.b_t) { n = e >> 4; k = e & 15; } else { k = e >> 6; n = e & 63; }
            const int gn = n0 + n;
            const int gk2 = k0 + k;
            v = 0.f;
            if (gn < g.N && gk2 < g.K)
                v = to_float<T>(g.b_t ? B[(size_t)gn * g.ldb + gk2] : B[(size_t)gk2 * g.ldb + gn]);
            Bs[k][n] = v;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = As[kk][ty * 4 + i]; b[i] = Bs[kk][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + ty * 4 + i;
        if (m >= g.M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + tx * 4 + j;
            if (n >= g.N) continue;
            float v = acc[i][j];
            const size_t o = (size_t)m * g.ldc + n;
            if (g.accumulate) {
                float* c = (float*)g.C + o;
                *c = g.accumulate == 2 ? v : *c + v;
            } else {
                if (g.bias) v += g.bias[n];
                if (g.residual) v += to_float<T>(((const T*)g.residual)[o]);
                ((T*)g.C)[o] = from_float<T>(v);
            }
        }
    }
}

hipError_t launch_gemm_generic(int dtype, const GemmArgs& g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipErrorInvalidValue;
    dim3 grid((g.N + 63) / 64, (g.M + 63) / 64), block(256);
    if (dtype == BF16)
        hipLaunchKernelGGL((gemm_generic_kernel<bf16_t>), grid, block, 0, s, g);
    else
        hipLaunchKernelGGL((gemm_generic_kernel<float>), grid, block, 0, s, g);
    return hipGetLastError();
}

// ------------------------------------------------------------------ attention, one row per block
template <typename T>
__global__ __launch_bounds__(128) void attn_fwd_generic_kernel(AttnArgs a, float scale) {
    extern __shared__ float smem[];
    attn_fwd_row<T>(a, scale, blockIdx.x, blockIdx.y, blockIdx.z, smem);
}
template <typename T>
__global__ __launch_bounds__(128) void attn_bwd_dq_generic_kernel(AttnArgs a, float scale) {
    extern __shared__ float smem[];
    attn_bwd_dq_row<T>(a, scale, blockIdx.x, blockIdx.y, blockIdx.z, smem);
}
template <typename T>
__global__ __launch_bounds__(128) void attn_bwd_dkv_generic_kernel(AttnArgs a, float scale) {
    extern __shared__ float smem[];
    attn_bwd_dkv_row<T>(a, scale, blockIdx.x, blockIdx.y, blockIdx.z, smem);
}

hipError_t launch_attn_fwd_generic(int dtype, const AttnArgs& a, hipStream_t s) {
    const float scale = 1.f / sqrtf((float)a.d);
    dim3 grid(a.S, a.heads, a.B), block(128);
    const size_t sm = attn_row_lds_fwd(a);
    if (sm > kMaxAttnRowLds) return hipErrorInvalidValue;
    if (dtype == BF16)
        hipLaunchKernelGGL((attn_fwd_generic_kernel<bf16_t>), grid, block, sm, s, a, scale);
    else
        hipLaunchKernelGGL((attn_fwd_generic_kernel<float>), grid, block, sm, s, a, scale);
    return hipGetLastError();
}

hipError_t launch_attn_bwd_generic(int dtype, const AttnArgs& a, hipStream_t s) {
    const float scale = 1.f / sqrtf((float)a.d);
    dim3 grid(a.S, a.heads, a.B), block(128);
    const size_t sm1 = attn_row_lds_dq(a), sm2 = attn_row_lds_dkv(a);
    if (sm1 > kMaxAttnRowLds || sm2 > kMaxAttnRowLds) return hipErrorInvalidValue;
    if (dtype == BF16) {
        hipLaunchKernelGGL((attn_bwd_dq_generic_kernel<bf16_t>), grid, block, sm1, s, a, scale);
        hipLaunchKernelGGL((attn_bwd_dkv_generic_kernel<bf16_t>), grid, block, sm2, s, a, scale);
    } else {
        hipLaunchKernelGGL((attn_bwd_dq_generic_kernel<float>), grid, block, sm1, s, a, scale);
        hipLaunchKernelGGL((attn_bwd_dkv_generic_kernel<float>), grid, block, sm2, s, a, scale);
    }
    return hipGetLastError();
}

}  // namespace bp
