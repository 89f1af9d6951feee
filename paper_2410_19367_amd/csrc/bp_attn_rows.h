// Attention of a single row by all threads of a block, in fp32: forward and dQ of one query, dK and dV of one
// key.  Nothing but the row's own keys (queries) is read.  The kernels of one row per block are made of these, and
// the matrix-core kernels (fp32, and bf16 at lengths that are no multiple of 64) fall back on them for a block of
// 64 causal rows whose diagonal tile is not finite: masked probabilities are zero there, but zero times NaN is
// not, and a token must not reach those before it.  The look at the diagonal tiles costs 1 - 10 % of a causal launch (bf16,
// B 1, S 2249, 12 heads of 40, backward 84 -> 88 us; B 3, S 294, 8 heads of 128 36 -> 39 us; fp32 1 - 5 %).
#pragma once
#include "bp_kernels.h"
#include "bp_device.h"

namespace bp {

// bytes of LDS that a row takes
inline size_t attn_row_lds_fwd(const AttnArgs& a) { return (size_t)(a.S + a.d + 8) * sizeof(float); }
inline size_t attn_row_lds_dq(const AttnArgs& a) { return (size_t)(a.S + 2 * a.d + 8) * sizeof(float); }
inline size_t attn_row_lds_dkv(const AttnArgs& a) { return (size_t)(2 * a.S + 2 * a.d) * sizeof(float); }
constexpr size_t kMaxAttnRowLds = 60000;

__device__ __forceinline__ float block_reduce(float v, float* red, bool is_max) {
    v = is_max ? wave_max(v) : wave_sum(v);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    float r = red[0];
    for (int i = 1; i < nw; ++i) r = is_max ? fmaxf(r, red[i]) : r + red[i];
    return r;
}

template <typename T>
__device__ __forceinline__ void attn_fwd_row(const AttnArgs& a, float scale, int i, int h, int b, float* smem) {
    __syncthreads();              // the row before is done with the LDS
    float* sc = smem;             // [S]
    float* qs = sc + a.S;         // [d]
    float* red = qs + a.d;        // [8]
    const int H = a.heads * a.d, ld = 3 * H;
    const T* qkv = (const T*)a.qkv;
    const T* qrow = qkv + ((size_t)(b * a.S + i)) * ld + h * a.d;
    const T* kbase = qkv + ((size_t)b * a.S) * ld + H + h * a.d;
    const T* vbase = kbase + H;
    const int kend = a.causal ? i + 1 : (a.lens ? a.lens[b] : a.S);
    for (int c = threadIdx.x; c < a.d; c += blockDim.x) qs[c] = to_float<T>(qrow[c]);
    __syncthreads();
    float mx = -INFINITY;
    for (int j = threadIdx.x; j < kend; j += blockDim.x) {
        const T* kr = kbase + (size_t)j * ld;
        float dot = 0.f;
        for (int c = 0; c < a.d; ++c) dot += qs[c] * to_float<T>(kr[c]);
        dot *= scale;
        sc[j] = dot;
        mx = fmaxf(mx, dot);
    }
    mx = block_reduce(mx, red, true);
    float sum = 0.f;
    for (int j = threadIdx.x; j < kend; j += blockDim.x) {
        const float e = __expf(sc[j] - mx);
        sc[j] = e;
        sum += e;
    }
    sum = block_reduce(sum, red, false);
    const float inv = 1.f / sum;
    T* out = (T*)a.ctx + ((size_t)(b * a.S + i)) * H + h * a.d;
    for (int c = threadIdx.x; c < a.d; c += blockDim.x) {
        float acc = 0.f;
        for (int j = 0; j < kend; ++j) acc += sc[j] * to_float<T>(vbase[(size_t)j * ld + c]);
        out[c] = from_float<T>(acc * inv);
    }
    if (threadIdx.x == 0) a.lse[((size_t)b * a.heads + h) * a.S + i] = mx + __logf(sum);
}

// dq and delta of one query
template <typename T>
__device__ __forceinline__ void attn_bwd_dq_row(const AttnArgs& a, float scale, int i, int h, int b, float* smem) {
    __syncthreads();              // the row before is done with the LDS
    float* ds = smem;             // [S]
    float* qs = ds + a.S;         // [d]
    float* dos = qs + a.d;        // [d]
    float* red = dos + a.d;       // [8]
    const int H = a.heads * a.d, ld = 3 * H;
    const T* qkv = (const T*)a.qkv;
    const size_t tok = (size_t)(b * a.S + i);
    const T* qrow = qkv + tok * ld + h * a.d;
    const T* kbase = qkv + ((size_t)b * a.S) * ld + H + h * a.d;
    const T* vbase = kbase + H;
    const T* orow = (const T*)a.ctx + tok * H + h * a.d;
    const T* dorow = (const T*)a.dctx + tok * H + h * a.d;
    const int kend = a.causal ? i + 1 : (a.lens ? a.lens[b] : a.S);
    float part = 0.f;
    for (int c = threadIdx.x; c < a.d; c += blockDim.x) {
        qs[c] = to_float<T>(qrow[c]);
        const float dv = to_float<T>(dorow[c]);
        dos[c] = dv;
        part += dv * to_float<T>(orow[c]);
    }
    const float delta = block_reduce(part, red, false);
    const size_t li = ((size_t)b * a.heads + h) * a.S + i;
    const float lse = a.lse[li];
    if (threadIdx.x == 0) a.delta[li] = delta;
    for (int j = threadIdx.x; j < kend; j += blockDim.x) {
        const T* kr = kbase + (size_t)j * ld;
        const T* vr = vbase + (size_t)j * ld;
        float s = 0.f, dp = 0.f;
        for (int c = 0; c < a.d; ++c) {
            s += qs[c] * to_float<T>(kr[c]);
            dp += dos[c] * to_float<T>(vr[c]);
        }
        const float p = __expf(s * scale - lse);
        ds[j] = p * (dp - delta);
    }
    __syncthreads();
    T* dq = (T*)a.dqkv + tok * ld + h * a.d;
    for (int c = threadIdx.x; c < a.d; c += blockDim.x) {
        float acc = 0.f;
        for (int j = 0; j < kend; ++j) acc += ds[j] * to_float<T>(kbase[(size_t)j * ld + c]);
        dq[c] = from_float<T>(acc * scale);
    }
}

// dk and dv of one key.  Needs delta from the dq kernel, or with OWN_DELTA takes it from ctx and dctx.
template <typename T, bool OWN_DELTA = false>
__device__ __forceinline__ void attn_bwd_dkv_row(const AttnArgs& a, float scale, int j, int h, int b, float* smem) {
    __syncthreads();              // the row before is done with the LDS
    float* ps = smem;             // [S]
    float* dss = ps + a.S;        // [S]
    float* ks = dss + a.S;        // [d]
    float* vs = ks + a.d;         // [d]
    const int H = a.heads * a.d, ld = 3 * H;
    const T* qkv = (const T*)a.qkv;
    const size_t tok = (size_t)(b * a.S + j);
    const T* qbase = qkv + ((size_t)b * a.S) * ld + h * a.d;
    const T* krow = qkv + tok * ld + H + h * a.d;
    const T* vrow = krow + H;
    const T* dobase = (const T*)a.dctx + ((size_t)b * a.S) * H + h * a.d;
    const T* obase = (const T*)a.ctx + ((size_t)b * a.S) * H + h * a.d;
    T* dk = (T*)a.dqkv + tok * ld + H + h * a.d;
    T* dv = dk + H;
    const int klen = a.causal ? a.S : (a.lens ? a.lens[b] : a.S);
    if (j >= klen) {   // masked key: no query attends it
        for (int c = threadIdx.x; c < a.d; c += blockDim.x) {
            dk[c] = from_float<T>(0.f);
            dv[c] = from_float<T>(0.f);
        }
        return;
    }
    const int i0 = a.causal ? j : 0;
    for (int c = threadIdx.x; c < a.d; c += blockDim.x) {
        ks[c] = to_float<T>(krow[c]);
        vs[c] = to_float<T>(vrow[c]);
    }
    __syncthreads();
    const float* lse = a.lse + ((size_t)b * a.heads + h) * a.S;
    const float* delta = a.delta + ((size_t)b * a.heads + h) * a.S;
    for (int i = i0 + threadIdx.x; i < a.S; i += blockDim.x) {
        const T* qr = qbase + (size_t)i * ld;
        const T* dor = dobase + (size_t)i * H;
        float s = 0.f, dp = 0.f, dl = 0.f;
        for (int c = 0; c < a.d; ++c) {
            s += to_float<T>(qr[c]) * ks[c];
            dp += to_float<T>(dor[c]) * vs[c];
            if (OWN_DELTA) dl += to_float<T>(dor[c]) * to_float<T>(obase[(size_t)i * H + c]);
        }
        if (!OWN_DELTA) dl = delta[i];
        const float p = __expf(s * scale - lse[i]);
        ps[i] = p;
        dss[i] = p * (dp - dl);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < a.d; c += blockDim.x) {
        float av = 0.f, ak = 0.f;
        for (int i = i0; i < a.S; ++i) {
            av += ps[i] * to_float<T>(dobase[(size_t)i * H + c]);
            ak += dss[i] * to_float<T>(qbase[(size_t)i * ld + c]);
        }
        dv[c] = from_float<T>(av);
        dk[c] = from_float<T>(ak * scale);
    }
}

// the statistics of 32 queries, one lane each
__device__ __forceinline__ bool stats_finite(const float* lse, const float* delta, int lane) {
    const float z = 0.f * lse[lane & 31] + 0.f * delta[lane & 31];
    return __builtin_amdgcn_ballot_w64(z != 0.f) == 0;
}

// After a kernel's last tile: has any wave of the block seen a diagonal tile that is not finite?
__device__ __forceinline__ bool any_wave(bool mine, void* smem) {
    int* flag = (int*)smem;
    const int nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) flag[threadIdx.x >> 6] = mine;
    __syncthreads();
    int any = 0;
    for (int i = 0; i < nw; ++i) any |= flag[i];
    return __builtin_amdgcn_readfirstlane(any) != 0;
}

}  // namespace bp
