// Device-side pieces shared by the GEMM and attention kernels that load their operands straight into LDS:
// the swizzle of k-major tiles, buffer descriptors, the load itself and the wait for it, the order of output tiles.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bp {

// (a 16-byte fragment read serves 16 lanes = 16 consecutive rows per cycle: the XOR has to give
// those rows 16 different chunk positions modulo the 256-byte bank period)
template <int BKT> __device__ __forceinline__ int kmaj_swz(int row) {
    return BKT >= 128 ? (row & 15) : BKT == 64 ? ((row >> 1) & 7) : ((row >> 2) & 3);
}
// byte offset of logical 16-byte chunk c of `row` in a k-major tile [R][BKT]
template <int BKT> __device__ __forceinline__ int kmaj_off(int row, int c) {
    return row * (BKT * 2) + ((c ^ kmaj_swz<BKT>(row)) << 4);
}

// One wave instruction moves 64 x 16 bytes from global memory straight into 1 KiB of consecutive LDS.
// The global address is a buffer descriptor (wave-uniform tile origin) plus a per-lane 32-bit byte
// offset plus a wave-uniform byte offset (the K slice), so issuing a load costs no vector ALU work.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes = 0xffffffffu) {
    // raw buffer, stride 0, loads at or beyond `bytes` give zeros (default: no bounds clamp below
    // 4 GiB - 1); dword 3 as for untyped 32-bit data on gfx9
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void dma16(rsrc_t rsrc, uint32_t lane_off, uint32_t slice_off, char* lds_wave_base) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (void __attribute__((address_space(3)))*)lds_wave_base, 16,
                                             (int)lane_off, (int)slice_off, 0, 0);
}

// LDS transpose read: lane i of a group of 16 receives element i % 4 of the four 8-byte pieces that lanes
// 4 r + i / 4 (r = 0 .. 3) address.  `__restrict__` is what this function is for.  A bare call of the builtin is
// taken to read what any load into LDS still on its way may write, and the compiler waits for all of them
// (vmcnt(0)) in front of the first transpose read after a request: every kernel that prefetches the next slice and
// then reads this one transposed waited a whole memory latency per slice (plain LDS reads carry the alias scope that
// the parameter gives these).  The waits that are needed are the callers' own, in front of their barriers.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef s16x4 __attribute__((address_space(3))) lds_s16x4;
__device__ __forceinline__ s16x4 lds_read_tr(const lds_s16x4* __restrict__ p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(const_cast<lds_s16x4*>(p));
}

// s_waitcnt with only vmcnt set (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
#define BP_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (((N) >> 4) << 14) | (7 << 4) | (15 << 8))

constexpr uint32_t kOutside = 0xffffff00u;          // beyond the size of every ragged operand's descriptor

// Tile order: each XCD (blocks are dealt round-robin over 8 XCDs) gets a contiguous range of ids,
// walked in groups of 4 tile rows so that concurrent blocks share A rows and B columns.
__device__ __forceinline__ void tile_coords(int t, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int nblk = tiles_m * tiles_n;
    if (nblk % 8 == 0) t = (t & 7) * (nblk >> 3) + (t >> 3);
    constexpr int GM = 4;
    const int per_group = GM * tiles_n;
    const int group = t / per_group, in_group = t - group * per_group;
    const int first_m = group * GM;
    const int gsize = tiles_m - first_m;
    if (gsize >= GM) {          // a full group: no second division on the way to a block's first load
        tm = first_m + in_group % GM;
        tn = in_group / GM;
    } else {
        tn = in_group / gsize;
        tm = first_m + in_group - tn * gsize;
    }
}

}  // namespace bp
