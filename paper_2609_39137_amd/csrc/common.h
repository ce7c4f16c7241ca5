// Internal helpers shared by the gfx950 kernels of the ID Balancing router
// step.  Device code only; the C ABI lives in abi.cpp.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace idb {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Device status codes (same values as idb_status in include/idb.h).
constexpr int32_t kStatusOk = 0;
constexpr int32_t kStatusInvalid = 1;
constexpr int32_t kStatusEmpty = 3;

// Largest number of experts selected per token on the GPU paths.
constexpr int kMaxK = 32;

// The order of the biased-score ranking (Eq. pid-routing: value descending,
// lowest index first among equal values, -0 == +0) as one unsigned 64-bit key,
// larger first.  High word: the float's bits mapped to an unsigned order
// (after -0 -> +0, so equal values get equal words); low word: ~index, so the
// lower index wins ties.  Key 0 ranks below every finite or infinite value and
// serves as "no entry".
__device__ __forceinline__ unsigned long long rank_key(float v, int idx) {
    const unsigned u = __float_as_uint(v + 0.0f);  // -0 + +0 = +0
    const unsigned o = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((unsigned long long)o << 32) | (unsigned)(~(unsigned)idx);
}

// The value of a rank key (inverse of its high word; -0 comes back as +0).
__device__ __forceinline__ float rank_key_value(unsigned long long key) {
    const unsigned o = (unsigned)(key >> 32);
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// Orders a wave's LDS writes before the same wave's later LDS reads of what
// other lanes wrote: one wave's LDS instructions execute in issue order, so
// only the compiler has to be kept from moving memory operations across.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Score activation s = sigmoid(z) = 1 / (1 + 2^(-z log2 e)) with the hardware
// exp2 and reciprocal (each about 1 ulp).  Saturates to exactly 0 and 1.
__device__ __forceinline__ float sigmoid_fast(float z) {
    float e = __builtin_amdgcn_exp2f(z * -1.4426950408889634f);
    return __builtin_amdgcn_rcpf(1.0f + e);
}

// x of the lane R below in the same 16-lane row (cyclic).
template <int R>
__device__ __forceinline__ int row_rot(int x) {
    return __builtin_amdgcn_update_dpp(0, x, 0x120 + R, 0xF, 0xF, false);
}
template <int R>
__device__ __forceinline__ float row_rot(float x) {
    return __builtin_bit_cast(float, row_rot<R>(__builtin_bit_cast(int, x)));
}
template <int R>
__device__ __forceinline__ double row_rot(double x) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)row_rot<R>((int)(unsigned)u), hi = (unsigned)row_rot<R>((int)(unsigned)(u >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Four floats at any 4-byte aligned address (rows of odd length).
struct __attribute__((packed, aligned(4))) f4u {
    float v[4];
};

// Raw buffer resource over [base, base + bytes) (bytes < 2^32) and a 16-byte
// load at per-lane offset voff plus scalar offset soff.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 bload16(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

// One 16-byte unit of both operands: bf16 -> one 32x32x16 MFMA; fp32 -> four
// 32x32x2 MFMAs, float i of each lane's unit feeding the i-th.
template <bool F32>
__device__ __forceinline__ floatx16 mfma_unit(uint4 a, uint4 b, floatx16 c) {
    if constexpr (F32) {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, a.x), __builtin_bit_cast(float, b.x), c,
                                                 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, a.y), __builtin_bit_cast(float, b.y), c,
                                                 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, a.z), __builtin_bit_cast(float, b.z), c,
                                                 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, a.w), __builtin_bit_cast(float, b.w), c,
                                                 0, 0, 0);
        return c;
    } else {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
    }
}

// XCD-aware block order: consecutive blocks land on different XCDs, so remap
// to give each XCD a contiguous run of (tile, slice) pairs; the slices of one
// token tile then share their token rows in that XCD's L2.
__device__ __forceinline__ int xcd_block_order() {
    const int nb = gridDim.x;
    int L = blockIdx.x;
    if ((nb & 7) == 0) L = (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3);
    return L;
}

}  // namespace idb
