// Device-side helpers shared by the HIP kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace edl {

typedef uint16_t bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// Two floats to two packed bf16 (a in the low half), round to nearest even:
// the hardware's packed conversion.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack2_bf16(float a, float b) {
    const floatx2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(pack2_bf16(f, 0.f) & 0xffffu); }

template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int VEC = 4;  // elements per 16-byte vector
    static __device__ __forceinline__ float to_f32(float v) { return v; }
    static __device__ __forceinline__ float from_f32(float v) { return v; }
};
template <> struct Elem<bf16_t> {
    static constexpr int VEC = 8;
    static __device__ __forceinline__ float to_f32(bf16_t v) { return bf16_to_f32(v); }
    static __device__ __forceinline__ bf16_t from_f32(float v) { return f32_to_bf16(v); }
};

// 16-byte vector of T with element access
template <typename T> union Vec16 {
    uint4 u;
    T e[16 / sizeof(T)];
};

template <typename T> __device__ __forceinline__ Vec16<T> load_vec(const T* p) {
    Vec16<T> v;
    v.u = *reinterpret_cast<const uint4*>(p);
    return v;
}
template <typename T> __device__ __forceinline__ void store_vec(T* p, const Vec16<T>& v) {
    *reinterpret_cast<uint4*>(p) = v.u;
}

// What lanes of a wave have written to LDS that only this wave uses is there for its other lanes, and what they have read may be
// overwritten.  The hardware keeps a wave's LDS accesses in order; the fence keeps the compiler from moving one across this
// point (a wave barrier alone says nothing about memory).  It orders LDS only: one over all memory, or two of them, cost the
// joins of streaming 1x1 convolutions at K = 128 3%.
__device__ __forceinline__ void wave_lds_handover() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// Shard and rows [r0, r1) of block b of a row cut.  b is uniform over the workgroup; the search is unrolled over
// scalar loads of the kernel's arguments (a loop of dependent loads would cost their latency per shard).
__device__ __forceinline__ int shard_of_block(const RowCut& c, int b) {
    int s = 0;
    if (c.p > 1) {
        #pragma unroll
        for (int i = 1; i < kMaxP; ++i) s = (i < c.p && b >= c.blk0[i]) ? i : s;
    }
    return s;
}
__device__ __forceinline__ int locate_block(const RowCut& c, int b, int& r0, int& r1) {
    const int s = shard_of_block(c, b);
    r0 = c.row0[s] + (b - c.blk0[s]) * c.rows_per_block;
    const int end = c.row0[s + 1];
    r1 = r0 + c.rows_per_block < end ? r0 + c.rows_per_block : end;
    return s;
}

}  // namespace edl
