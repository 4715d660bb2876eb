// Device helpers shared by the GEMM translation units (gfx950): bounds-checked buffer
// loads, the wait counter, and the masked input's sources and split.
#pragma once
#include "common.hpp"

namespace {

constexpr int WAVE = 64;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8_t, v); }

// ------------------------------------------------- bounds-checked buffer loads
// Operands are read with buffer loads whose resource covers exactly the matrix:
// a lane whose row or k lies outside it gets an offset beyond the extent and
// reads zeros, which pads every tail.  A bfloat16 K tile is 64 k = 8 units of 16
// bytes per row.

constexpr int BK = 64;
constexpr uint32_t OOB = 0x80000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ uint4 load16(__amdgpu_buffer_rsrc_t r, uint32_t voff)
{
    u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// waits until at most N of this wave's vector-memory operations are outstanding
template <int N>
__device__ __forceinline__ void wait_vmem()
{
    static_assert(N >= 0 && N < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Where a decode kernel's masked input comes from: NPL bfloat16 planes A
// (plane p at A + p * pstride), or (MASK) float32 X and mask eta, from which the
// kernel forms fl32(X + eta) and its planes itself.
struct SkSrc {
    const uint16_t* A; int64_t lda, pstride;
    const float* X; int64_t ldx;
    const float* eta; int64_t ld_eta;
};

// 8 float32 of the masked input as NPL bfloat16 planes
template <int NPL>
__device__ __forceinline__ void planes_of(const float (&x)[8], uint4 (&q)[NPL])
{
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        if (NPL == 1) {
            reinterpret_cast<uint32_t*>(&q[0])[h] = splitee::bf16x2_rne(x[2 * h], x[2 * h + 1]);
        } else {
            splitee::split3_bf16x2(x[2 * h], x[2 * h + 1], reinterpret_cast<uint32_t*>(&q[0])[h],
                                   reinterpret_cast<uint32_t*>(&q[1])[h], reinterpret_cast<uint32_t*>(&q[2])[h]);
        }
    }
}

}  // namespace
