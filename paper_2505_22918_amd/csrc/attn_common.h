// Building blocks shared by the attention kernels (attn.hip, attn_dense.hip):
// vector types, the LDS geometry of a K / V row, packing, waits and LDS DMAs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rt {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) int32_t* csr_ptr;
typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) uint32_t lds_u32;

constexpr float kJump = 18446744073709551616.0f;  // 2^64: stale-max limit on a probability
constexpr int kOob = 0x40000000;                   // buffer offset past every record: reads zero

// Geometry of one 32-key chunk of K or V in LDS.
template <int D>
struct Geo;
template <>
struct Geo<64> {
    static constexpr int DK = 64;      // Q K^T contraction width (multiple of 16)
    static constexpr int DV = 64;      // rows of O^T (multiple of 32)
    static constexpr int SLOTS = 8;    // 16-byte slots per row
    static constexpr bool SWZ = true;  // XOR-swizzle slots by row
};
template <>
struct Geo<72> {
    static constexpr int DK = 80;
    static constexpr int DV = 96;
    static constexpr int SLOTS = 9;
    static constexpr bool SWZ = false;
};

// K rows: 8 consecutive rows read the same slot -> XOR with r & 7.
template <int D>
__device__ __forceinline__ int kswz(int r) {
    return Geo<D>::SWZ ? (r & 7) : 0;
}
// V rows: a transpose read covers 4 consecutive rows and, per row, the two
// slots s and s ^ 2 -> XOR with {0, 1, 4, 5}[r & 3] keeps the 8 (row, slot)
// pairs of a half-wave on distinct banks.
template <int D>
__device__ __forceinline__ int vswz(int r) {
    return Geo<D>::SWZ ? (((r & 2) << 1) | (r & 1)) : 0;
}

__device__ __forceinline__ float pair_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float pair_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float lo_f(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    const bf16x2 v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding:
// vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] at [15:14]).
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// 16 bytes per lane from buffer `rsrc` at byte offset `voff` into LDS at
// m0 + 16 * lane (buffer_load_dwordx4 ... lds).  m0 is reserved by the compiler
// (never allocated) and is set before every use; this is sound only while the
// compiled code keeps nothing else in m0, which the tests check on the
// assembly of every build.  Issued from inline assembly so
// the compiler neither orders these loads against LDS reads of other stages nor
// waits for them; the kernel waits on the vector-memory counter itself.
__device__ __forceinline__ void dma16(uint32_t lds_addr, int voff, i32x4 rsrc) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "buffer_load_dwordx4 %1, %2, 0 offen lds"
        :
        : "s"(lds_addr), "v"(voff), "s"(rsrc)
        : "memory");
}

// Four such loads at byte offsets voff + 1024 n into LDS m0 + 1024 n + 16 * lane,
// n = 0..3: the instruction offset moves both the source and the LDS destination.
__device__ __forceinline__ void dma16x4(uint32_t lds_addr, int voff, i32x4 rsrc) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "buffer_load_dwordx4 %1, %2, 0 offen lds\n\t"
        "buffer_load_dwordx4 %1, %2, 0 offen offset:1024 lds\n\t"
        "buffer_load_dwordx4 %1, %2, 0 offen offset:2048 lds\n\t"
        "buffer_load_dwordx4 %1, %2, 0 offen offset:3072 lds"
        :
        : "s"(lds_addr), "v"(voff), "s"(rsrc)
        : "memory");
}

// 16 bytes per lane from buffer `rsrc` at byte offset `voff` into registers.
// The data lands later: the caller waits on the vector-memory counter and
// then passes the value through settle() before reading it.
__device__ __forceinline__ u32x4 vload16(int voff, i32x4 rsrc) {
    u32x4 v;
    asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen" : "=&v"(v) : "v"(voff), "s"(rsrc) : "memory");
    return v;
}
__device__ __forceinline__ void settle(u32x4& v) { asm volatile("" : "+v"(v)); }

__device__ __forceinline__ i32x4 buffer_rsrc(const void* base, int bytes) {
    const uint64_t p = (uint64_t)(uintptr_t)base;
    return i32x4{(int)(uint32_t)p, (int)((uint32_t)(p >> 32) & 0xffffu), bytes, 0x00020000};
}

}  // namespace
}  // namespace rt
