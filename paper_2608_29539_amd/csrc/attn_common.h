// attn_common.h -- device helpers shared by the attention kernels (forward
// and backward): vector types, lane-pair reductions, raw buffer descriptors,
// global -> LDS loads, the LDS transpose read and bf16 packing.  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace logo {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr float kNegInf = -__builtin_inff();

// Value of the partner lane (l ^ 32) and own value, combined.
__device__ __forceinline__ float pair_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Wave-uniform value, made explicit so the compiler keeps it in SGPRs.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Buffer resource word 3 for raw (untyped, stride 0) buffer loads.
constexpr int kRawBufferFlags = 0x00020000;

// Raw buffer descriptor over nbytes (>= 0) bytes from p: loads at or past
// nbytes return zeros.  Words: base address (48 bits, stride 0), size, flags.
__device__ __forceinline__ u32x4 raw_rsrc(const void *p, int nbytes) {
    const uint64_t a = (uint64_t)p;
    u32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) & 0xFFFFu;
    r[2] = __builtin_amdgcn_readfirstlane(nbytes);
    r[3] = kRawBufferFlags;
    return r;
}

// One 16-byte-per-lane global -> LDS load (buffer_load_dwordx4 ... lds: lane
// i writes the 16 bytes at lds + 16 i).  Issued as inline assembly so that
// the compiler does not make every later LDS read wait for it: the buffer it
// fills is only read after the wait + barrier that ends the pipeline step.
// M0 (the LDS base of the load) is saved and restored around it.
__device__ __forceinline__ void lds_load16_at(u32x4 r, uint32_t lds, int voffset) {
    const uint32_t lds_addr = __builtin_amdgcn_readfirstlane(lds);
    uint32_t saved;
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %1\n\t"
        "s_nop 0\n\t"
        "buffer_load_dwordx4 %2, %3, 0 offen lds\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "s"(lds_addr), "v"(voffset), "s"(r)
        : "memory");
}
// LDS address (byte offset in the workgroup's LDS) of a shared object.
__device__ __forceinline__ uint32_t lds_addr_of(const void *lds) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)lds;
}
__device__ __forceinline__ void lds_load16(u32x4 r, const void *lds, int voffset) {
    lds_load16_at(r, lds_addr_of(lds), voffset);
}

// The same with 4 bytes per lane (lane i writes the 4 bytes at lds + 4 i).
__device__ __forceinline__ void lds_load4_at(u32x4 r, uint32_t lds, int voffset) {
    const uint32_t lds_addr = __builtin_amdgcn_readfirstlane(lds);
    uint32_t saved;
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %1\n\t"
        "s_nop 0\n\t"
        "buffer_load_dword %2, %3, 0 offen lds\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "s"(lds_addr), "v"(voffset), "s"(r)
        : "memory");
}

// s_waitcnt operand that waits for vmcnt = 0 only (lgkmcnt and expcnt at
// their maximum).  Issued through the builtin so the compiler knows that no
// vector-memory load is outstanding afterwards.
constexpr int kWaitVmcnt0 = 0x0F70;

// Completion of this wave's LDS-bound loads, then the workgroup barrier.
__device__ __forceinline__ void dma_wait_barrier() {
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
}

// The same where the kPending newest of this wave's LDS-bound loads may still
// be in flight (kPending < 16): a bare barrier, whose memory fence would wait
// for them.  Every LDS read before it has returned its data already (the
// caller's products took it), and the compiler may not move accesses across.
template <int kPending>
__device__ __forceinline__ void dma_wait_barrier_but() {
    static_assert(kPending >= 0 && kPending < 16, "vmcnt field");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0 | kPending);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// gfx950 LDS transpose read of two 8-byte addresses (8 rows apart in the
// callers' layouts): within each 16-lane group, lane 4b+e receives element e
// of the 4-element rows addressed by lanes b, b+4, b+8, b+12.
__device__ __forceinline__ bf16x8 lds_tr_pair(const void *a0, const void *a1) {
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)a0);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)a1);
    const s16x4 ab[2] = {a, b};
    return __builtin_bit_cast(bf16x8, ab);
}

// Two fp32 -> two bf16 (round to nearest even) in one v_cvt_pk_bf16_f32.
__device__ __forceinline__ bf16x2 cvt_bf16x2(float a, float b) {
    return __builtin_convertvector(f32x2{a, b}, bf16x2);
}
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, cvt_bf16x2(a, b));
}

// Column of the LP matrix that row r of its permuted copy holds: bits 2 and 3
// of r (within its 32-row block) swapped.  With A'[h][r][k] = A[h][k][perm(r)]
// as the A operand of the 32x32x16 MFMA and a lane's Q fragments as the B
// operand, accumulator element 8 j + e of lane (g, m) is output channel
// 16 j + 8 g + e of its 32-channel block for query row m -- the layout of the
// B operand of the next product, so the rounded result replaces the
// fragments directly.
__device__ __forceinline__ int lp_perm(int r) { return (r & ~0xC) | ((r & 4) << 1) | ((r & 8) >> 1); }

}  // namespace
}  // namespace logo
