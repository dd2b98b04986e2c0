// Shared device-side vocabulary of the gfx950 attention kernels: vector types, the CDNA4 matrix
// instructions that both contractions run on, and the lane <-> matrix-element maps they imply.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace flat {

typedef __bf16 bf16;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;

// v_mfma_f32_32x32x16_bf16:  D[32x32] += A[32x16] * B[16x32], one wavefront.
//   A operand: lane l holds row (l % 32), contraction indices 8*(l/32) .. 8*(l/32)+7
//   B operand: lane l holds column (l % 32), contraction indices 8*(l/32) .. 8*(l/32)+7
//   C/D:       lane l holds column (l % 32); register r (0..15) is row 8*(r/4) + 4*(l/32) + (r%4)
__device__ __forceinline__ floatx16 mfma_bf16_32x32x16(bf16x8 a, bf16x8 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// v_mfma_f32_32x32x2_f32:  D[32x32] += A[32x2] * B[2x32].
//   A: lane l holds row (l % 32), contraction index (l / 32);  B: column (l % 32), index (l / 32);
//   C/D as above.
__device__ __forceinline__ floatx16 mfma_f32_32x32x2(float a, float b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Row of the 32x32 accumulator tile held in register r of a lane in wave half `half` (= lane / 32).
__device__ __forceinline__ int acc_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// ds_read_b64_tr_b16: within each group of 16 lanes, lane 4*j + q supplies the address of four
// consecutive 16-bit elements (row j, columns 4q..4q+3 of a 4 x 16 block); lane i receives the four
// elements of column i, one from each row j = 0..3.  It turns a row-major [contraction][column]
// tile in LDS into the "contraction index contiguous per lane" form an MFMA operand needs.
__device__ __forceinline__ bf16x4 lds_read_tr16(const void* lds_ptr) {
    typedef short4v __attribute__((address_space(3))) * lds_s4_ptr;
    short4v t = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(uintptr_t)lds_ptr);
    return __builtin_bit_cast(bf16x4, t);
}

// Same, from a 32-bit LDS byte address.
__device__ __forceinline__ bf16x4 lds_read_tr16_at(int lds_addr) {
    typedef short4v __attribute__((address_space(3))) * lds_s4_ptr;
    short4v t = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(uintptr_t)(uint32_t)lds_addr);
    return __builtin_bit_cast(bf16x4, t);
}

__device__ __forceinline__ bf16x8 concat(bf16x4 lo, bf16x4 hi) {
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    floatx2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));  // v_cvt_pk_bf16_f32, RNE
}

// Combine a value across the two halves of a wavefront (lanes l and l ^ 32).  v_permlane32_swap
// exchanges the upper half of one register with the lower half of another; fed the same value
// twice it returns {x[l % 32], x[l % 32 + 32]} in some order, and max / + do not care which.
__device__ __forceinline__ float halves_max(float x) {
    uint32_t u = __builtin_bit_cast(uint32_t, x);
    auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ float halves_sum(float x) {
    uint32_t u = __builtin_bit_cast(uint32_t, x);
    auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

// Largest x of a wavefront, in every lane.  (row_ror 8, 4, 2, 1 within 16 lanes)
__device__ __forceinline__ float wave_max(float x) {
    x = halves_max(x);
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    x = __builtin_fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
    x = __builtin_fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x128, 0xf, 0xf, true)));
    x = __builtin_fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x124, 0xf, 0xf, true)));
    x = __builtin_fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x122, 0xf, 0xf, true)));
    return __builtin_fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x121, 0xf, 0xf, true)));
}

// Quotients n / d of 0 <= n < 2^31 by a divisor known when the kernel is launched: mul = ceil(2^(32+shift) / d) with 2^shift < d <=
// 2^(shift+1), so mul < 2^32, mul d - 2^(32+shift) < d <= 2^(shift+1), and the error n (mul d - 2^(32+shift)) / (d 2^(32+shift)) stays below 1 / d.
// A division by a kernel argument takes about 40 dependent scalar instructions (200 cycles at the start of every workgroup), this five.
struct Divisor {
    uint32_t mul;  // 0: d = 1
    int shift;
    explicit Divisor(int d) : mul(0), shift(0) {
        if (d <= 1) return;
        while ((2ll << shift) < d) ++shift;
        mul = (uint32_t)(((1ull << (32 + shift)) + (uint64_t)d - 1) / (uint64_t)d);
    }
    __host__ __device__ int quotient(int n) const { return (int)((uint32_t)(((uint64_t)(uint32_t)n * mul) >> 32) >> shift) + (mul ? 0 : n); }
};

// The lower half's value in both halves.
__device__ __forceinline__ float lower_half(float x) {
    uint32_t u = __builtin_bit_cast(uint32_t, x);
    return __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_permlane32_swap(u, u, false, false)[0]);
}

// One wave-wide global -> LDS copy, 16 bytes per lane: lane l's bytes land at lds_base + 16 l.
// Issued as inline asm so that the compiler does not serialise later LDS reads of OTHER stages
// behind it; completion is awaited explicitly with wait_vm<n>() before the stage is published by
// a barrier.  lds_base must be wave-uniform.  The statement overwrites m0, which the compiler reserves and does
// not accept on a clobber list; the kernels here contain nothing else that lives in m0 (no indirect register
// indexing, no LDS-direct or message instructions), and a host-side test checks the generated assembly for that.
__device__ __forceinline__ void dma16(const void* gbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(voff), "s"(gbase) : "memory");
}
// s_waitcnt vmcnt(CNT) with the other counters left alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14,
// expcnt 6:4, lgkmcnt 11:8).  Emitted through the builtin so that the compiler's own wait bookkeeping
// sees it.
template <int CNT>
__device__ __forceinline__ void wait_vm() {
    static_assert(CNT >= 0 && CNT < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((CNT & 15) | ((CNT >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Slot of 16-byte chunk c of row r in an LDS tile of ROWB-byte rows: c ^ lds_swizzle(r).  The LDS serves 256 bytes per clock: a ds_read_b128
// touches 16 rows at one chunk index per clock, a ds_read_b64_tr_b16 4 rows x 64 bytes; both then hit every bank once.
template <int ROWB>
__device__ __forceinline__ int lds_swizzle(int r) {
    if (ROWB == 64) return (r >> 2) & 3;                                                    // 4 rows per 256 B
    if (ROWB == 128) return (((r >> 1) & 1) << 2) | (((r >> 2) & 1) << 1) | ((r >> 3) & 1);  // 2 rows per 256 B
    return ((r & 3) << 2) | ((r >> 2) & 3);                                                 // rows of 256 B or more
}

// XCD-aware remap of a 1-D grid.  Consecutive workgroup ids are dealt round-robin to the 8 XCDs;
// this makes each XCD own a contiguous range of logical ids, so that the workgroups sharing one
// head's K/V also share one L2.
__device__ __forceinline__ int xcd_logical_block(int bid, int blocks_per_xcd) {
    return (bid & 7) * blocks_per_xcd + (bid >> 3);
}

}  // namespace flat
