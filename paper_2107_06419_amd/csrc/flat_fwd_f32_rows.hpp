// Fused attention forward for gfx950 in fp32 throughout (fp32 MFMA 32x32x2, fp32 probabilities).
// Same dataflow as the bf16 kernel (paper sections 4-5: one pass over blocks of query rows with
// Logit, softmax and Attend interleaved).
#pragma once
#include "flat_common.hpp"

#include <float.h>
#include <math.h>

#include <type_traits>

namespace flat {

// One workgroup owns 32 query rows and its NW wavefronts divide the KEYS: wavefront w takes the 32-key tiles w, w + NW, ...
// and keeps a running result (reference maximum m, row sum l, unnormalised O) of its own; the partial results are merged
// through LDS at the end.
//
// What bounds it: the fp32 matrix pipe.  A 32x32x2 MFMA takes 64 cycles for 4096 flops and a 32 x 32 block of logits needs D of
// them, against about 110 vector instructions, so one wavefront per SIMD keeps the pipe busy if nothing it waits for
// stands between two MFMAs.  Hence:
//   - Tiles are private to a wavefront (no barrier in the loop): 32 keys of K and of V in LDS, one buffer each, filled by
//     global_load_lds.  A buffer is free as soon as its operands sit in registers, so the next tile's loads go out at the
//     start of the phase that multiplies them and have almost two phases (7000 cycles at D = 128) to land.
//   - Two phases per tile: A = Logit(i + 1) with the exponentials of tile i between its MFMAs, B = Attend(i) with the row
//     maximum of tile i + 1 between its MFMAs.  The second half of a phase reads the operands of the other one from LDS.
//   - The contraction index of a product may be permuted, if both operands agree, and so may the rows of its result.  Half h of
//     a wavefront takes head-dim elements 8 g + 4 h .. + 3 of K and Q for four Logit MFMAs (one ds_read_b128 per operand), and
//     row i of accumulator db is head-dim column DB i + db, so one read of DB consecutive values of V serves the DB Attend
//     MFMAs of a key.
//   - The row maximum is exact but lazy: a reference maximum is set 2^4 above the row maximum, and O and l are rescaled only
//     when that is passed (the quotient O / l does not depend on the reference).  So probabilities are at most 1, as with the row
//     maximum itself, and O and l overflow no earlier; and they are at least 2^-4 at the maximum, so values down to the smallest
//     normal floats lose nothing (relative error at values of 2e-38: 1.3e-7, with 2^8 1.2e-6).  Measured against the row maximum
//     as the reference: 16 causal heads of 2049, d = 128, 170.6 -> 163.0 us; 128 x 512 causal 91.6 -> 86.1.
// LDS: chunk c (16 bytes) of K row r lives in slot c ^ (r & 15): a ds_read_b128 touches 16 rows at one chunk index per clock and
// then meets 16 different slots.  V rows are read along the row and need no swizzle.
// Measured: 16 heads of 8192 positions at d = 128 without a mask 128 TFLOP/s, 32 heads of 4096 at d = 64 130 (a large fp32
// matrix product reaches 154 on this card; this loop with loads, operand reads and exponentials taken out 145).  Before, with
// 128-row workgroups around one shared LDS tile and operands read a float at a time: 110 and 113; and short of 1024 such
// workgroups, where the keys were split over unpipelined wavefronts: 16 causal heads of 2049 positions at d = 128 344 -> 163 us,
// 12 heads of 512 at d = 64 21 -> 13 us.
template <int D>
struct F32Cfg {
    static constexpr int ROWB = D * 4;             // bytes of a row
    static constexpr int TILE = 32 * ROWB;         // one 32-key tile of K or V
    static constexpr int CHUNKS = ROWB / 16;
    static constexpr int RPL = 1024 / ROWB;        // rows filled by one wave-wide load
    static constexpr int LOADS = 32 / RPL;         // loads per tile and tensor
    static constexpr int G = D / 8;                // groups of four Logit MFMAs
    static constexpr int DB = D / 32;              // accumulator blocks
    static constexpr int WAVE_LDS = 2 * TILE;
    static constexpr int WAVES_PER_CU = D == 64 ? 8 : 4;                     // two and one per SIMD
    static constexpr int LDS_RESERVED = 160 * 1024 / WAVES_PER_CU;           // of a wavefront: no third one on some SIMDs
};

constexpr float kF32Headroom = 4.0f;  // of the reference maximum above the row maximum, log2 units
constexpr float kF32LargestExponent = 96.0f;  // 2^31 probabilities of 2^96 are still a number

// 32 query rows, row block qt of head bh, by NW wavefronts of a workgroup, this one the wave-th of them, in their part of LDS.  With NW > 1 there
// is one barrier, for the whole workgroup: every other group of NW has to come to one as well.
template <int D, int NW, bool CAUSAL>
__device__ __forceinline__ void f32_rows(char* const smem, const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                                         float* __restrict__ O, int N, int bh, int qt, float c, int wave, int lane) {
    using C = F32Cfg<D>;
    constexpr int G = C::G, DB = C::DB, LOADS = C::LOADS;
    typedef float floatdb __attribute__((ext_vector_type(DB)));
    typedef const floatx4 __attribute__((address_space(3))) * lds_f4_ptr;
    typedef const floatdb __attribute__((address_space(3))) * lds_fdb_ptr;
    const int l32 = lane & 31, half = lane >> 5;
    const size_t head = (size_t)bh * N * D;
    const char* const Kh = (const char*)(K + head);
    const char* const Vh = (const char*)(V + head);
    const int q0 = qt * 32, qrow = q0 + l32;

    const int kv_len = CAUSAL ? min(N, q0 + 32) : N;
    const int n_tiles = (kv_len + 31) / 32;
    const int n_mine = (n_tiles - wave + NW - 1) / NW;  // tiles wave, wave + NW, ... of this wavefront

    // ---- global -> LDS.  Load i of a tile fills rows RPL i .. of it; lane l fills slot l % CHUNKS of row RPL i + l / CHUNKS.
    // Keys beyond N are clamped to the last one; their logits are masked and their values replaced by zeros when the last tile is used.
    const uint32_t lds_k = (uint32_t)(uintptr_t)smem + (uint32_t)wave * C::WAVE_LDS, lds_v = lds_k + C::TILE;
    const int ld_row = lane / C::CHUNKS, ld_slot = lane % C::CHUNKS;
    const int ld_kchunk = (ld_slot ^ ld_row) * 16, ld_vchunk = ld_slot * 16;
    auto load_part = [&](bool is_k, int tile, int i) __attribute__((always_inline)) {
        const int jbase = tile * 32;
        const int row = min(C::RPL * i + ld_row, N - 1 - jbase);
        const char* base = (is_k ? Kh : Vh) + (size_t)jbase * C::ROWB;
        const uint32_t voff = (uint32_t)row * C::ROWB + (uint32_t)(is_k ? ld_kchunk ^ (((C::RPL * i) & 15) * 16) : ld_vchunk);
        dma16(base, voff, (is_k ? lds_k : lds_v) + (uint32_t)i * 1024);
    };
    auto tile_of = [&](int i) __attribute__((always_inline)) { return wave + NW * i; };

    // ---- operands
    floatx4 qf[G], kf[G];
    floatdb vf[16];
    int koff[8];  // lane part of the K reads: chunk 2 g + half of row l32, for g mod 8
#pragma unroll
    for (int g = 0; g < 8; ++g) koff[g] = (int)lds_k + l32 * C::ROWB + (((2 * g + half) ^ (l32 & 15)) << 4);
    const int voff = (int)lds_v + 4 * half * C::ROWB + l32 * DB * 4;
    auto read_k = [&](int g) __attribute__((always_inline)) { kf[g] = *(lds_f4_ptr)(uintptr_t)(uint32_t)(koff[g & 7] + (g >> 3) * 256); };
    auto read_v = [&](int r) __attribute__((always_inline)) {
        vf[r] = *(lds_fdb_ptr)(uintptr_t)(uint32_t)(voff + (8 * (r >> 2) + (r & 3)) * C::ROWB);
    };
    auto fence = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };
    constexpr int kLgkm0 = (63 & 15) | ((63 >> 4) << 14) | (7 << 4) | (0 << 8);  // s_waitcnt lgkmcnt(0), the rest left alone

    floatx16 oacc[DB], xn;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
    float m = -INFINITY, lsum = 0.f;
    float x[16], p[16];  // logits (an array: the vector ALU's copy of an accumulator) and probabilities of the current tile

    auto logit_group = [&](int g, floatx16& s) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) s = mfma_f32_32x32x2(kf[g][e], qf[g][e], s);
    };
    auto attend_key = [&](int r) __attribute__((always_inline)) {
#pragma unroll
        for (int db = 0; db < DB; ++db) oacc[db] = mfma_f32_32x32x2(vf[r][db], p[r], oacc[db]);
    };
    auto exponentiate = [&](int r) __attribute__((always_inline)) {
        p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], c, -m));
        lsum += p[r];
        asm volatile("" : "+v"(p[r]), "+v"(lsum));  // here, between the MFMAs, not where p is used
    };
    // Masked logits leave the row maximum here and the sums in the last tile's exponentials: scaled, -infinity need not stay what
    // it is (scale 0 makes it a NaN).
    auto partly_masked = [&](int tile) __attribute__((always_inline)) { return tile * 32 + 32 > N || (CAUSAL && tile * 32 + 31 > q0); };
    auto visible = [&](int tile, int r) __attribute__((always_inline)) {
        const int key = tile * 32 + acc_row(r, half);
        return key < N && (!CAUSAL || key <= qrow);
    };
    auto mask = [&](int tile, floatx16& s) __attribute__((always_inline)) {
        if (partly_masked(tile)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = visible(tile, r) ? s[r] : -INFINITY;
        }
    };
    // With 512 registers the MFMA accumulators live in the upper half of the file; kept there by name, or the compiler
    // carries them through the lower half around every trip.
    auto keep_high = [&]() __attribute__((always_inline)) {
        if (D == 128) {
#pragma unroll
            for (int db = 0; db < DB; ++db) asm volatile("" : "+a"(oacc[db]));
        }
    };
    // Reference maximum of a row maximum S.  Where c S has steps so coarse (from 1e9) that the headroom is lost and a key's exponent against its
    // own rounded logit overflows, it is the next step up.
    auto reference = [&](float s) __attribute__((always_inline)) {
        const float above = __builtin_fmaxf(s * c + kF32Headroom, -FLT_MAX);  // finite, so that a first tile of -infinity only has weight 0
        return __builtin_fmaf(s, c, -above) > kF32LargestExponent ? __builtin_fmaf(__builtin_fabsf(above), FLT_EPSILON, above) : above;
    };
    // raise the reference maximum where the row maximum s is above it, and bring O and l to it
    auto rescale = [&](float s) __attribute__((always_inline)) {
        const float m_new = s * c > m ? reference(s) : m;
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        lsum *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
        keep_high();
        m = m_new;
    };

    if (n_mine > 0) {
        // ---- prologue: tile 0 and Q arrive together; Logit of tile 0; operands of the first two phases
#pragma unroll
        for (int i = 0; i < LOADS; ++i) load_part(true, tile_of(0), i);
#pragma unroll
        for (int i = 0; i < LOADS; ++i) load_part(false, tile_of(0), i);
        const float* Qr = Q + head + (size_t)min(qrow, N - 1) * D + 4 * half;
#pragma unroll
        for (int g = 0; g < G; ++g) qf[g] = *(const floatx4*)(Qr + 8 * g);
        wait_vm<0>();
        fence();
#pragma unroll
        for (int g = 0; g < G; ++g) read_k(g);
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        fence();
        if (n_mine > 1) {
#pragma unroll
            for (int i = 0; i < LOADS; ++i) load_part(true, tile_of(1), i);
        }
        fence();
#pragma unroll
        for (int r = 0; r < 16; ++r) xn[r] = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g) logit_group(g, xn);
        mask(tile_of(0), xn);
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            x[r] = xn[r];
            asm volatile("" : "+v"(x[r]));
            mx = __builtin_fmaxf(mx, x[r]);
        }
        m = reference(halves_max(mx));
        if (n_mine > 1) {
            wait_vm<0>();
            fence();
#pragma unroll
            for (int g = 0; g < G; ++g) read_k(g);
        }

        // One trip: the two phases of tile i.  `more`: there is a tile i + 2 to fetch K of; without it tile i + 1 is the last
        // one, the only one that can be partly masked.
        auto trip = [&](int i, auto more) __attribute__((always_inline)) {
            // ---- A: Logit of tile i + 1, exponentials of tile i
            __builtin_amdgcn_s_waitcnt(kLgkm0);
            fence();
#pragma unroll
            for (int r = 0; r < 16; ++r) xn[r] = 0.f;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                logit_group(g, xn);
#pragma unroll
                for (int r = g * 16 / G; r < (g + 1) * 16 / G; ++r) exponentiate(r);
                if (more && g < G / 2) {
#pragma unroll
                    for (int k = g * LOADS / (G / 2); k < (g + 1) * LOADS / (G / 2); ++k) load_part(true, tile_of(i + 2), k);
                }
                if (g == G / 2 - 1) {  // V of tile i has landed
                    wait_vm<more ? LOADS : 0>();
                    fence();
                }
                if (g >= G / 2 && g < G * 3 / 4) {
                    constexpr int PER = 16 / (G / 4);
#pragma unroll
                    for (int r = 0; r < PER; ++r) read_v((g - G / 2) * PER + r);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!more) mask(tile_of(i + 1), xn);
            // ---- B: Attend of tile i, row maximum of tile i + 1
            __builtin_amdgcn_s_waitcnt(kLgkm0);
            fence();
            keep_high();
            float mx = -INFINITY, top = 0.f;
            bool risen = false;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                attend_key(r);
                if (r >= 4 && r < 12) {  // the first keys' MFMAs cover the latency of the last Logit MFMA
#pragma unroll
                    for (int k = 2 * (r - 4); k < 2 * (r - 3); ++k) {
                        x[k] = xn[k];
                        asm volatile("" : "+v"(x[k]));
                        mx = __builtin_fmaxf(mx, x[k]);
                    }
                }
                if (r == 13) {
                    top = halves_max(mx);
                    risen = __builtin_amdgcn_ballot_w64(top * c > m) != 0;
                }
                if (r < 8) {
#pragma unroll
                    for (int k = r * LOADS / 8; k < (r + 1) * LOADS / 8; ++k) load_part(false, tile_of(i + 1), k);
                }
                if (more && r == 7) {  // K of tile i + 2 has landed
                    wait_vm<LOADS>();
                    fence();
                }
                if (more && r >= 8 && r < 12) {
#pragma unroll
                    for (int g = (r - 8) * G / 4; g < (r - 7) * G / 4; ++g) read_k(g);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (__builtin_expect(risen, 0)) rescale(top);
        };
        int i = 0;
#pragma unroll 1
        for (; i + 2 < n_mine; ++i) trip(i, std::true_type{});
        if (i + 1 < n_mine) trip(i, std::false_type{});
        // ---- the last tile: nothing left to fetch
        wait_vm<0>();
        fence();
#pragma unroll
        for (int r = 0; r < 16; ++r) read_v(r);
        const int last = tile_of(n_mine - 1);
        const bool masked = partly_masked(last);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], c, -m));
            if (masked) p[r] = visible(last, r) ? p[r] : 0.f;
            lsum += p[r];
        }
        if (last * 32 + 32 > N) {  // keys past N add nothing, also where the last row, which their loads were clamped to, is infinite
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int db = 0; db < DB; ++db) vf[r][db] = last * 32 + acc_row(r, half) < N ? vf[r][db] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) attend_key(r);
    }

    // ---- merge: every wavefront leaves (O, m, l) in its own region (layout [value][lane], conflict-free), then each sums
    // a share of the accumulator registers over all wavefronts.  A wavefront without a tile has m = -inf: weight 0.
    lsum = halves_sum(lsum);
    constexpr int SHARE = 16 / NW;  // registers per accumulator block and wavefront
    float inv = 1.0f / lsum;
    floatdb out[SHARE];
    if (NW > 1) {
        constexpr int REGION = C::WAVE_LDS / 4;
        float* const all = (float*)smem;
        float* const mine = all + wave * REGION;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) mine[(db * 16 + r) * 64 + lane] = oacc[db][r];
        mine[DB * 16 * 64 + lane] = m;
        mine[(DB * 16 + 1) * 64 + lane] = lsum;
        __syncthreads();
        float M = -INFINITY, L = 0.f, w[NW];
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            w[v] = all[v * REGION + DB * 16 * 64 + lane];
            M = __builtin_fmaxf(M, w[v]);
        }
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            w[v] = __builtin_amdgcn_exp2f(w[v] - M);
            L += w[v] * all[v * REGION + (DB * 16 + 1) * 64 + lane];
        }
        inv = 1.0f / L;
#pragma unroll
        for (int s = 0; s < SHARE; ++s)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                float acc = 0.f;
#pragma unroll
                for (int v = 0; v < NW; ++v) acc += w[v] * all[v * REGION + (db * 16 + wave * SHARE + s) * 64 + lane];
                out[s][db] = acc * inv;
            }
    } else {
#pragma unroll
        for (int s = 0; s < SHARE; ++s)
#pragma unroll
            for (int db = 0; db < DB; ++db) out[s][db] = oacc[db][s % 16] * inv;
    }
    if (qrow < N) {
        float* const Or = O + head + (size_t)qrow * D;
#pragma unroll
        for (int s = 0; s < SHARE; ++s) {
            const int r = wave * SHARE + s;
            *(floatdb*)(Or + DB * acc_row(r, half)) = out[s];
        }
    }
}

}  // namespace flat
