// fp32 attention on the 16-bit matrix pipe: every factor is split into two fp16 pieces.
#include "flat_fwd_f32_rows.hpp"
#include "flat_launch.hpp"

namespace flat {

// x = h + l: h the nearest fp16 to x, l the nearest fp16 to x - h, which has at most 13 significant bits: h + l is x to 2^-23 of it at worst,
// 2^-24.4 in the root mean square (three floats of four are held exactly).  A product of two floats is hh' + (hl' + lh'); ll', left out, is below 2^-22 of it with either sign and 2^-25 in the mean.
// Three fp16 MFMAs of 32x32x16 take 96 cycles for what 8 fp32 MFMAs of 32x32x2 take 512 for.  Their sums are rounded less often than those of the
// latter: every 16 products instead of every two, and products with a lower piece are summed apart.
// Measured error against 64 bits, 86 random problems of 128 to 4096 positions, normal inputs, fp32 MFMAs and this: 2-norm 4.3e-7 and 2.7e-7 on average, the
// smaller one in all of them (0.90 of the other at most); worst row 1.3e-6 and 6.7e-7 (0.84 at most); largest element over the root mean square 7.3e-6 and 4.3e-6
// (in 8 of the 86 the larger one, 1.26 times at most).  With Q three times as large and uniform values 4.6e-7 and 2.2e-7, Q four and K twice as large 1.3e-6 and
// 6.1e-7.  Below 128 positions there is little to gain and at d = 64 little difference in error (32 causal ones 1.7e-7 against 1.6e-7), so f32_rows
// keeps them.  Where it is the less accurate one: rows of few keys or of one heavy key (an element off by a bit more), logits that are almost equal (24 heads, Q
// times 1e-6: 130 to 390 causal positions 1.8e-7 against 1.2e-7 to 1.3e-7; from 1000 on the better one), and values that are (1 +- 0.001, d = 128, 1000 and 2049
// positions without a mask, 1.9e-7 and 2.6e-7 against 1.5e-7 and 2.0e-7).  Query 0 of a causal call, which sees one key, gets that key's value itself.
//
// One workgroup = four wavefronts = RG = 4 / KG blocks of 32 query rows times KG groups of keys.  A step takes 32 KG keys.  All four wavefronts
// fetch them to registers, split them and leave the pieces in LDS, where the layouts and operand reads are those of the bf16 kernel
// (chunks of 16 bytes swizzled by row, V through ds_read_b64_tr_b16), so the splitting (6 vector instructions for two floats) is shared by RG
// wavefronts.  There are two buffers for each tensor and one barrier per step, which has two phases:
//   A: S(i + 1) from the K pieces, with the exponentials of tile i, the pieces of its probabilities, and V(i + 1) on its way into LDS;
//   B: Attend(i) from the V pieces, with the row maximum of tile i + 1 and K(i + 2) on its way into LDS.
// A chunk's next fetch goes out when its registers have been split, one step ahead.  Masks and the reference maximum are those of f32_rows.
//
// What bounds it: the issue of one wavefront's instructions at d = 128, where the registers (O and its small part 128, Q 64) leave room for one
// wavefront per SIMD: 16 heads x 4096 433 us; at d = 64 (two per SIMD) 32 x 4096 431.  Before, with fp32 MFMAs: 1087 and 1050.  16 causal heads x 2049, d = 128,
// 161 -> 93; 256 x 700, d = 64, 279 -> 120.  (Before values were scaled and small ones looked for, 429 and 420: of it 240 and 231 with the MFMAs taken out, 260 and 243 with
// nothing but them and the operand reads.)
// Tried on that: three bf16 pieces and six products (exact splits of any float, 679 and 665 us; errors like these); one accumulator for S with a third piece of Q
// (2^-11 h: 424 and 419, but spills with two key groups); the left-out product added (no smaller error); one buffer per tensor and two barriers per step (439, 442).
//
// What the pieces cannot hold goes to f32_rows, for the 32 RG rows of the workgroup:
//   infinities and NaN, and |x| beyond 65504 (h is infinite, x - h infinite or a NaN, and the result no number);
//   logits where |q|max c d^1/2 >= 2^10 (a key below 2^-14 is off by up to 2^-36, which then moves a logit by 2^-26; q is scaled by row);
//   rows of Q below 2^-88 where the scale is above 2^30 (their power of two would be above 2^100);
//   V whose largest element in the first tile and the last keys is infinite or below 2^-104, or which grows to 8 to 16 times that in between;
//   a column of V with nothing but values below 2^-20 of that element in the rows of the first tile that one wavefront fetches;
//   a scale of 0 with masked keys.
// f32_rows then takes the workgroup's RG row blocks at once, with KG wavefronts each.  Logits, and what the first tile and the last four keys show, are known before
// any work: 16 x 4096, d = 128, padding of -1e5 at the end 1086 us with fp32 MFMAs alone, 1084; 16 causal x 2049 160 and 143, but 256 x 300 130 and 154, for the
// rows that a workgroup of 128 has too many; 128 causal x 512, scale 0, 85 and 102.  What else comes up costs the pass on top, where the results are seen: an infinity in
// the middle 1056 and 1477, 128 causal x 512 85 and 118.  A column at 1e-6 of the others, 16 x 4096, 1076 (1588 before it was looked for in the first tile).
// V is held times the power of two that brings that element to 2^12 .. 2^13.  Elements that are then below 2^-14, a part in 2^26 of it, are off by up to
// 2^-36, so a result that is made of those alone would not be what it was, whatever the keys hold that its row does not see or barely.  Results of 2^-14 and
// more are at most 2^-22 away through them, and so are those of rows that have half of their weight on other keys.  The loop keeps the smallest and the largest
// value by pair of columns (zeros count as small); only if a smaller result stands in a pair with both, V is read once more for the number of small values in
// each column, and the rows go to f32_rows if that many keys may have half of the weight.  Of 16 x 4096, d = 128, 430 us, a column of zeros beside an
// ordinary one takes 530 then, a column 1e-4 of the others 1045 (fp32 MFMAs alone 1086), zeros for half of the values 436.
// Probabilities are held times 2^15 below the reference maximum, the lower piece times 2^11 as those of K and V: weights above 2^-25 of a row's largest have
// all of their bits, smaller ones a step of 2^-48 of it.  Where such weights are all that a column gets (values that select keys) the result is small for
// its zeros, and the rows go to f32_rows as above.
constexpr float kPieceStep = 2048.0f;        // the lower piece is held times this
constexpr float kTopExponent = 15.0f;        // probabilities are held times 2^15
constexpr float kSmallestExact = 0x1p-14f;   // what the pieces hold to all of their bits

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ floatx16 mfma_f16_32x32x16(half8 a, half8 b, floatx16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ half2v pack_f16(float a, float b) {  // to nearest
    const floatx2 v = {a, b};
    return __builtin_convertvector(v, half2v);
}

template <int D, int KG>
struct F32PiecesCfg {
    static constexpr int RG = 4 / KG, BR = 32 * RG, BC = 32 * KG;
    static constexpr int GROWB = 4 * D, ROWB = 2 * D;        // bytes of a row in memory, and of one piece of it in LDS
    static constexpr int CHUNKS = D / 8;                     // of 8 elements
    static constexpr int ROWS = 256 / CHUNKS, CH = BC / ROWS;  // a thread fetches the same chunk of CH rows, ROWS apart
    static constexpr int PIECE = BC * ROWB;
    static constexpr int BUF = 2 * PIECE;                    // both pieces of a tile; buffers: K of even tiles, of odd ones, V of even, of odd
    static constexpr int V_AT = 2 * BUF, LDS_TILES = 4 * BUF;
    static constexpr int LDS_ROWS = 4 * F32Cfg<D>::WAVE_LDS;  // what f32_rows uses
    static constexpr int LDS_BYTES = (LDS_TILES > LDS_ROWS ? LDS_TILES : LDS_ROWS) + 32;  // and two flags of each wavefront
    // in the tiles' place, behind the loop: the largest value of each column and the smallest, or the number of small ones, as each row of threads has found
    // them, and what columns are suspected of
    static constexpr int LARGEST_AT = 0, SMALL_AT = LARGEST_AT + ROWS * D * 4, SUSPECTS_AT = SMALL_AT + ROWS * D * 4;
    static_assert(SUSPECTS_AT + D * 4 <= LDS_BYTES - 32, "no room for them");
};

template <int D, int KG, bool CAUSAL>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void fwd_f32_pieces_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                                                                                       const float* __restrict__ V, float* __restrict__ O, int N,
                                                                                       int n_qtiles, int n_blocks, int blocks_per_xcd, int n_heads,
                                                                                       const Divisor by_qtiles, const Divisor by_heads, float c) {
    using C = F32PiecesCfg<D, KG>;
    constexpr int RG = C::RG, BR = C::BR, BC = C::BC, CH = C::CH, DS = D / 16, DB = D / 32, ROWB = C::ROWB;
    typedef const half8 __attribute__((address_space(3))) * lds_frag_ptr;
    typedef uint4v __attribute__((address_space(3))) * lds_u4_ptr;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    asm("" : "+s"(n_blocks), "+s"(blocks_per_xcd) : "s"(Q), "s"(K), "s"(V), "s"(O), "s"(N), "s"(n_qtiles), "s"(n_heads), "s"(by_qtiles.mul), "s"(by_qtiles.shift),
        "s"(by_heads.mul), "s"(by_heads.shift), "s"(c));
    int bh, qt;
    if (!CAUSAL) {
        const int logical = xcd_logical_block(blockIdx.x, blocks_per_xcd);
        if (logical >= n_blocks) return;
        bh = by_qtiles.quotient(logical);
        qt = logical - bh * n_qtiles;
    } else {
        const int rank = blockIdx.x;
        if (rank >= n_blocks) return;
        const int from_end = by_heads.quotient(rank);
        bh = rank - from_end * n_heads;
        qt = n_qtiles - 1 - from_end;
    }

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = wave % KG, rg = wave / KG;
    const size_t head = (size_t)bh * N * D;
    const char* const Kh = (const char*)(K + head);
    const char* const Vh = (const char*)(V + head);
    const int q0w = qt * BR + 32 * rg, qrow = q0w + l32;
    const int kv_len = CAUSAL ? min(N, qt * BR + BR) : N;
    const int n_tiles = (kv_len + BC - 1) / BC;

    // The lane's number for what follows the loop; with `lane` what that has in common with the start is kept through the loop, some of it in scratch memory.
    auto lane_again = [&]() __attribute__((always_inline)) {
        int l = threadIdx.x & 63;
        asm("" : "+v"(l));
        return l;
    };
    auto fence = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };
    // Barrier for LDS alone: loads to registers stay in flight across it.
    auto meet = [&]() __attribute__((always_inline)) {
        fence();
        __builtin_amdgcn_s_waitcnt((63 & 15) | ((63 >> 4) << 14) | (7 << 4) | (0 << 8));  // lgkmcnt(0), the rest left alone
        __builtin_amdgcn_s_barrier();
        fence();
    };

    // ---- memory -> registers -> pieces in LDS.  Keys past the last one repeat it; they are masked.
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const int ld_row = tid / C::CHUNKS, ld_chunk = tid % C::CHUNKS;
    const uint32_t st = lds0 + ld_row * ROWB + ((ld_chunk ^ lds_swizzle<ROWB>(ld_row)) << 4);  // (the swizzle looks at row bits below 16)
    floatx4 rk[CH][2], rv[CH][2];
    auto fetch_chunk = [&](const char* base, int tile, int i, floatx4 (&raw)[2]) __attribute__((always_inline)) {
        const int first = min(tile, n_tiles - 1) * BC;
        const char* const from = base + (size_t)first * C::GROWB;
        const uint32_t at = (uint32_t)min(C::ROWS * i + ld_row, N - 1 - first) * C::GROWB + (uint32_t)ld_chunk * 32;
        raw[0] = *(const floatx4*)(from + at);
        raw[1] = *(const floatx4*)(from + at + 16);
    };
    auto fetch = [&](const char* base, int tile, floatx4 (&raw)[CH][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < CH; ++i) fetch_chunk(base, tile, i, raw[i]);
    };
    auto bits = [](float x) __attribute__((always_inline)) { return __builtin_bit_cast(uint32_t, x); };
    auto split2 = [&](float a, float b, half2v& h, half2v& l) __attribute__((always_inline)) {
        h = pack_f16(a, b);
        // (x - h, which is exact, as 2^11 x - 2^11 h)
        l = pack_f16(__builtin_fmaf((float)h[0], -kPieceStep, a * kPieceStep), __builtin_fmaf((float)h[1], -kPieceStep, b * kPieceStep));
    };
    auto split_pair = [&](const floatx4& a, const floatx4& b, int e, uint4v (&piece)[2]) __attribute__((always_inline)) {  // pair e of a chunk's four
        half2v h, l;
        split2(e < 2 ? a[2 * e] : b[2 * e - 4], e < 2 ? a[2 * e + 1] : b[2 * e - 3], h, l);
        piece[0][e] = __builtin_bit_cast(uint32_t, h);
        piece[1][e] = __builtin_bit_cast(uint32_t, l);
    };
    auto split8 = [&](const floatx4& a, const floatx4& b, uint4v (&piece)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) split_pair(a, b, e, piece);
    };
    auto store_pieces = [&](const uint4v (&piece)[2], int i, int at) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < 2; ++p) *(lds_u4_ptr)(uintptr_t)(uint32_t)(st + at + p * C::PIECE + i * C::ROWS * ROWB) = piece[p];
    };
    auto store_chunk = [&](const floatx4 (&raw)[2], int i, int at) __attribute__((always_inline)) {
        uint4v piece[2];
        split8(raw[0], raw[1], piece);
        store_pieces(piece, i, at);
    };
    float v_up = 1.f, v_up_step = kPieceStep;  // V is held times v_up
    auto split_values = [&](const floatx4 (&raw)[2], int e, uint4v (&piece)[2]) __attribute__((always_inline)) {  // as split_pair, scaled
        const float a = raw[e / 2][2 * (e % 2)], b = raw[e / 2][2 * (e % 2) + 1];
        const half2v h = pack_f16(a * v_up, b * v_up);
        const half2v l = pack_f16(__builtin_fmaf((float)h[0], -kPieceStep, a * v_up_step), __builtin_fmaf((float)h[1], -kPieceStep, b * v_up_step));
        piece[0][e] = __builtin_bit_cast(uint32_t, h);
        piece[1][e] = __builtin_bit_cast(uint32_t, l);
    };
    floatx4 vmax, vmin;  // largest and smallest of the values fetched, by pair of columns
#pragma unroll
    for (int e = 0; e < 4; ++e) vmax[e] = 0.f, vmin[e] = INFINITY;
    auto extremes_of_pair = [&](const floatx4 (&raw)[2], int e) __attribute__((always_inline)) {
        const float a = raw[e / 2][2 * (e % 2)], b = raw[e / 2][2 * (e % 2) + 1];
        asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(vmax[e]) : "v"(a), "v"(b));  // (fmaxf is two instructions)
        asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(vmin[e]) : "v"(a), "v"(b));
    };

    // ---- operands
    half8 qf[2][DS], kf[3][2], vf[3][2];
    uint32_t koff[DS];
    int voff[DB][2];
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) koff[ds] = lds0 + (kg * 32 + l32) * ROWB + (((2 * ds + half) ^ lds_swizzle<ROWB>(l32)) << 4);
    const int i16 = lane & 15, g16 = lane >> 4;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            const int r = 8 * hi + 4 * (g16 >> 1) + (i16 >> 2);        // row within 16 keys
            const int ch = 4 * db + 2 * (g16 & 1) + ((i16 >> 1) & 1);  // chunk that holds this lane's 4 columns
            voff[db][hi] = (int)lds0 + C::V_AT + (kg * 32 + r) * ROWB + ((ch ^ lds_swizzle<ROWB>(r)) << 4) + (i16 & 1) * 8;
        }
    auto read_k = [&](int ds, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < 2; ++p) kf[ds % 3][p] = *(lds_frag_ptr)(uintptr_t)(uint32_t)(koff[ds] + buf * C::BUF + p * C::PIECE);
    };
    auto read_v = [&](int g, int buf) __attribute__((always_inline)) {  // group g: 16 keys g / DB, 32 columns g mod DB
        const int t = g / DB, db = g % DB;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int at = buf * C::BUF + p * C::PIECE + t * 16 * ROWB;
            vf[g % 3][p] = __builtin_bit_cast(half8, concat(lds_read_tr16_at(voff[db][0] + at), lds_read_tr16_at(voff[db][1] + at)));
        }
    };

    // S = xa + 2^-11 xb and O = oacc + 2^-11 osmall: the products of the upper pieces, and those with a lower one.
    floatx16 oacc[DB], osmall[DB], xa, xb;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = osmall[db][r] = 0.f;
    float m, lsum = 0.f, x[16], cq;
    half2v pf[2][8];  // pieces of the probabilities

    auto keep_high = [&]() __attribute__((always_inline)) {  // with 512 registers: see f32_rows
        if (D == 128) {
#pragma unroll
            for (int db = 0; db < DB; ++db) asm volatile("" : "+a"(oacc[db]), "+a"(osmall[db]));
        }
    };
    auto logit_group = [&](int ds) __attribute__((always_inline)) {
        if (D == 128) asm volatile("" : "+a"(qf[0][ds]), "+a"(qf[1][ds]));
        xb = mfma_f16_32x32x16(kf[ds % 3][1], qf[0][ds], xb);
        xa = mfma_f16_32x32x16(kf[ds % 3][0], qf[0][ds], xa);
        xb = mfma_f16_32x32x16(kf[ds % 3][0], qf[1][ds], xb);
    };
    auto attend_group = [&](int g) __attribute__((always_inline)) {
        const int t = g / DB, db = g % DB;
        half8 p[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) p[i][e] = pf[i][4 * t + e / 2][e % 2];
        osmall[db] = mfma_f16_32x32x16(vf[g % 3][0], p[1], osmall[db]);
        oacc[db] = mfma_f16_32x32x16(vf[g % 3][0], p[0], oacc[db]);
        osmall[db] = mfma_f16_32x32x16(vf[g % 3][1], p[0], osmall[db]);
    };
    uint32_t one_one = 0x3c003c00, steps = 0x10001000;  // (in registers: not as inline constants, which do not fill both halves)
    asm("" : "+s"(one_one), "+s"(steps));
    const half2v ones = __builtin_bit_cast(half2v, one_one), small_ones = __builtin_bit_cast(half2v, steps);  // 1 and 1 / kPieceStep
    float psum;  // of a tile's probabilities
    float ex[8][2];
    auto exponentiate = [&](int j) __attribute__((always_inline)) {  // probabilities 2 j and 2 j + 1 of a lane
        ex[j][0] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * j], cq, -m));
        ex[j][1] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * j + 1], cq, -m));
    };
    auto split_probabilities = [&](int j) __attribute__((always_inline)) {
        half2v h, l;
        split2(ex[j][0], ex[j][1], h, l);
        pf[0][j] = h;
        pf[1][j] = l;
        // the sum of what is multiplied, so that an error common to a row's probabilities cancels
        psum = __builtin_amdgcn_fdot2(l, small_ones, j == 0 ? 0.f : psum, false);
        psum = __builtin_amdgcn_fdot2(h, ones, psum, false);
        asm volatile("" : "+v"(pf[0][j]), "+v"(pf[1][j]), "+v"(psum));  // here, between the MFMAs, not where they are used
    };
    auto first_key = [&](int i) __attribute__((always_inline)) { return i * BC + kg * 32; };
    auto mask = [&](int i) __attribute__((always_inline)) {
        const int first = first_key(i);
        if (first + 32 > N || (CAUSAL && first + 31 > q0w)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = first + acc_row(r, half);
                const bool visible = key < N && (!CAUSAL || key <= qrow);
                xa[r] = visible ? xa[r] : -INFINITY;
                xb[r] = visible ? xb[r] : 0.f;
            }
        }
    };
    auto reference = [&](float s) __attribute__((always_inline)) {  // as in f32_rows
        const float above = __builtin_fmaxf(s * cq + (kF32Headroom - kTopExponent), -FLT_MAX);
        return __builtin_fmaf(s, cq, -above) > kF32LargestExponent ? __builtin_fmaf(__builtin_fabsf(above), FLT_EPSILON, above) : above;
    };
    auto rescale = [&](float s) __attribute__((always_inline)) {
        keep_high();
        const float m_new = s * cq > m + kTopExponent ? reference(s) : m;
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        lsum *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha, osmall[db][r] *= alpha;
        keep_high();
        m = m_new;
    };
    // The vector work of a group of MFMAs, spread evenly through it.
    auto spread = [&](auto per_mfma) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x002, per_mfma, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int GA = DS, GB = 2 * DB;  // groups of three MFMAs in phase A and B
    using PerA = std::integral_constant<int, (8 * 11 + 4 * CH * 10 + 3 * GA - 1) / (3 * GA)>;
    using PerB = std::integral_constant<int, (4 * CH * 6 + 24 + 3 * GB - 1) / (3 * GB)>;

    // ---- prologue
    fetch(Kh, 0, rk);
    floatx4 rq[DS][2];
    {
        const float* const Qr = Q + head + (size_t)min(qrow, N - 1) * D + 8 * half;
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            rq[ds][0] = *(const floatx4*)(Qr + 16 * ds);
            rq[ds][1] = *(const floatx4*)(Qr + 16 * ds + 4);
        }
    }
    fetch(Vh, 0, rv);
    // the last four keys, one per wavefront: keys marked as padding by a large number, and values that have grown, are mostly to be seen there
    const size_t last_at = (size_t)max(kv_len - 1 - wave, 0) * C::GROWB + lane * (C::GROWB / 64);
    typedef float lane_part __attribute__((ext_vector_type(D / 64)));
    const lane_part last_k = *(const lane_part*)(Kh + last_at), last_v = *(const lane_part*)(Vh + last_at);
    float kmax = 0.f, v0 = 0.f;
    auto largest_of = [&](const floatx4 (&raw)[CH][2], float& top) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < CH; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(top) : "v"(raw[i][0][e]), "v"(raw[i][1][e]));
    };
    largest_of(rk, kmax);
#pragma unroll
    for (int i = 0; i < CH; ++i) store_chunk(rk[i], i, 0);
    fetch(Kh, 1, rk);
    float qmax = 0.f;
#pragma unroll
    for (int ds = 0; ds < DS; ++ds)
#pragma unroll
        for (int e = 0; e < 4; ++e) qmax = __builtin_fmaxf(__builtin_fmaxf(qmax, __builtin_fabsf(rq[ds][0][e])), __builtin_fabsf(rq[ds][1][e]));
    qmax = halves_max(qmax);
    // each row times the power of two that brings its largest element to 2^12 .. 2^13
    const int shift = min(100, max(-100, 139 - (int)(bits(qmax) >> 23)));
    const float up = __builtin_bit_cast(float, (uint32_t)(127 + shift) << 23);
    cq = c * __builtin_bit_cast(float, (uint32_t)(127 - shift) << 23);
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) {
        uint4v piece[2];
        split8(rq[ds][0] * up, rq[ds][1] * up, piece);
#pragma unroll
        for (int p = 0; p < 2; ++p) qf[p][ds] = __builtin_bit_cast(half8, piece[p]);
    }
    largest_of(rv, v0);
#pragma unroll
    for (int e = 0; e < D / 64; ++e) {
        kmax = __builtin_fmaxf(kmax, __builtin_fabsf(last_k[e]));
        v0 = __builtin_fmaxf(v0, __builtin_fabsf(last_v[e]));
    }
    // (a scale of 0 makes a NaN of the exponents of masked keys; with a scale below 2^30 rows too small for `up` have logits below 2^-35)
    bool unfit = !(qmax * c < (D == 64 ? 128.0f : 90.5f)) || kmax > 65504.0f || (c == 0.f && (CAUSAL || N % BC != 0)) ||
                 (qmax > 0.f && qmax < 0x1p-88f && c > 0x1p30f);
    int* const flags = (int*)(smem + C::LDS_BYTES - 32);
    auto any_unfit = [&]() __attribute__((always_inline)) {  // of the workgroup; the flags are written on the way into a barrier
        return (flags[0] | flags[1] | flags[2] | flags[3]) != 0;
    };
    auto raise_flag = [&]() __attribute__((always_inline)) {
        const bool any = __builtin_amdgcn_ballot_w64(unfit) != 0;
        if (lane == 0) flags[wave] = any;
    };
    v0 = wave_max(v0);
    if (lane == 0) flags[4 + wave] = (int)bits(v0);
    // A column that has nothing but values below 2^-20 of that, and not only zeros, in the rows of this wavefront: its results would be found too small.
    // (Of a pair of columns the smaller value: either of them.)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float top = 0.f;
#pragma unroll
        for (int i = 0; i < CH; ++i) top = __builtin_fmaxf(top, __builtin_fminf(__builtin_fabsf(rv[i][e / 2][2 * (e % 2)]), __builtin_fabsf(rv[i][e / 2][2 * (e % 2) + 1])));
        uint64_t low = __builtin_amdgcn_ballot_w64(top < v0 * 0x1p-20f), some = __builtin_amdgcn_ballot_w64(top > 0.f);
#pragma unroll
        for (int by = 32; by >= C::CHUNKS; by /= 2) low &= low >> by, some |= some >> by;
        unfit |= (low & some & ((1ull << C::CHUNKS) - 1)) != 0;
    }
    raise_flag();
    meet();
    // V times the power of two that brings the largest value of the first tile and the last keys to 2^12 .. 2^13 (4 if there are zeros only)
    const int v0_exponent = __builtin_amdgcn_readfirstlane(max(max(flags[4], flags[5]), max(flags[6], flags[7]))) >> 23;
    const int v_shift = 139 - (v0_exponent ? v0_exponent : 129);
    v_up = __builtin_bit_cast(float, (127 + v_shift) << 23);
    v_up_step = __builtin_bit_cast(float, (127 + 11 + v_shift) << 23);
    unfit = any_unfit() || (v0_exponent && v0_exponent < 23) || v0_exponent == 255;
    if (!unfit) {
#pragma unroll
        for (int r = 0; r < 16; ++r) xa[r] = xb[r] = 0.f;
        read_k(0, 0);
        read_k(1, 0);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            uint4v piece[2];
#pragma unroll
            for (int e = 0; e < 4; ++e) extremes_of_pair(rv[i], e), split_values(rv[i], e, piece);
            store_pieces(piece, i, C::V_AT);
            store_chunk(rk[i], i, C::BUF);
        }
        fetch(Vh, 1, rv);
        fetch(Kh, 2, rk);
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            if (ds + 2 < DS) read_k(ds + 2, 0);
            logit_group(ds);
        }
        mask(0);
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            x[r] = __builtin_fmaf(xb[r], 1.0f / kPieceStep, xa[r]);
            mx = __builtin_fmaxf(mx, x[r]);
        }
        m = reference(halves_max(mx));
        meet();

        auto trip = [&](int i, auto odd, auto more) __attribute__((always_inline)) {  // odd: i is; more: there is a tile i + 1
            // ---- A
            keep_high();
            if (more) {
#pragma unroll
                for (int r = 0; r < 16; ++r) xa[r] = xb[r] = 0.f;
                read_k(0, 1 - odd);
                read_k(1, 1 - odd);
            }
            constexpr int EXPS = 8 / GA, PAIRS_A = 4 * CH / GA, PAIRS_B = 4 * CH / GB;  // pairs of probabilities, and of V and K, per group
            uint4v piece[2];
#pragma unroll
            for (int j = 0; j < EXPS; ++j) exponentiate(j);
#pragma unroll
            for (int g = 0; g < GA; ++g) {
                if (more) {
                    if (g + 2 < GA)
                        read_k(g + 2, 1 - odd);
                    else
                        read_v(g + 2 - GA, odd);
                    logit_group(g);
                }
#pragma unroll
                for (int j = EXPS * g; j < EXPS * (g + 1); ++j) {
                    if (j + EXPS < 8) exponentiate(j + EXPS);
                    split_probabilities(j);
                }
                if (more) {
#pragma unroll
                    for (int k = PAIRS_A * g; k < PAIRS_A * (g + 1); ++k) {
                        extremes_of_pair(rv[k / 4], k % 4);
                        split_values(rv[k / 4], k % 4, piece);
                        if (k % 4 == 3) {
                            store_pieces(piece, k / 4, C::V_AT + (1 - odd) * C::BUF);
                            fetch_chunk(Vh, i + 2, k / 4, rv[k / 4]);
                        }
                    }
                    spread(PerA{});
                } else {
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (more) {
                mask(i + 1);
            } else {
                read_v(0, odd);
                read_v(1, odd);
            }
            // ---- B
            lsum += psum;
            keep_high();
            float mx = -INFINITY, top = 0.f;
            bool risen = false;
#pragma unroll
            for (int g = 0; g < GB; ++g) {
                if (g + 2 < GB) read_v(g + 2, odd);
                attend_group(g);
                if (more) {
#pragma unroll
                    for (int k = PAIRS_B * g; k < PAIRS_B * (g + 1); ++k) {
                        split_pair(rk[k / 4][0], rk[k / 4][1], k % 4, piece);
                        if (k % 4 == 3) {
                            store_pieces(piece, k / 4, odd * C::BUF);
                            fetch_chunk(Kh, i + 3, k / 4, rk[k / 4]);
                        }
                    }
                    if (g >= 1 && g <= GB / 2) {  // the last MFMAs of S have had their latency
#pragma unroll
                        for (int r = 16 * (g - 1) / (GB / 2); r < 16 * g / (GB / 2); ++r) {
                            x[r] = __builtin_fmaf(xb[r], 1.0f / kPieceStep, xa[r]);
                            mx = __builtin_fmaxf(mx, x[r]);
                        }
                    }
                    if (g == GB - 1) {
                        top = halves_max(mx);
                        risen = __builtin_amdgcn_ballot_w64(top * cq > m + kTopExponent) != 0;
                    }
                    spread(PerB{});
                }
            }
            if (more) {
                keep_high();
                if (__builtin_expect(risen, 0)) rescale(top);
            }
            meet();
        };
        using Even = std::integral_constant<int, 0>;
        using Odd = std::integral_constant<int, 1>;
        int i = 0;
#pragma unroll 1
        for (; i + 2 < n_tiles; i += 2) {
            trip(i, Even{}, std::true_type{});
            trip(i + 1, Odd{}, std::true_type{});
        }
        if (i + 1 < n_tiles) {
            trip(i, Even{}, std::true_type{});
            trip(i + 1, Odd{}, std::false_type{});
        } else {
            trip(i, Even{}, std::false_type{});
        }

        // ---- results: key groups meet in LDS, in the lane layout they have; each merges its share of the columns
        constexpr int QUADS = D / 8, OQ = QUADS / KG;
        const float total = halves_sum(lsum), v_down = __builtin_bit_cast(float, (127 - v_shift) << 23);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] = __builtin_fmaf(osmall[db][r], 1.0f / kPieceStep, oacc[db][r]);
        floatx4 out[OQ];
        float weights = total;  // of a row's keys, the largest at most 2^kTopExponent
        if (KG > 1) {
            floatx4* const part = (floatx4*)smem + lane;
            float* const stat = (float*)(smem + 4 * QUADS * 1024) + lane;
#pragma unroll
            for (int q = 0; q < QUADS; ++q) part[(wave * QUADS + q) * 64] = floatx4{oacc[q / 4][4 * (q % 4)], oacc[q / 4][4 * (q % 4) + 1], oacc[q / 4][4 * (q % 4) + 2], oacc[q / 4][4 * (q % 4) + 3]};
            stat[wave * 64] = half ? total : m;
            meet();
        }
        if (KG > 1) {
            const floatx4* const part = (const floatx4*)smem + lane;
            const float* const stat = (const float*)(smem + 4 * QUADS * 1024) + lane;
            float M = -FLT_MAX, L = 0.f, w[KG];
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                w[k] = stat[(rg * KG + k) * 64 - 32 * half];
                M = __builtin_fmaxf(M, w[k]);
            }
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                w[k] = __builtin_amdgcn_exp2f(w[k] - M);
                L += w[k] * stat[(rg * KG + k) * 64 + 32 * (1 - half)];
            }
            weights = L;
            const float inv = 1.0f / L;
#pragma unroll
            for (int i = 0; i < OQ; ++i) {
                floatx4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < KG; ++k) {
                    const floatx4 o = part[((rg * KG + k) * QUADS + kg * OQ + i) * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[e] += w[k] * o[e];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) out[i][e] = a[e] * inv;
            }
        } else {
            const float inv = 1.0f / total;
#pragma unroll
            for (int q = 0; q < OQ; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) out[q][e] = oacc[q / 4][4 * (q % 4) + e] * inv;
        }
#pragma unroll
        for (int q = 0; q < OQ; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) unfit |= !(__builtin_fabsf(out[q][e]) < INFINITY);
        const float limit = kSmallestExact * v_down;
        const bool suspect = __builtin_fminf(__builtin_fminf(vmin[0], vmin[1]), __builtin_fminf(vmin[2], vmin[3])) < limit;
        const int state = (__builtin_amdgcn_ballot_w64(unfit) != 0 ? 1 : 0) | (__builtin_amdgcn_ballot_w64(suspect) != 0 ? 2 : 0);
        if (lane == 0) flags[wave] = state;
        meet();
        const int states = flags[0] | flags[1] | flags[2] | flags[3];
        unfit = (states & 1) != 0;
        if (__builtin_expect(states == 2, 0)) {
            float* const largest = (float*)(smem + C::LARGEST_AT);
            float* const small = (float*)(smem + C::SMALL_AT);
            float* const suspects = (float*)(smem + C::SUSPECTS_AT);
            auto leave = [&](float* at, const floatx4& lo, const floatx4& hi) __attribute__((always_inline)) {
                *(floatx4*)(at + ld_row * D + 8 * ld_chunk) = lo;
                *(floatx4*)(at + ld_row * D + 8 * ld_chunk + 4) = hi;
            };
            // a small result in a column whose n small values may have half of the row's weight between them (n: suspects[column])
            auto any_harmed = [&](int at) __attribute__((always_inline)) {
                bool mine = false;
#pragma unroll
                for (int q = 0; q < OQ; ++q) {
                    const floatx4 n = *(const floatx4*)(suspects + 8 * (kg * OQ + q) + 4 * half);
#pragma unroll
                    for (int e = 0; e < 4; ++e) mine |= __builtin_fabsf(out[q][e]) < kSmallestExact && n[e] * 0x1p16f > weights;
                }
                const bool any = __builtin_amdgcn_ballot_w64(mine) != 0;
                if (lane == 0) flags[at + wave] = any;
                meet();
                return (flags[at] | flags[at + 1] | flags[at + 2] | flags[at + 3]) != 0;
            };
            leave(largest, vmax.xxyy, vmax.zzww);
            leave(small, vmin.xxyy, vmin.zzww);
            meet();
            if (tid < D) {
                float top = 0.f, low = INFINITY;
#pragma unroll
                for (int r = 0; r < C::ROWS; ++r) {
                    top = __builtin_fmaxf(top, largest[r * D + tid]);
                    low = __builtin_fminf(low, small[r * D + tid]);
                }
                suspects[tid] = top > 0.f && low < limit ? INFINITY : 0.f;
            }
            meet();
            if (any_harmed(4)) {
                floatx4 hi[2], n[2];
#pragma unroll
                for (int e = 0; e < 4; ++e) hi[0][e] = hi[1][e] = n[0][e] = n[1][e] = 0.f;
#pragma unroll 4
                for (int key = ld_row; key < kv_len; key += C::ROWS) {
                    const char* const from = Vh + (size_t)key * C::GROWB + ld_chunk * 32;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const floatx4 x = *(const floatx4*)(from + 16 * i);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            hi[i][e] = __builtin_fmaxf(hi[i][e], __builtin_fabsf(x[e]));
                            n[i][e] += __builtin_fabsf(x[e]) < limit ? 1.f : 0.f;
                        }
                    }
                }
                leave(largest, hi[0], hi[1]);
                leave(small, n[0], n[1]);
                meet();
                if (tid < D) {
                    float top = 0.f, all = 0.f;
#pragma unroll
                    for (int r = 0; r < C::ROWS; ++r) {
                        top = __builtin_fmaxf(top, largest[r * D + tid]);
                        all += small[r * D + tid];
                    }
                    suspects[tid] = top > 0.f ? all : 0.f;
                }
                meet();
                unfit = any_harmed(0);
            }
        }
        const int row = q0w + (lane_again() & 31);
        if (!unfit && row < N) {
            float* const Or = O + head + (size_t)row * D + 4 * half;
            if (CAUSAL && row == 0) {  // of its one key, which the pieces may hold to a bit less
                const float* const Vr = V + head + 4 * half;
#pragma unroll
                for (int q = 0; q < OQ; ++q) *(floatx4*)(Or + 8 * (kg * OQ + q)) = *(const floatx4*)(Vr + 8 * (kg * OQ + q));
            } else {
#pragma unroll
                for (int q = 0; q < OQ; ++q) *(floatx4*)(Or + 8 * (kg * OQ + q)) = out[q] * v_down;
            }
        }
    }
    if (__builtin_expect(unfit, 0)) {  // of the whole workgroup
        __syncthreads();
        if (q0w < N)
            f32_rows<D, KG, CAUSAL>(smem + rg * KG * F32Cfg<D>::WAVE_LDS, Q, K, V, O, N, bh, qt * RG + rg, c, kg, lane_again());
        else if (KG > 1)
            __syncthreads();  // the one in f32_rows
    }
}

template <int D, int KG, bool CAUSAL>
hipError_t launch_fwd_f32_pieces(const float* Q, const float* K, const float* V, float* O, int BH, int N, float scale, hipStream_t stream) {
    using C = F32PiecesCfg<D, KG>;
    const int n_qtiles = (N + C::BR - 1) / C::BR;
    if ((long long)BH * n_qtiles > 0x7ffffff0LL) return hipErrorInvalidValue;
    const int n_blocks = BH * n_qtiles, blocks_per_xcd = (n_blocks + 7) / 8;
    auto kern = fwd_f32_pieces_kernel<D, KG, CAUSAL>;
    static std::atomic<uint64_t> attr_done{0};
    const hipError_t e = allow_dynamic_lds((const void*)kern, C::LDS_BYTES, &attr_done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(blocks_per_xcd * 8), dim3(256), C::LDS_BYTES, stream, Q, K, V, O, N, n_qtiles, n_blocks, blocks_per_xcd, BH,
                       Divisor(n_qtiles), Divisor(BH), scale * kLog2e);
    return hipGetLastError();
}

#define FLAT_INSTANTIATE_F32_PIECES(D, KG)                                                                                              \
    template hipError_t launch_fwd_f32_pieces<D, KG, false>(const float*, const float*, const float*, float*, int, int, float, hipStream_t); \
    template hipError_t launch_fwd_f32_pieces<D, KG, true>(const float*, const float*, const float*, float*, int, int, float, hipStream_t);
FLAT_INSTANTIATE_F32_PIECES(64, 1)
FLAT_INSTANTIATE_F32_PIECES(64, 2)
FLAT_INSTANTIATE_F32_PIECES(128, 1)
FLAT_INSTANTIATE_F32_PIECES(128, 2)

}  // namespace flat
