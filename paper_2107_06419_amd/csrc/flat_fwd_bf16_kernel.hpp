// Fused attention forward for gfx950, bf16 in / fp32 accumulate / bf16 out.
//
// Dataflow (paper sections 4-5: fused Logit-softmax-Attend with a shared outer loop over batch,
// head and blocks of query rows, the two inner loops interleaved):
//   one workgroup = one (batch, head, block of BR query rows); its NW wavefronts own QW = BR/NW
//   rows each.  The key/value sequence is streamed in tiles of 64 keys through a ring of LDS stages
//   (the paper's double-buffered operand tiles, deepened to hide HBM/L2 latency).  Each tile is
//   consumed as two blocks of 32 keys; per block a wavefront computes
//       S^T = K_blk Q^T            (Logit, MFMA 32x32x16 bf16; the transposed product is chosen so
//                                   that a lane owns ONE query column: row max / row sum are then
//                                   in-lane reductions plus one exchange between wave halves)
//       P   = exp2(c S - m)        (row softmax numerator against a reference max m, fp32 -> bf16 RNE)
//       O^T += V_blk^T P^T         (Attend; the accumulator layout of S^T is already the B-operand
//                                   layout of this product, so P never leaves registers;
//                                   V^T operands come from ds_read_b64_tr_b16 on row-major V)
// and only Q, K, V are read and O written: the N x N intermediate never exists off-chip.
// Unlike the paper's row-granularity tile, which keeps a whole R x N logit slab on chip, the row
// max and sum are carried as running values, so on-chip state is independent of N.
//
// Reference max and optimistic exponentiation.  softmax is invariant to the constant subtracted per
// row, so m need not be the exact running maximum.  It starts as the (scaled) logit of the first key of the
// wavefront's first block: key 0, which every query sees, so the row sum is at least 1 relative to it and can never
// underflow (where keys are divided, a share of which the row sees nothing has sum 0 and is left out).  The steady
// state exponentiates against the current m WITHOUT computing the block maximum; a logit far above m
// shows up as a jump of the fp32 row sum (more than kSumJump per lane and block, i.e. some
// probability above 2^10), and only then the block takes the exact path: row maximum, raise m,
// rescale O and l, recompute the block's probabilities from its logits (not from what is left of them in c S - m: the
// first key may be one whose logit says it does not count, -1e9 say, and c S + 1e9 is a multiple of 64).  Probabilities
// therefore stay below 2^14 relative to m, far inside bf16/fp32 range, and for typical data the exact path runs in the first
// blocks only.
#pragma once
#include "flat_common.hpp"
#include "flat_launch.hpp"

#include <float.h>

namespace flat {

constexpr int kLgkm0 = (63 & 15) | ((63 >> 4) << 14) | (7 << 4) | (0 << 8);  // s_waitcnt: lgkmcnt(0), the other counters left alone
constexpr float kSumJump = 16384.0f;  // per lane and 32-key block: 16 probabilities
constexpr float kFar = 1024.0f;  // log2 units: for reference maxima, and keys above them, no larger than this, c S - m holds the logits to 2^-13
constexpr float kLargestExponent = 96.0f;  // 2^31 probabilities of 2^96 are still a number

// Checking build (-DFLAT_SYNC_EVERY_PHASE): nothing is left in flight across a phase of the ring.  Every
// streaming load is awaited in full and fenced by a barrier on both sides, and every LDS operand read is awaited
// before the step goes on.  The release build overlaps these phases and counts on its vmcnt arithmetic and on
// one barrier per tile; the two builds must produce bit-identical results, which a GPU test checks.
#ifdef FLAT_SYNC_EVERY_PHASE
constexpr bool kSyncEveryPhase = true;
#else
constexpr bool kSyncEveryPhase = false;
#endif

// Head dimensions.  D is the head dimension of the tensors in memory (32, 64, 96, 128 or 256); rows in LDS are DP = D rounded
// up to a power of two (96 -> 128, for the swizzle and the streaming loads), the matrix products touch the D columns that
// exist.  (At d = 96, multiplying the padded columns as well, as zeros, cost: 16 heads x 8192 432 us against 402.)
// A tile holds BC keys: 64 (two 32-key blocks), or 32 at d = 256, where 64 keys of K and V would take 64 KiB; a tile
// shape may ask for another multiple of 32 (BCX: 32, 64 or 128) so that this axis of the map space can be measured too.
//
// LDS tile layout.  Rows are stored unpadded (ROWB = 2 DP bytes) because tiles arrive by
// global_load_lds_dwordx4, which writes the 64 lanes of a wavefront to 1024 contiguous LDS bytes
// (lane l at base + 16 l).  Bank conflicts are avoided instead by an XOR swizzle of the 16-byte
// chunk index within a row: chunk c of row r lives in slot c ^ swz(r).  The LDS serves 256 bytes
// per clock: a ds_read_b128 touches 16 rows at one chunk index per clock, a ds_read_b64_tr_b16
// touches 4 rows x 64 bytes; swz() is chosen so that both patterns hit every bank once.
template <int D, int STAGES, int NW, int BCX = 0>
struct Bf16Cfg {
    static_assert(D == 32 || D == 64 || D == 96 || D == 128 || D == 256, "head dimension not built");
    static constexpr int DP = D == 96 ? 128 : D;      // row length of the tiles in LDS
    static constexpr int BC = BCX ? BCX : bf16_keys_per_tile(D);  // keys per tile
    static constexpr int ROWB = DP * 2;               // bytes per row in LDS
    static constexpr int GROWB = D * 2;               // bytes per row in global memory
    static constexpr int CHUNKS = ROWB / 16;          // 16-byte chunks per LDS row
    static constexpr int GCHUNKS = GROWB / 16;        // ... of which this many exist in memory
    static constexpr int KBYTES = BC * ROWB;
    static constexpr int VBYTES = BC * ROWB;
    static constexpr int STAGE = KBYTES + VBYTES;
    // Where the tiles of a ring stage lie: K beside V, or (d = 256) the K tiles of all stages before the V tiles: each lot is then within the
    // 64 KiB that the offset field of an LDS read reaches, and no address is computed in the loop.
    static constexpr bool SPLIT_RING = DP == 256;
    static constexpr int K_STEP = SPLIT_RING ? KBYTES : STAGE, V_AT = SPLIT_RING ? STAGES * KBYTES : KBYTES;
    static constexpr int ROWS_PER_LOAD = 1024 / ROWB; // rows covered by one wave-wide 16-byte-per-lane load
    static constexpr int LOADS = BC / ROWS_PER_LOAD / NW; // such loads per wavefront per tensor per tile
    static_assert(LOADS >= 1 && LOADS * ROWS_PER_LOAD * NW == BC, "the wavefronts must share a tile's rows evenly");
    static constexpr int LDS_BYTES = STAGES * STAGE;
    __device__ static __forceinline__ int swz(int r) {
        return lds_swizzle<ROWB>(r);
    }
};

constexpr int kMaxSparseTiles = 2048;  // block-sparse: listed tiles per row block that fit the LDS copy of the list (8 KiB)

// Template parameters: D head dimension (32, 64, 96, 128, 256), QB 32-row blocks per wavefront, NW wavefronts per workgroup, STAGES
// depth of the K/V ring, CAUSAL mask, MODE: kDense, kSparse = block-sparse variant (the workgroup visits only the 64-key tiles
// listed for its row block, ids ascending, staged in LDS behind the ring; everything else as in the dense kernel).
// Two wavefronts per SIMD (256 registers each), except 64 rows per wavefront at d = 128 and every shape at d = 256,
// whose accumulators alone need more: those run one wavefront per SIMD with the full 512 registers.  The 128-row shapes of d = 32 leave
// room in LDS for five and are held to the 96 registers that five need.

// Key groups (KG > 1): NW / KG wavefronts' worth of rows per workgroup, the keys of every tile divided over KG wavefronts per row
// block.  For launches of few rows, which are bound by the chain of steps of one workgroup: KG times fewer steps, paid for
// with K and V read from L2 KG times as often per flop and a merge through LDS (about 1 us).
// kSplit = the keys of one row block are divided over prob.n_splits workgroups, each of which leaves its
// unnormalised result (reference maximum, row sum, accumulators) in a workspace for split_merge_kernel.
constexpr int kDense = 0, kSparse = 1, kSplit = 2;
constexpr bool loops_over_blocks(int d, bool causal, int mode, int key_groups) {
    return mode == kDense && !causal && key_groups == 1 && (d == 96 || d == 128);
}

// How the workgroups of a launch are numbered: n_blocks = n_heads * n_qtiles, n_qtiles = row blocks (times splits) per head.  stride:
// workgroups launched per XCD; the workgroup in position t of an XCD takes blocks t, t + stride, ... of it.
struct LaunchGrid {
    int n_qtiles, n_blocks, blocks_per_xcd, stride, n_heads, n_row_blocks;
    int xcd_range, head_step, xcd_head;  // without a mask: XCD x takes block t as number x xcd_range + t, whose head h stands for head_step h + x xcd_head
    Divisor by_qtiles, by_heads, by_splits, by_heads_per_batch;
};

template <int D, int QB, int NW, int STAGES, bool CAUSAL, int MODE = kDense, int BCX = 0, int KG = 1>
__global__ __launch_bounds__(64 * NW, (D == 256 || (D == 128 && QB == 2)) ? 1 : D == 32 && QB == 1 && NW == 4 && KG == 1 ? 5 : 2) void fwd_bf16_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ K,
                                                          const bf16* __restrict__ V, bf16* __restrict__ O,
                                                          const Bf16Problem prob, const LaunchGrid grid, float c) {
    using C = Bf16Cfg<D, STAGES, NW, BCX>;
    constexpr bool SPARSE = MODE == kSparse, SPLIT = MODE == kSplit;
    constexpr int DP = C::DP, QW = 32 * QB, BR = NW / KG * QW, BC = C::BC, DS = D / 16, DB = D / 32;
    constexpr int KBT = BC / 32, KB = KBT / KG;  // 32-key blocks per tile, and of those per wavefront
    constexpr int KB64 = 64 / BC;  // tiles per 64 keys (the unit of a block-sparse list)
    static_assert(NW % KG == 0 && KBT % KG == 0 && D / 8 % KG == 0, "key groups share wavefronts, keys and output columns evenly");
    static_assert(KG == 1 || (!SPARSE && BC % 64 == 0), "the block-sparse variant has one key group");
    static_assert(KB == 1 || KB == 2 || KB == 4, "a wavefront takes one, two or four 32-key blocks of a tile");
    static_assert(!SPARSE || KB64 >= 1, "block-sparse lists name 64-key tiles");
    constexpr int LOADS_PER_TILE = 2 * C::LOADS;  // DMA instructions per wavefront per tile (K and V)
    // With one block per wavefront and tile, a step is done with its V tile and with the NEXT K tile, so K runs one tile
    // ahead of V in the ring: one more tile in flight for the same LDS, and two stages are enough.
    constexpr bool kHigh = D == 256 || (D == 128 && QB == 2);  // one wavefront per SIMD: the accumulators and Q live in the upper half of its 512 registers
    // Which shapes take two_phase_step (below) and which the step that spreads all MFMAs of a block through the softmax of its neighbour.  Two
    // wavefronts of 64 rows per SIMD, or eight wavefronts in lock step, fill each other's gaps in the latter: there two phases are slower (d = 64,
    // 16 heads x 16384 1110 -> 1141 us; d = 96, 768 causal heads x 512 82.1 -> 86.6).  With less to fill gaps with they win: 128-row shapes of d = 64,
    // 64 causal heads x 2048 48.6 -> 46.5, d = 128, 16 heads x 8192 566 -> 551, d = 96 471 -> 463; 64 rows per wavefront at d = 32, 16 heads x 8192
    // 183 -> 178, and at d = 128 (one wavefront per SIMD) 618 -> 490.
    // With one block per wavefront and tile there is no choice: K of a block is gone from the ring when the exact path of the other step asks for it.
    constexpr bool kTwoPhase = KB == 1 || (KB == 2 && (kHigh || (NW > 1 && (D == 32 || (QB == 1 && NW <= 4)))));
    constexpr bool kStagger = kTwoPhase;
    static_assert(STAGES >= (KB == 1 ? 2 : 3), "the ring is too short to keep a tile in flight");
    extern __shared__ __attribute__((aligned(16))) char smem[];

    // Which (head, row block) this workgroup takes.  Workgroup ids are dealt round-robin to the 8 XCDs, so XCD x
    // sees the ids x, x+8, ...: position t = id / 8 of its own sequence.
    // Without a mask all blocks cost the same: XCD x takes the contiguous range [x, x+1) * blocks_per_xcd of
    // (head, row block) pairs, so that the workgroups sharing one head's K/V share one L2.
    // With the causal mask row block q costs ~ q+1 tiles, and the order decides the load balance.  All blocks are
    // ranked heaviest first across ALL heads (rank g = rows-from-the-end * heads + head) and dealt to the XCDs
    // like cards (XCD x gets ranks x, x+8, ...): every XCD gets the same mix, its late, dynamically placed
    // workgroups are the light ones, and with a head count that is a multiple of 8 it still sees only its own
    // heads.  When two workgroups fit a compute unit the hardware places positions t and t+32 of an XCD's
    // sequence on the same unit in the first round; the second half of every 64 positions is therefore taken in
    // reverse, which pairs the k-th heaviest of the 64 with the k-th lightest.
    // Without a mask all blocks are equal, and a workgroup that has its compute unit to itself goes on to another one: nothing else covers the
    // fetch of a block's Q rows and first tile (8000 of 41000 cycles at d = 128 and 512 keys), so the next block's go out before the results of
    // this one are put together.  (How many: launch_cfg.)  At d = 64 and 32 a second workgroup covers it, and the loop costs registers (16 x 16384, d = 64, 977 -> 1019 us); at d = 256 Q goes to
    // registers the accumulators' store still needs (256 x 128 16.5 -> 17.2 us).  Key counts that differ leave the dealing to the hardware.
    constexpr bool kLoop = loops_over_blocks(D, CAUSAL, MODE, KG);
    static_assert(!(CAUSAL && SPARSE), "the block-sparse variant has no causal form");
    // All arguments in one round trip: left alone, the compiler fetches some, waits, divides, and fetches the rest (a first workgroup
    // of a compute unit pays about 600 cycles for each).
    const int n_qtiles = grid.n_qtiles, blocks_per_xcd = grid.blocks_per_xcd;
    int n_blocks = grid.n_blocks, xcd_range = grid.xcd_range;
    asm("" : "+s"(n_blocks), "+s"(xcd_range) : "s"(Q), "s"(K), "s"(V), "s"(O), "s"(prob.Nq), "s"(prob.Nk), "s"((uint64_t)prob.kv_lens), "s"(prob.causal_offset), "s"(n_qtiles),
        "s"(blocks_per_xcd), "s"(grid.n_heads), "s"(grid.head_step), "s"(grid.xcd_head), "s"(grid.by_qtiles.mul), "s"(grid.by_qtiles.shift), "s"(grid.by_heads_per_batch.mul), "s"(grid.by_heads_per_batch.shift), "s"(c));
    int bh, qt, block_of_xcd = blockIdx.x >> 3;
    if (!CAUSAL) {
        // Where key counts differ and a range of heads is one batch entry or two, an XCD takes every eighth head instead: 8 entries of 16 heads,
        // 300 rows over 1000 to 2000 keys, d = 64, 36.4 -> 33.1 us; 8 x 25 heads, 500 over 750 to 1500, d = 128, 87.5 -> 80.9.  With 16 entries
        // and more the ranges are even enough (within 2 % either way), and few heads that eight does not divide would be dealt unevenly.
        const int x = blockIdx.x & 7, logical = x * xcd_range + block_of_xcd, head = grid.by_qtiles.quotient(logical);
        bh = head * grid.head_step + x * grid.xcd_head;
        if (bh >= grid.n_heads) return;
        qt = logical - head * n_qtiles;
    } else {
        constexpr int kByLds = (160 * 1024) / bf16_lds_bytes(D, QB, NW, STAGES, BCX, KG), kByRegs = 8 / NW;  // two wavefronts per SIMD
        constexpr bool kTwoPerUnit = (kByLds < kByRegs ? kByLds : kByRegs) == 2;
        const int x = blockIdx.x & 7, t = blockIdx.x >> 3;
        int r = t;
        if (kTwoPerUnit && (t | 63) < blocks_per_xcd && (t & 32)) r = (t & ~31) + 31 - (t & 31);
        const int g = 8 * r + x;
        if (g >= n_blocks) return;
        const int from_end = grid.by_heads.quotient(g);
        bh = g - from_end * grid.n_heads;
        qt = n_qtiles - 1 - from_end;
    }

    int split = 0;
    if (SPLIT) {  // the launch counts (row block, split) pairs per head; the splits of a row block are neighbours
        const int block = grid.by_splits.quotient(qt);
        split = qt - block * prob.n_splits;
        qt = block;
    }
    // (the wavefront's number as a scalar: what follows from it is then computed once per wavefront, not in its lanes.  12 heads x 512, d = 64,
    // 5.12 -> 4.91 us; 8 x 1001, d = 128, 10.96 -> 10.59; 768 causal heads x 512, d = 64, 55.0 -> 52.1.)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    // Nq query rows per head; N = number of keys of this head that count (the padded tail of a shorter batch
    // entry is masked like the tail of a ragged tile); causal: query i sees keys 0 .. i + off.
    const int Nq = prob.Nq, off = prob.causal_offset;
    // Key groups: wavefronts rg * KG + kg, kg = 0 .. KG-1, own the same QW query rows and take KB of every tile's blocks each.
    const int kg = KG == 1 ? 0 : wave % KG, rg = KG == 1 ? wave : wave / KG;
    int N, q0w;
    const char *Qh, *Kh, *Vh;
    bf16* Oh;
    auto place = [&]() __attribute__((always_inline)) {  // of block (bh, qt)
        N = prob.Nk;
        if (prob.kv_lens) N = max(1, min(prob.Nk, prob.kv_lens[grid.by_heads_per_batch.quotient(bh)]));
        const size_t head_q = (size_t)bh * Nq * D, head_k = (size_t)bh * prob.Nk * D;
        Qh = (const char*)(Q + head_q);
        Kh = (const char*)(K + head_k);
        Vh = (const char*)(V + head_k);
        Oh = O + head_q;
        q0w = qt * BR + rg * QW;
    };
    place();

    // Block-sparse: copy this row block's tile list into LDS (ids forced into range; a wrong list can give a
    // wrong result but no stray access).
    int* const sp_ids = (int*)(smem + C::LDS_BYTES);
    int sp_count = 0;
    if (SPARSE) {
        const int n_ktiles = (N + 63) / 64;  // list entries name 64-key tiles
        const int row_block = bh * ((Nq + 255) / 256) + (qt * BR) / 256;  // lists are per 256 query rows; BR divides 256
        const int lo = max(0, min(prob.n_tile_ids, prob.tile_offsets[row_block]));
        const int hi = max(lo, min(prob.n_tile_ids, prob.tile_offsets[row_block + 1]));
        sp_count = min(hi - lo, kMaxSparseTiles);
        for (int i = tid; i < sp_count; i += 64 * NW) sp_ids[i] = max(0, min(n_ktiles - 1, prob.tile_ids[lo + i]));
        __syncthreads();
    }
    // Split keys: this workgroup takes tiles [t0, t0 + tiles_per_split) of those its row block sees.
    int kv_len = N;
    if (CAUSAL) kv_len = min(N, qt * BR + BR + off);
    const int t0 = SPLIT ? split * prob.tiles_per_split : 0;
    // j-th tile this workgroup visits (a listed 64-key tile is KB64 consecutive tiles)
    auto tile_of = [&](int j) __attribute__((always_inline)) {
        if (SPLIT) return t0 + j;
        if (!SPARSE) return j;
        return KB64 == 1 ? sp_ids[j] : sp_ids[j / KB64] * KB64 + j % KB64;
    };

    float m[QB];          // reference max of each row, set in the prologue below
    bf16x8 qf[QB][DS];    // Q^T fragments (B operand of S^T = K Q^T): column = query, 8 consecutive head-dim elements

    floatx16 oacc[QB][DB];
    float lsum[QB];

    const int n_tiles_seen = (kv_len + BC - 1) / BC;  // tiles the row block sees
    int n_tiles = SPARSE ? sp_count * KB64                                              // tiles this workgroup visits
                        : SPLIT ? max(0, min(n_tiles_seen - t0, prob.tiles_per_split)) : n_tiles_seen;

    // ---- global -> LDS streaming.  Wave w issues load i of a tile for the 1024-byte LDS block
    // (NW i + w); lane l fills slot (l % CHUNKS) of row (l / CHUNKS) of that block, so it fetches
    // the chunk whose swizzled position that is (for a padded head dimension, a chunk that does not
    // exist in memory is replaced by one of the same row that does: its content never matters).
    // Keys beyond N are clamped to the last key: their logits are masked and their (finite) values
    // meet a zero probability.
    const uint32_t smem_base = (uint32_t)(uintptr_t)smem;
    int ld_row[C::LOADS], ld_chunk_off[C::LOADS];
#pragma unroll
    for (int i = 0; i < C::LOADS; ++i) {
        ld_row[i] = (NW * i + wave) * C::ROWS_PER_LOAD + lane / C::CHUNKS;
        const int chunk = (lane % C::CHUNKS) ^ C::swz(ld_row[i]);
        ld_chunk_off[i] = (chunk < C::GCHUNKS ? chunk : chunk - (C::CHUNKS - C::GCHUNKS)) * 16;
    }
    auto issue_tile_loads = [&](int j, int stage, bool k_tile = true, bool v_tile = true) __attribute__((always_inline)) {  // j-th visited tile, stage = j % STAGES
        const uint32_t stage_base = smem_base + (uint32_t)stage * C::K_STEP;
        const int tile = tile_of(j);
#pragma unroll
        for (int i = 0; i < C::LOADS; ++i) {
            const int key = min(tile * BC + ld_row[i], N - 1);
            const uint32_t voff = (uint32_t)key * C::GROWB + ld_chunk_off[i];
            const uint32_t lds_k = __builtin_amdgcn_readfirstlane(stage_base + (NW * i + wave) * 1024);
            if (k_tile) dma16(Kh, voff, lds_k);
            if (v_tile) dma16(Vh, voff, lds_k + C::V_AT);
        }
    };

    // per-lane LDS byte addresses of the MFMA operand reads (ring base + row part + swizzled chunk), one per
    // compile-time chunk index
    int koff[DS];
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) koff[ds] = (int)smem_base + (kg * KB * 32 + l32) * C::ROWB + (((2 * ds + half) ^ C::swz(l32)) << 4);
    const int i16 = lane & 15, g16 = lane >> 4;
    int voff[DB][2];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            const int r = 8 * hi + 4 * (g16 >> 1) + (i16 >> 2);         // row within a 16-key step
            const int ch = 4 * db + 2 * (g16 & 1) + ((i16 >> 1) & 1);  // 16-byte chunk holding this lane's 4 columns
            voff[db][hi] = (int)smem_base + (C::SPLIT_RING ? C::V_AT : 0) + (kg * KB * 32 + r) * C::ROWB + ((ch ^ C::swz(r)) << 4) + (i16 & 1) * 8;
        }
    const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};

    // ---- block = 32 keys.  Pieces of the per-block work; the main loop below software-pipelines them so
    // that the matrix pipe works on PV of block b-1 and on S of block b+1 while the vector ALU does the
    // softmax of block b.
    // (stage, kb) locate a block: ring stage of its tile and which half of the tile.  In the unrolled main loop
    // both are compile-time constants and fold into the immediate offsets of the LDS reads.
    auto read_k = [&](int stage, int kb, bf16x8 (&kf)[DS]) __attribute__((always_inline)) {  // K fragments (A operand of S^T = K Q^T) of one block
        typedef const bf16x8 __attribute__((address_space(3))) * lds_frag_ptr;
        const int block_off = stage * C::K_STEP + kb * 32 * C::ROWB;
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            // Declaring the lane offset "modified" keeps (offset + constant) from being hoisted out of the loop
            // into one register per stage; inside the loop the constant folds into the DS offset field.
            asm volatile("" : "+v"(koff[ds]));
            kf[ds] = *(lds_frag_ptr)(uintptr_t)(uint32_t)(koff[ds] + block_off);
        }
    };
    auto read_v = [&](int stage, int kb, bf16x8 (&vf)[2][DB]) __attribute__((always_inline)) {  // V^T fragments (A operand of O^T += V^T P^T)
        const int block_off = stage * C::K_STEP + (C::SPLIT_RING ? 0 : C::V_AT) + kb * 32 * C::ROWB;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            asm volatile("" : "+v"(voff[db][0]), "+v"(voff[db][1]));
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int off = block_off + t * 16 * C::ROWB;  // swz() only looks at row bits below 16
                vf[t][db] = concat(lds_read_tr16_at(voff[db][0] + off), lds_read_tr16_at(voff[db][1] + off));
            }
        }
    };
    auto logits = [&](const bf16x8 (&kf)[DS], floatx16 (&x)[QB]) __attribute__((always_inline)) {  // S^T = K Q^T
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int r = 0; r < 16; ++r) x[qb][r] = 0.f;
#pragma unroll
        for (int ds = 0; ds < DS; ++ds)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) x[qb] = mfma_bf16_32x32x16(kf[ds], qf[qb][ds], x[qb]);
    };
    auto attend = [&](const bf16x8 (&vf)[2][DB], const uint32_t (&p)[QB][8]) __attribute__((always_inline)) {  // O^T += V^T P^T
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    uint4v pw = {p[qb][4 * t], p[qb][4 * t + 1], p[qb][4 * t + 2], p[qb][4 * t + 3]};
                    oacc[qb][db] = mfma_bf16_32x32x16(vf[t][db], __builtin_bit_cast(bf16x8, pw), oacc[qb][db]);
                }
    };
    auto first_key = [&](int blk) __attribute__((always_inline)) { return blk * 32 + acc_row(0, half); };  // of a lane's 16 of a block
    auto is_visible = [&](int first, int qb, int r) __attribute__((always_inline)) {
        const int key = first + acc_row(r, 0);
        return key < N && (!CAUSAL || key <= q0w + 32 * qb + l32 + off);
    };
    // x <- c S - m (masked keys -> -inf)
    auto shift = [&](int blk, bool masked, floatx16 (&x)[QB]) __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float mref = m[qb];
#pragma unroll
            for (int r = 0; r < 16; ++r) x[qb][r] = __builtin_fmaf(x[qb][r], c, -mref);
            if (masked) {
#pragma unroll
                for (int r = 0; r < 16; ++r) x[qb][r] = is_visible(first_key(blk), qb, r) ? x[qb][r] : -INFINITY;  // exp2 -> probability exactly 0
            }
        }
    };
    // p <- bf16(exp2(x)); bsum <- this block's sum of the ROUNDED probabilities (so that the row sum and the
    // Attend operand agree).  One accumulator chain per query block: its links are spread through the step
    // anyway, and a second chain costs more in merging than it gains.
    auto softmax_b = [&](const auto (&x)[QB], uint32_t (&p)[QB][8], float (&bsum)[QB]) __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float l0 = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                float e[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) e[i] = __builtin_amdgcn_exp2f(x[qb][r + i]);
                const uint32_t pk0 = pack_bf16(e[0], e[1]), pk1 = pack_bf16(e[2], e[3]);
                p[qb][r >> 1] = pk0;
                p[qb][(r >> 1) + 1] = pk1;
                l0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk0), ones, l0, false);
                l0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk1), ones, l0, false);
            }
            bsum[qb] = l0;
        }
    };
    // Rare path: raise the reference max of every row whose block maximum lies above it, rescale O and l (by alpha), and leave the block's
    // exponents in x.  This one starts from the logits S: c S - m has lost them if m is the logit of a key far below the others, -1e9 say.  Where
    // c S has steps so coarse (from 1e9) that a key's exponent against its own rounded logit overflows, m is the next step up.
    auto block_max = [&](const auto &x) __attribute__((always_inline)) {
        float top = x[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) top = __builtin_fmaxf(top, x[r]);
        return halves_max(top);
    };
    auto raise_from_logits = [&](int blk, bool masked, auto (&x)[QB], float (&alpha)[QB]) __attribute__((always_inline)) {
        int first = first_key(blk);
        asm("" : "+v"(first));  // or the compiler keeps the comparisons of the step for here
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (masked) x[qb][r] = is_visible(first, qb, r) ? x[qb][r] : -INFINITY;
            const float top = block_max(x[qb]);
            float raised = __builtin_fmaxf(__builtin_fmaxf(m[qb], top * c), -FLT_MAX);
            if (__builtin_fmaf(top, c, -raised) > kLargestExponent) raised = __builtin_fmaf(__builtin_fabsf(raised), FLT_EPSILON, raised);
            alpha[qb] = __builtin_amdgcn_exp2f(m[qb] - raised);
            m[qb] = raised;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float e = __builtin_fmaf(x[qb][r], c, -raised);
                x[qb][r] = masked && x[qb][r] == -INFINITY ? -INFINITY : e;  // (c may be 0)
            }
        }
    };
    auto rescale = [&](const float (&alpha)[QB]) __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            lsum[qb] *= alpha[qb];
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[qb][db][r] *= alpha[qb];
        }
    };
    // ---- prologue.  The workgroup's Q rows arrive through LDS like the tiles: whole rows, 1024 contiguous bytes per load, where
    // fragments straight from memory touch 32 bytes of each of 32 rows per load.  They lie at the end of the ring, and what
    // they leave free in front is filled with the first tiles at once; the rest of the ring follows when the fragments are in
    // registers.  So a workgroup starts after one round trip of Q and the first tile.  768 heads x 512, d = 64: 62 -> 61 us, d = 128
    // 147 -> 139, d = 96 112 -> 109; 8 x 1001, d = 128, 12.6 -> 11.9; 4 x 4096, d = 64, 25.7 -> 24.5.  At d = 256 the 64 KiB of Q take
    // longer into LDS and out again (2 x 8 causal heads of 3001: 130 us straight to registers, 132 through LDS), so they go
    // straight to registers, with the whole ring filled behind them.
    constexpr bool kQThroughLds = D != 256;
    constexpr int kQBytes = kQThroughLds ? BR * C::ROWB : 0;
    constexpr int kQAt = C::LDS_BYTES - kQBytes >= C::STAGE ? C::LDS_BYTES - kQBytes : C::STAGE;
    static_assert(kQAt + kQBytes <= bf16_lds_bytes(D, QB, NW, STAGES, BCX, KG), "the Q rows must fit the LDS a launch asks for");
    static_assert(!SPARSE || kQAt + kQBytes <= C::LDS_BYTES, "the Q rows must not reach the block-sparse list behind the ring");
    constexpr int kEarlyTiles = kQAt / C::STAGE < STAGES - 1 ? kQAt / C::STAGE : STAGES - 1;
    auto load_q = [&]() __attribute__((always_inline)) {
        // (addresses from a lane index the compiler cannot follow, or it keeps them all in registers for the next block)
        int ln = lane;
        if (kLoop) asm volatile("" : "+v"(ln));
        if (kQThroughLds) {
            constexpr int kQLoads = BR / C::ROWS_PER_LOAD;
#pragma unroll
            for (int i = 0; i < (kQLoads + NW - 1) / NW; ++i) {
                const int blk = NW * i + wave;  // 1024-byte block of the Q rows
                if (kQLoads % NW != 0 && blk >= kQLoads) break;
                const int r = blk * C::ROWS_PER_LOAD + ln / C::CHUNKS, chunk = (ln % C::CHUNKS) ^ C::swz(r);
                const int row = min(qt * BR + r, Nq - 1);  // rows past the end repeat the last one; they are never stored
                const uint32_t off_q = (uint32_t)row * C::GROWB + (chunk < C::GCHUNKS ? chunk : chunk - (C::CHUNKS - C::GCHUNKS)) * 16;
                dma16(Qh, off_q, __builtin_amdgcn_readfirstlane(smem_base + kQAt + blk * 1024));
            }
        } else {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int ds = 0; ds < DS; ++ds) {
                    const int row = q0w + 32 * qb + (ln & 31);
                    uint4v z = {0, 0, 0, 0};
                    if (row < Nq) z = *(const uint4v*)(Qh + (size_t)row * C::GROWB + ds * 32 + (ln >> 5) * 16);
                    qf[qb][ds] = __builtin_bit_cast(bf16x8, z);
                }
        }
    };
    auto fill = [&](int t) __attribute__((always_inline)) {
        if (t >= n_tiles) return;
        if (kStagger) {  // K first, in the order the loop goes on with and its wait counts: K(t), V(t), K(t+1), ...
            issue_tile_loads(t, t, true, false);
            if (t < STAGES - 1) issue_tile_loads(t, t, false, true);
        } else {
            issue_tile_loads(t, t);
        }
    };
    auto start_loads = [&]() __attribute__((always_inline)) {
        load_q();
#pragma unroll
        for (int t = 0; t < kEarlyTiles; ++t) fill(t);
    };
    auto await_first = [&]() __attribute__((always_inline)) {
        if (kQThroughLds && !kSyncEveryPhase && n_tiles >= kEarlyTiles)
            wait_vm<(kEarlyTiles - 1) * LOADS_PER_TILE>();
        else
            wait_vm<0>();
    };
    start_loads();
    await_first();
    for (;;) {  // over the blocks of this workgroup, to the end of the kernel (not indented)
    __syncthreads();
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        lsum[qb] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[qb][db][r] = 0.f;
    }
    bf16x8 kf[DS];  // K fragments of one block
    read_k(0, 0, kf);
    if (kQThroughLds) {
        typedef const bf16x8 __attribute__((address_space(3))) * lds_frag_ptr;
        int ln = lane;
        if (kLoop) asm volatile("" : "+v"(ln));
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int ds = 0; ds < DS; ++ds)
                qf[qb][ds] = *(lds_frag_ptr)(uintptr_t)(smem_base + kQAt + (rg * QW + 32 * qb + (ln & 31)) * C::ROWB + (((2 * ds + (ln >> 5)) ^ C::swz(ln & 31)) << 4));
    }
    if (kQThroughLds) __syncthreads();  // every wavefront has its fragments: the ring takes their place
#pragma unroll
    for (int t = kEarlyTiles; t < STAGES - (kStagger ? 0 : 1); ++t) fill(t);

    // With d = 128 two sets of V fragments do not fit the register file next to the accumulators: then one
    // set is used, refilled in the middle of each step right after the MFMAs that consumed it were issued.
    constexpr bool kTwoVSets = (DP <= 64);
    // Pipeline state: xA/xB hold the logits of the current / next block, pA/pB and vfA/vfB the
    // probabilities and V fragments of the block whose Attend is still owed.
    floatx16 xA[QB], xB[QB];
    uint32_t pA[QB][8], pB[QB][8];
    bf16x8 vfA[2][DB], vfB[2][DB];  // vfB stays unused with one set
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int i = 0; i < 8; ++i) pB[qb][i] = 0u;  // the Attend owed before block 0 adds nothing
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int db = 0; db < DB; ++db) vfA[t][db] = vfB[t][db] = __builtin_bit_cast(bf16x8, (uint4v){0, 0, 0, 0});
    // ---- pieces of a two-phase step
    float xv[QB][16];  // logits of the current block
    // One wavefront per SIMD: kept in the upper half of the register file by name.  Left to itself the compiler carries all accumulators (128 at
    // d = 256) through the lower half in every step, for the rescaling that hardly ever happens.
    auto keep_high = [&]() __attribute__((always_inline)) {
        if (!kHigh) return;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int db = 0; db < DB; ++db) asm volatile("" : "+a"(oacc[qb][db]));
    };
    // V^T fragments of 32 columns (both 16-key halves), and one of the K fragments
    auto read_v_block = [&](int stage, int kb, int db) __attribute__((always_inline)) {
        const int at = stage * C::K_STEP + (C::SPLIT_RING ? 0 : C::V_AT) + kb * 32 * C::ROWB;
        asm volatile("" : "+v"(voff[db][0]), "+v"(voff[db][1]));
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int off = at + t * 16 * C::ROWB;
            vfA[t][db] = concat(lds_read_tr16_at(voff[db][0] + off), lds_read_tr16_at(voff[db][1] + off));
        }
        if (kSyncEveryPhase) __builtin_amdgcn_s_waitcnt(kLgkm0);
    };
    auto read_k_frag = [&](int stage, int kb, int ds) __attribute__((always_inline)) {
        typedef const bf16x8 __attribute__((address_space(3))) * lds_frag_ptr;
        asm volatile("" : "+v"(koff[ds]));
        kf[ds] = *(lds_frag_ptr)(uintptr_t)(uint32_t)(koff[ds] + stage * C::K_STEP + kb * 32 * C::ROWB);
        if (kSyncEveryPhase) __builtin_amdgcn_s_waitcnt(kLgkm0);
    };
    logits(kf, xA);
    // Reference max of each row: its scaled logit with the first key of its first block, which is row 0 of S^T: register 0 of the lower half.
    // (A dot product of its own, taken before, was a chain of d products in the start of every workgroup: 12 heads x 512, d = 64, 5.64 -> 5.42
    // us, 768 causal heads x 512, d = 96, 90.8 -> 85.0, 8 x 512, d = 256, 17.5 -> 16.5.)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) m[qb] = n_tiles > 0 ? lower_half(xA[qb][0]) * c : 0.f;

    // One step = one block b:   matrix pipe: Attend(b-1) and S(b+1);   vector ALU: softmax(b).
    // Stage bookkeeping (tile j = blocks 2j, 2j+1; reads of step b touch K of block b+1 and V of block b):
    //   after step 2j   : wait for tile j+1, barrier  (also: every wave is past step 2j-1, the last reader of tile j-1)
    //   before step 2j+1: start streaming tile j+STAGES-1 into the stage that held tile j-1
    auto step = [&](int blk, int stage, int next_stage, bool masked, floatx16 (&xc)[QB], floatx16 (&xn)[QB], const uint32_t (&pp)[QB][8],
                    const bf16x8 (&vp)[2][DB], uint32_t (&pc)[QB][8], bf16x8 (&vc)[2][DB]) __attribute__((always_inline)) {
        read_k(next_stage, (blk + 1) & (KB - 1), kf);
        if (kTwoVSets) read_v(stage, blk & (KB - 1), vc);
        if (kSyncEveryPhase) __builtin_amdgcn_s_waitcnt(kLgkm0);
        __builtin_amdgcn_sched_barrier(0);  // keep the LDS reads at the top: they have a whole step to land
        float bsum[QB];
        constexpr int kMfmaPerStep = 2 * QB * DB + QB * DS, kValuPerMfma = (QB * 48) / kMfmaPerStep;
        if (kTwoVSets) {
            // one scheduling region: spread the MFMAs evenly through the softmax instructions
            attend(vp, pp);
            logits(kf, xn);
            shift(blk, masked, xc);
            softmax_b(xc, pc, bsum);
#pragma unroll
            for (int g = 0; g < kMfmaPerStep; ++g) {  // vector work first: measured about 1 % faster than MFMA first
                __builtin_amdgcn_sched_group_barrier(0x002, kValuPerMfma, 0);  // one MFMA's share of the vector work
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);             // one MFMA
            }
        } else {
            // two regions; the single V fragment set (vp and vc are the same registers) is refilled between them
            attend(vp, pp);
            shift(blk, masked, xc);
#pragma unroll
            for (int g = 0; g < 2 * QB * DB; ++g) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, (QB * 16) / (2 * QB * DB), 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            read_v(stage, blk & (KB - 1), vc);
            if (kSyncEveryPhase) __builtin_amdgcn_s_waitcnt(kLgkm0);
            __builtin_amdgcn_sched_barrier(0);
            logits(kf, xn);
            softmax_b(xc, pc, bsum);
#pragma unroll
            for (int g = 0; g < QB * DS; ++g) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, (QB * 32) / (QB * DS), 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        bool jump = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) jump |= !(bsum[qb] <= kSumJump);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(jump) != 0, 0)) {  // exact path: xc holds c S - m of this block
            float by[QB], alpha[QB];
            bool far = false;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                by[qb] = __builtin_fmaxf(block_max(xc[qb]), 0.f);
                alpha[qb] = __builtin_amdgcn_exp2f(-by[qb]);
                far |= by[qb] > kFar || __builtin_fabsf(m[qb]) > kFar;
            }
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(far) != 0, 0)) {
                read_k(stage, blk & (KB - 1), kf);  // S once more: the block's K is still in the ring
                logits(kf, xc);
                raise_from_logits(blk, masked, xc, alpha);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) by[qb] = 0.f;
            }
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                m[qb] += by[qb];
#pragma unroll
                for (int r = 0; r < 16; ++r) xc[qb][r] -= by[qb];
            }
            rescale(alpha);
            softmax_b(xc, pc, bsum);
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            lsum[qb] += bsum[qb];
        }
    };
    // Ring bookkeeping around the steps of one tile.  sync_before_last_step: wait for tile j+1 (of the tiles in
    // flight only STAGES-3 may still be outstanding), barrier (every wavefront is then also past its last read of
    // tile j-1), and start streaming tile j+STAGES-1 into the stage that held tile j-1.
    auto sync_and_stream = [&](int j, int sj) __attribute__((always_inline)) {
        // A single wavefront has no barrier to wait at: its reads of the stage that is refilled below must be back first.
        if (NW == 1) __builtin_amdgcn_s_waitcnt(kLgkm0);
        if (kStagger) {  // the step needs V of tile j and K of tile j+1, which were started together; two blocks per tile: both of tile j+1
            if (kSyncEveryPhase || j + STAGES - 1 >= n_tiles)
                wait_vm<0>();
            else
                wait_vm<KB == 1 ? (STAGES - 2) * LOADS_PER_TILE : STAGES < 3 ? 0 : (STAGES - 3) * LOADS_PER_TILE + C::LOADS>();
            __syncthreads();
            if (j + STAGES - 1 < n_tiles) issue_tile_loads(j + STAGES - 1, sj == 0 ? STAGES - 1 : sj - 1, false, true);
            if (j + STAGES < n_tiles) issue_tile_loads(j + STAGES, sj, true, false);
        } else {
            if (kSyncEveryPhase || j + STAGES - 2 >= n_tiles)
                wait_vm<0>();
            else
                wait_vm<(STAGES < 3 ? 0 : STAGES - 3) * LOADS_PER_TILE>();
            __syncthreads();
            if (j + STAGES - 1 < n_tiles) issue_tile_loads(j + STAGES - 1, sj == 0 ? STAGES - 1 : sj - 1);
        }
        if (kSyncEveryPhase) {  // every wavefront runs this the same number of times, so the barrier is safe here
            wait_vm<0>();
            __syncthreads();
        }
    };
    // Launches of few rows, split keys, the 128-row shapes, d = 32 and d = 256 (kTwoPhase), where a SIMD has few wavefronts or one, and nobody to
    // hide the waits of a step behind.  So a step is two phases, each multiplying operands that are in registers already while the operands
    // of the other one are read from LDS:
    //   A: S(b+1) over kf, with the softmax of block b and the reads of V(b) between its MFMAs;
    //   B: Attend(b) over vfA, with the reads of K(b+2) between its MFMAs.
    // The ring moves on between the phases (two blocks per tile: of the tile's first step): V(b) and K(b+1) have left LDS by then.
    // d = 256: at most three vector instructions and four LDS reads between two MFMAs.  A step still takes 2020 cycles for the 1024 of its 32 MFMAs
    // (matrix pipes 51 % busy, LDS 25 %, a third of the wavefronts' cycles spent waiting to issue; the 16 MFMAs of S are one chain on one
    // accumulator): 16 heads of 8192 positions without a mask 1342 -> 982 us (1119 TFLOP/s), 2 x 8 causal heads of 3001 131 -> 89.
    // Before, a step read its operands at its start and moved the accumulators twice between the halves of the register file.
    // Key groups: 12 heads x 512, d = 64, 5.31 -> 5.06 us; 4 causal heads x 8192 58.1 -> 50.4; 8 causal x 1024, d = 128, 11.9 -> 10.8; a step of
    // a workgroup alone on its compute unit 900 -> 790 cycles (256 of matrix pipe).  Split keys: 16 heads x 65536 45.7 -> 44.4.
    auto two_phase_step = [&](int blk, int j, int stage, int kb, bool masked) __attribute__((always_inline)) {  // block kb of tile j
        const int stage1 = (stage + 1) % STAGES, stage_k = KB == 1 ? (stage + 2) % STAGES : stage1;
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        __builtin_amdgcn_sched_barrier(0);
        float bsum[QB], e[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            bsum[qb] = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) xA[qb][r] = 0.f;
        }
#pragma unroll
        for (int g = 0; g < DS; ++g) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                if (kHigh) asm volatile("" : "+a"(qf[qb][g]));
                xA[qb] = mfma_bf16_32x32x16(kf[g], qf[qb][g], xA[qb]);
                if (qb == 0 && g < DB) read_v_block(stage, kb, g);
#pragma unroll
                for (int r = 16 * g / DS; r < 16 * (g + 1) / DS; ++r) {
                    float x = __builtin_fmaf(xv[qb][r], c, -m[qb]);
                    if (masked) x = is_visible(first_key(blk), qb, r) ? x : -INFINITY;  // exp2 -> probability exactly 0
                    if (r & 1) {
                        pA[qb][r >> 1] = pack_bf16(e[qb], __builtin_amdgcn_exp2f(x));
                        bsum[qb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pA[qb][r >> 1]), ones, bsum[qb], false);
                    } else {
                        e[qb] = __builtin_amdgcn_exp2f(x);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        bool jump = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) jump |= !(bsum[qb] <= kSumJump);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(jump) != 0, 0)) {  // exact path, before this block's Attend
            keep_high();
            float alpha[QB];
            raise_from_logits(blk, masked, xv, alpha);
            rescale(alpha);
            softmax_b(xv, pA, bsum);
            keep_high();
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) lsum[qb] += bsum[qb];
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        if (KB == 1)
            sync_and_stream(j + 1, stage1);
        else if (kb == 0)
            sync_and_stream(j, stage);
        keep_high();
#pragma unroll
        for (int g = 0; g < 2 * DB; ++g) {
            const int t = g / DB, db = g % DB;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const uint4v pw = {pA[qb][4 * t], pA[qb][4 * t + 1], pA[qb][4 * t + 2], pA[qb][4 * t + 3]};
                oacc[qb][db] = mfma_bf16_32x32x16(vfA[t][db], __builtin_bit_cast(bf16x8, pw), oacc[qb][db]);
            }
            if (g < DS / 2) read_k_frag(stage_k, kb, 2 * g), read_k_frag(stage_k, kb, 2 * g + 1);
            // the logits move to the vector ALU's half of the registers when the last MFMA of S has had its latency
            if (kHigh && g == DB / 2) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) asm volatile("" : "+a"(xA[qb]));
            }
            if (kHigh && g >= DB / 2 && g < DB / 2 + DB) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int r = 16 * (g - DB / 2) / DB; r < 16 * (g - DB / 2 + 1) / DB; ++r) {
                        xv[qb][r] = xA[qb][r];
                        asm volatile("" : "+v"(xv[qb][r]));
                    }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!kHigh) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int r = 0; r < 16; ++r) xv[qb][r] = xA[qb][r];
        }
    };
    // Where MFMAs are spread through the neighbour's softmax, the last step of a tile already reads K of the next tile, so the
    // synchronisation sits before it.
    auto tile_steps = [&](int j, int sj, bool masked) __attribute__((always_inline)) {  // sj = j % STAGES
        const int sn = sj + 1 == STAGES ? 0 : sj + 1;       // stage of tile j+1
        // first 32-key block of the tile, as a key position / 32 (only the masked form of a step looks at it)
        const int kb0 = KBT * (((SPARSE && masked) || SPLIT) ? tile_of(j) : j) + kg * KB;
        if (kTwoPhase) {
#pragma unroll
            for (int i = 0; i < KB; ++i) two_phase_step(kb0 + i, j, sj, i, masked);
        } else {
#pragma unroll
            for (int i = 0; i < KB; i += 2) {
                if (kTwoVSets)
                    step(kb0 + i, sj, sj, masked, xA, xB, pB, vfB, pA, vfA);
                else
                    step(kb0 + i, sj, sj, masked, xA, xB, pB, vfA, pA, vfA);
                const bool last = i + 2 == KB;
                if (last) sync_and_stream(j, sj);
                if (kTwoVSets)
                    step(kb0 + i + 1, sj, last ? sn : sj, masked, xB, xA, pA, vfA, pB, vfB);
                else
                    step(kb0 + i + 1, sj, last ? sn : sj, masked, xB, xA, pA, vfA, pB, vfA);
            }
        }
    };

    // Per wavefront the tiles fall into three consecutive ranges: fully visible, partly masked
    // (sequence tail or causal diagonal), and not visible at all (the wavefront then only keeps
    // streaming and synchronising for the others).
    // (block-sparse: the list is ascending, so only its last 64 keys can hold the ragged end of the sequence)
    // (split keys: the same ranges, counted from the first tile of the split and cut to its length)
    // A tile is fully visible to a key group when the last key of its share is, and active when the first one is.
    const int first_of_share = kg * KB * 32, end_of_share = first_of_share + KB * 32;
    const int all_see = CAUSAL ? min(q0w + off + 1, N) : N, any_sees = CAUSAL ? min(q0w + QW + off, N) : N;  // keys seen by all / any of the rows
    const int n_unm_all = all_see < end_of_share ? 0 : (all_see - end_of_share) / BC + 1;
    const int n_act_all = any_sees <= first_of_share ? 0 : (any_sees - first_of_share - 1) / BC + 1;
    const int n_unm_tiles = SPARSE ? max(n_tiles - KB64, 0) : max(0, min(n_unm_all - t0, n_tiles));
    const int n_act_tiles = SPARSE ? n_tiles : max(0, min(n_act_all - t0, n_tiles));
    int j = 0;
    if (kTwoPhase) {
        if (KB == 1) sync_and_stream(0, 0);
        read_k(KB == 1 ? 1 : 0, KB - 1, kf);  // of the second block
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int r = 0; r < 16; ++r) xv[qb][r] = xA[qb][r];
        __builtin_amdgcn_sched_barrier(0);
    }
    // main loop: STAGES fully visible tiles per trip, so that every ring stage index is a constant
#pragma unroll 1
    for (; j + STAGES <= n_unm_tiles; j += STAGES) {
#pragma unroll
        for (int sj = 0; sj < STAGES; ++sj) tile_steps(j + sj, sj, false);
    }
    // remaining visible tiles and the partly masked ones (masking a fully visible tile changes nothing)
    int sj = 0;  // j is a multiple of STAGES here
#pragma unroll 1
    for (; j < n_unm_tiles; ++j) {
        tile_steps(j, sj, false);
        sj = sj + 1 == STAGES ? 0 : sj + 1;
    }
#pragma unroll 1
    for (; j < n_act_tiles; ++j) {
        tile_steps(j, sj, true);
        sj = sj + 1 == STAGES ? 0 : sj + 1;
    }
    if (!kTwoPhase) attend(kTwoVSets ? vfB : vfA, pB);  // still owed for the last block; a two-phase step runs its own
#pragma unroll 1
    for (; j < n_tiles; ++j) {
        constexpr bool kAhead = kTwoPhase && KB == 1;  // a tile's step has gone past the synchronisation of the next one
        if (kAhead) sj = sj + 1 == STAGES ? 0 : sj + 1;
        sync_and_stream(j + (kAhead ? 1 : 0), sj);
        if (!kAhead) sj = sj + 1 == STAGES ? 0 : sj + 1;
    }

    // ---- key groups: the partial results (reference maximum, row sum, accumulators) of a row's wavefronts meet in the ring's
    // LDS, in the lane layout they have; each wavefront then merges and writes its share of the output columns.
    if (KG > 1) {
        constexpr int QUADS = D / 8, OQ = QUADS / KG;  // accumulator quads of a lane per row block, and of those per wavefront
        floatx4* const part = (floatx4*)smem + lane;
        float* const stat = (float*)(smem + NW * QB * QUADS * 1024) + lane;
        auto slot = [&](int k, int qb) __attribute__((always_inline)) { return (rg * KG + k) * QB + qb; };
        __syncthreads();  // every wavefront is past its last read of the ring
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float total = halves_sum(lsum[qb]);
            // a group none of whose keys the row sees weighs nothing, whatever its first key's logit was
            stat[slot(kg, qb) * 64] = half ? total : total > 0.f ? m[qb] : -INFINITY;
#pragma unroll
            for (int q = 0; q < QUADS; ++q) {
                const int db = q / 4, rq = q % 4;
                part[(slot(kg, qb) * QUADS + q) * 64] =
                    floatx4{oacc[qb][db][4 * rq], oacc[qb][db][4 * rq + 1], oacc[qb][db][4 * rq + 2], oacc[qb][db][4 * rq + 3]};
            }
        }
        __syncthreads();
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float mk[KG], w[KG], M = -FLT_MAX, L = 0.f;
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                mk[k] = stat[slot(k, qb) * 64 - 32 * half];
                M = __builtin_fmaxf(M, mk[k]);
            }
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                w[k] = __builtin_amdgcn_exp2f(mk[k] - M);
                L += w[k] * stat[slot(k, qb) * 64 + 32 * (1 - half)];
            }
            const int r_wg = rg * QW + 32 * qb + l32, row = qt * BR + r_wg;
            const float inv = SPLIT ? 1.f : 1.0f / L;
            float* ws = nullptr;
            if (SPLIT) {
                ws = prob.split_ws + ((size_t)(bh * grid.n_row_blocks + qt) * prob.n_splits + split) * (size_t)(BR * (DP + 2));
                if (row < Nq && kg == 0 && half == 0) {
                    ws[BR * DP + r_wg] = M;
                    ws[BR * DP + BR + r_wg] = L;
                }
            }
#pragma unroll
            for (int i = 0; i < OQ; ++i) {
                const int q = kg * OQ + i, dcol = 8 * q + 4 * half;
                float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < KG; ++k) {
                    const floatx4 o = part[(slot(k, qb) * QUADS + q) * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[e] = __builtin_fmaf(w[k], o[e], a[e]);
                }
                if (row >= Nq) continue;
                if (SPLIT) {
                    *(floatx4*)(ws + (size_t)r_wg * DP + dcol) = floatx4{a[0], a[1], a[2], a[3]};
                } else {
                    floatx2 w2;
                    w2[0] = __builtin_bit_cast(float, pack_bf16(a[0] * inv, a[1] * inv));
                    w2[1] = __builtin_bit_cast(float, pack_bf16(a[2] * inv, a[3] * inv));
                    *(floatx2*)(Oh + (size_t)row * D + dcol) = w2;
                }
            }
        }
        return;
    }

    // ---- split keys: leave the unnormalised partial result in the workspace.  Per (head, row block, split):
    // BR rows x DP accumulators, then BR reference maxima, then BR row sums, all fp32.
    if (SPLIT) {
        float* part = prob.split_ws + ((size_t)(bh * grid.n_row_blocks + qt) * prob.n_splits + split) * (size_t)(BR * (DP + 2));
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float total = halves_sum(lsum[qb]);
            const int r_wg = wave * QW + 32 * qb + l32;  // row within the row block
            if (qt * BR + r_wg >= Nq) continue;          // rows past the end are never merged
            if (half == 0) {
                part[BR * DP + r_wg] = m[qb];
                part[BR * DP + BR + r_wg] = total;
            }
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int rq = 0; rq < 4; ++rq) {
                    floatx4 w4 = {oacc[qb][db][4 * rq], oacc[qb][db][4 * rq + 1], oacc[qb][db][4 * rq + 2], oacc[qb][db][4 * rq + 3]};
                    *(floatx4*)(part + (size_t)r_wg * DP + 32 * db + 8 * rq + 4 * half) = w4;
                }
        }
        return;
    }
    // ---- epilogue: O = O_acc / l, rounded to bf16.  A lane holds 4 consecutive columns per register quad, its other half the next
    // 4; two quads are swapped across the halves so that every lane stores 8 consecutive columns.  Short sequences are bound by
    // memory and by their start and end: half as many stores of twice the width, 768 heads x 512, d = 64: 66 -> 62 us; 1024 x 128
    // 16.3 -> 15.0; d = 128, 768 x 512: 158 -> 147.
    // Where the workgroup has another block, its first loads go out before the results of this one are put together, and are awaited
    // before they are stored.
    bf16* const O_done = Oh;
    const int row_done = q0w + l32;
    bool more = false;
    if (kLoop) {
        block_of_xcd += grid.stride;
        const int logical = (blockIdx.x & 7) * blocks_per_xcd + block_of_xcd;
        more = block_of_xcd < blocks_per_xcd && logical < n_blocks;
        if (more) {
            bh = grid.by_qtiles.quotient(logical);
            qt = logical - bh * n_qtiles;
            place();
            n_tiles = (N + BC - 1) / BC;
            __syncthreads();  // every wavefront is past its last read of the ring
            start_loads();
        }
    }
    uint4v out[QB][DB][2];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float total = halves_sum(lsum[qb]);
        const float inv = (SPARSE && n_tiles == 0) ? 0.f : 1.0f / total;  // a row block with an empty list yields zeros
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int rp = 0; rp < 2; ++rp) {
                uint32_t w[2][2];
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int r = 8 * rp + 4 * q + 2 * e;
                        w[q][e] = pack_bf16(oacc[qb][db][r] * inv, oacc[qb][db][r + 1] * inv);
                    }
                const auto lo = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
                const auto hi = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
                out[qb][db][rp] = uint4v{(uint32_t)lo[0], (uint32_t)hi[0], (uint32_t)lo[1], (uint32_t)hi[1]};
                if (!kLoop && row_done + 32 * qb < Nq)
                    *(uint4v*)(O_done + (size_t)(row_done + 32 * qb) * D + 32 * db + 16 * rp + 8 * half) = out[qb][db][rp];
            }
    }
    if (!kLoop) return;
    if (more) await_first();
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int row = row_done + 32 * qb;
        if (row < Nq) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int rp = 0; rp < 2; ++rp) *(uint4v*)(O_done + (size_t)row * D + 32 * db + 16 * rp + 8 * half) = out[qb][db][rp];
        }
    }
    if (!more) return;
    }
}

template <int D, int QB, int NW, int STAGES, bool CAUSAL, int MODE = kDense, int BCX = 0, int KG = 1>
inline hipError_t launch_cfg(const void* Q, const void* K, const void* V, void* O, int BH, const Bf16Problem& prob, float scale,
                             hipStream_t stream) {
    constexpr int BR = 32 * QB * (NW / KG);
    // split keys: the kernel sees (row block, split) pairs where the other modes see row blocks
    const int n_row_blocks = (prob.Nq + BR - 1) / BR, n_splits = MODE == kSplit ? prob.n_splits : 1;
    const int n_qtiles = n_row_blocks * n_splits, n_blocks = BH * n_qtiles;
    auto kern = fwd_bf16_kernel<D, QB, NW, STAGES, CAUSAL, MODE, BCX, KG>;
    constexpr int lds = bf16_lds_bytes(D, QB, NW, STAGES, BCX, KG) + (MODE == kSparse ? kMaxSparseTiles * (int)sizeof(int) : 0);
    static_assert(lds <= 160 * 1024, "more LDS than a compute unit has");
    static std::atomic<uint64_t> attr_done{0};  // one flag per kernel instantiation
    hipError_t e = allow_dynamic_lds((const void*)kern, lds, &attr_done);
    if (e != hipSuccess) return e;
    const bool deal_heads = MODE == kDense && !CAUSAL && prob.kv_lens && BH < 16LL * prob.heads_per_batch && (BH % 8 == 0 || BH >= 128);
    const int blocks_per_xcd = deal_heads ? (BH + 7) / 8 * n_qtiles : (n_blocks + 7) / 8;
    int stride = blocks_per_xcd;
    if (loops_over_blocks(D, CAUSAL, MODE, KG) && !prob.kv_lens) {
        static std::atomic<int> per_cu{0};
        int n = per_cu.load(std::memory_order_relaxed);
        if (n == 0) {
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, 64 * NW, lds);
            if (e != hipSuccess) return e;
            if (n < 1) n = 1;
            per_cu.store(n, std::memory_order_relaxed);
        }
        // A workgroup takes two blocks where the launch has four rounds of them or more.  Blocks that belong to a workgroup do not move to a unit
        // that is free: beside another stream's launch that holds 32 of the 256 units, 512 heads x 512, d = 128 (four rounds; alone 97 us with a
        // workgroup for every block) takes 116 us with one block per workgroup, 128 with two and 156 with four, and alone 97, 92 and 89;
        // 1024 x 256 89, 91, 108 and alone 71, 63, 62; 2048 x 512 (16 rounds) 414 with one, 416 with two, 591 with 16, and alone 362, 350,
        // 343; 16 x 8192 (two rounds) 666 with one, 838 with two, and alone no difference.
        if (blocks_per_xcd >= 4 * 32 * n) stride = (blocks_per_xcd + 1) / 2;
    }
    const LaunchGrid grid{n_qtiles, n_blocks, blocks_per_xcd, stride, BH, n_row_blocks, deal_heads ? 0 : blocks_per_xcd, deal_heads ? 8 : 1, deal_heads, Divisor(n_qtiles), Divisor(BH), Divisor(n_splits),
                          Divisor(prob.heads_per_batch)};
    hipLaunchKernelGGL(kern, dim3(stride * 8), dim3(64 * NW), lds, stream, (const bf16*)Q, (const bf16*)K,
                       (const bf16*)V, (bf16*)O, prob, grid, scale * kLog2e);
    return hipGetLastError();
}

// The two mask variants of one tile shape behind one call; defined here, instantiated explicitly by the
// translation units that own the shapes (declared in flat_launch.hpp).
template <int D, int QB, int NW, int STAGES, int BCX>
hipError_t launch_fwd_bf16_shape(const void* Q, const void* K, const void* V, void* O, int BH, const Bf16Problem& prob, float scale,
                                 int causal, hipStream_t stream) {
    return causal ? launch_cfg<D, QB, NW, STAGES, true, kDense, BCX>(Q, K, V, O, BH, prob, scale, stream)
                  : launch_cfg<D, QB, NW, STAGES, false, kDense, BCX>(Q, K, V, O, BH, prob, scale, stream);
}

// Key-group form: KG groups of wavefronts share the keys of 32 QB NW / KG query rows.
template <int D, int QB, int NW, int STAGES, int BC, int KG>
hipError_t launch_fwd_bf16_groups(const void* Q, const void* K, const void* V, void* O, int BH, const Bf16Problem& prob, float scale,
                                  int causal, hipStream_t stream) {
    return causal ? launch_cfg<D, QB, NW, STAGES, true, kDense, BC, KG>(Q, K, V, O, BH, prob, scale, stream)
                  : launch_cfg<D, QB, NW, STAGES, false, kDense, BC, KG>(Q, K, V, O, BH, prob, scale, stream);
}

// Workgroups of this shape that fit one compute unit at a time (registers and LDS), as the runtime reports it.
template <int D, int QB, int NW, int STAGES, int BCX, int KG>
hipError_t fwd_bf16_shape_occupancy(int* workgroups_per_cu) {
    auto kern = fwd_bf16_kernel<D, QB, NW, STAGES, false, kDense, BCX, KG>;
    constexpr int lds = bf16_lds_bytes(D, QB, NW, STAGES, BCX, KG);  // as launched: the limit set here holds for launches too
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(workgroups_per_cu, kern, 64 * NW, lds);
}

// Block-sparse launch of one tile shape (its row block is the shape's rows per workgroup).
template <int D, int QB, int NW, int STAGES>
hipError_t launch_fwd_bf16_sparse_shape(const void* Q, const void* K, const void* V, void* O, int BH, const Bf16Problem& prob,
                                        float scale, hipStream_t stream) {
    return launch_cfg<D, QB, NW, STAGES, false, kSparse>(Q, K, V, O, BH, prob, scale, stream);
}

#define FLAT_INSTANTIATE_BF16_SHAPE_BC(D, QB, NW, STAGES, BCX)                                                               \
    template hipError_t launch_fwd_bf16_shape<D, QB, NW, STAGES, BCX>(const void*, const void*, const void*, void*, int,    \
                                                                      const Bf16Problem&, float, int, hipStream_t);        \
    template hipError_t fwd_bf16_shape_occupancy<D, QB, NW, STAGES, BCX>(int*);
#define FLAT_INSTANTIATE_BF16_GROUPS(D, QB, NW, STAGES, BC, KG)                                                              \
    template hipError_t launch_fwd_bf16_groups<D, QB, NW, STAGES, BC, KG>(const void*, const void*, const void*, void*, int, \
                                                                          const Bf16Problem&, float, int, hipStream_t);       \
    template hipError_t fwd_bf16_shape_occupancy<D, QB, NW, STAGES, BC, KG>(int*);
#define FLAT_INSTANTIATE_BF16_SHAPE(D, QB, NW, STAGES) FLAT_INSTANTIATE_BF16_SHAPE_BC(D, QB, NW, STAGES, 0)

}  // namespace flat
