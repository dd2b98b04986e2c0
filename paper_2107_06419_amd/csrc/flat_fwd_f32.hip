// fp32 entry point: the two kernels behind it and which of them takes a problem.
#include "flat_fwd_f32_rows.hpp"
#include "flat_launch.hpp"

namespace flat {

template <int D, int NW, bool CAUSAL>
__global__ __launch_bounds__(64 * NW, D == 64 ? 2 : 1) void fwd_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                                                                          const float* __restrict__ V, float* __restrict__ O, int N,
                                                                          int n_qtiles, int n_blocks, int blocks_per_xcd, int n_heads,
                                                                          const Divisor by_qtiles, const Divisor by_heads, float c) {
    extern __shared__ __attribute__((aligned(16))) char smem[];

    // Without a mask an XCD takes a contiguous range of (head, row block) pairs, so that a head's K and V stay in one L2; with the
    // causal mask the blocks are ranked heaviest first over all heads and dealt to the XCDs in turn.
    // (all arguments in one round trip, as in the bf16 kernel)
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

    f32_rows<D, NW, CAUSAL>(smem, Q, K, V, O, N, bh, qt, c, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63);
}

template <int D, int NW, bool CAUSAL>
static hipError_t launch_shape(const float* Q, const float* K, const float* V, float* O, int BH, int N, float scale, hipStream_t stream) {
    const int n_qtiles = (N + 31) / 32;
    if ((long long)BH * n_qtiles > 0x7ffffff0LL) return hipErrorInvalidValue;
    const int n_blocks = BH * n_qtiles;
    const int blocks_per_xcd = (n_blocks + 7) / 8;
    constexpr int lds = NW * F32Cfg<D>::LDS_RESERVED;
    auto kern = fwd_f32_kernel<D, NW, CAUSAL>;
    static std::atomic<uint64_t> attr_done{0};
    hipError_t e = allow_dynamic_lds((const void*)kern, lds, &attr_done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(blocks_per_xcd * 8), dim3(64 * NW), lds, stream, Q, K, V, O, N, n_qtiles, n_blocks, blocks_per_xcd, BH,
                       Divisor(n_qtiles), Divisor(BH), scale * kLog2e);
    return hipGetLastError();
}

// Wavefronts per workgroup (1, 2 or 4) by the time each would take, in units of one 32-key tile of a wavefront on a chip whose
// slots are full: a workgroup takes ceil(tiles / NW) units plus its start and merge (1.5 units at d = 128, 0.7 at d = 64 where a
// second wavefront on the SIMD hides half of it), and
//   without a mask all workgroups are equal and run in whole rounds;
//   with the causal mask they run heaviest first, so the time is their mean times their number, or the heaviest one alone.
// With fewer wavefronts than SIMDs a d = 64 wavefront has its SIMD to itself and takes half a unit per tile.
// Measured with 1 / 2 / 4 wavefronts (us; the rule's choice in brackets): d = 128, heads x positions: 16 x 8192 4322 / 4321 /
// 4346 [1]; 16 x 2049 causal 274 / 164 / 175 [2], without a mask 551 / 425 / 375 [4]; 128 x 512 causal 85 / 97 / 128 [1]; 128 x
// 128 22 / 17 / 20 [2]; 1024 x 33 33 / 36 / 63 [1].  d = 64: 12 x 512 37 / 20 / 13 [4]; 128 x 512 88 / 87 / 77 [4]; 1024 x 128
// 45 / 48 / 56 [1]; 1024 x 200 causal 85 / 92 / 110 [1].
template <int D>
static double predicted_units(int nw, int BH, int N, bool causal) {
    constexpr double kUnitsPerGroup = D == 128 ? 1.5 : 0.7, kSlots = 256.0 * F32Cfg<D>::WAVES_PER_CU;
    const double tiles = (N + 31) / 32, load = BH * tiles * nw / kSlots, longest = ceil(tiles / nw) + kUnitsPerGroup;
    double time = causal ? fmax(load * ((tiles / nw + 1.0) * 0.5 + kUnitsPerGroup), longest) : ceil(load) * longest;
    if (D == 64) time *= fmin(1.0, fmax(0.5, load));
    return time;
}

template <int D>
static int wavefronts_per_workgroup(int BH, int N, bool causal) {
    int best = 1;
    for (int nw = 2; nw <= 4; nw *= 2)
        if (predicted_units<D>(nw, BH, N, causal) < predicted_units<D>(best, BH, N, causal)) best = nw;
    return best;
}

// Key groups of the kernel of flat_fwd_f32_pieces.hip (1 or 2), or 0 where fwd_f32_kernel is predicted to take no more than 1.05 of its time, by the same
// arithmetic in us: a workgroup takes its steps and 6.5 us for its start and end; a step 1.65 us with one key group and 2.03 with two at d = 128, 1.64 and
// 1.9 at d = 64, where two workgroups share a compute unit and one alone takes half of that.  So at d = 64 a round that is partly filled counts
// half at least, and with the causal mask the heaviest workgroup is alone for half of its time; at d = 128 what is left of a second round follows a first
// one, if only of the lightest blocks.  A unit of the other kernel is 4.2 us.  Fewer than 128 positions: see there.  4096 is where the
// comparison of the two over random problems ends, in time and in error; no limit of the split products is known beyond it (32 x 4097, d = 64, 506 us and 5.1e-7 against 1134
// and 6.7e-7; 16 x 8192, d = 128, 1679 and 6.6e-7 against 4302 and 1.8e-6).
// Measured, one group / two / the other kernel (the rule's choice in brackets): d = 128, 16 x 2049 causal 104 / 93 / 162 [2], 128 x 512 causal 53 / 71 / 85 [1],
// 4 x 3000 141 / 95 / 202 [2], 256 x 300 71 / 88 / 131 [1]; d = 64, 12 x 512 18.3 / 13.6 / 12.6 [0], 1 x 2000 55 / 38 / 39 [0], 16 x 1000 causal 32 / 23 / 29
// [2], 1024 x 128 28 / 35 / 44 [1].  Over 500 random problems of 128 to 4096 positions 1.7 % behind the best of all on average, 69 % at worst (216 x 131, d = 64: 24.7 [0], one
// 14.0; 15 x 602, 25.3 [0], two 16.0).  Of the 355 that take the split products 12 are slower than with the other kernel, by up to 6 % (161 to 192 positions of few heads, d =
// 128: 16 x 163 14.7 against 14.4); the rest take 0.4 to 1.0 of its time, 0.7 on average.
template <int D>
static int key_groups_of_pieces(int BH, int N, bool causal) {
    if (N < 128 || N > 4096) return 0;
    constexpr double kStart = 6.5, kStep[2] = {D == 128 ? 1.65 : 1.64, D == 128 ? 2.03 : 1.9}, kSlots = D == 128 ? 256.0 : 512.0;
    int best = 0;
    double best_time = 0.95 * 4.2 * predicted_units<D>(wavefronts_per_workgroup<D>(BH, N, causal), BH, N, causal);
    for (int kg = 1; kg <= 2; ++kg) {
        const double load = BH * (double)((N + 128 / kg - 1) / (128 / kg)) / kSlots, steps = (N + 32 * kg - 1) / (32 * kg), u = kStep[kg - 1];
        const double longest = steps * u + kStart, mean = load * ((steps + 1.0) * 0.5 * u + kStart), part = load - floor(load);
        double time;
        if (D == 128)
            time = causal ? fmax(fmax(mean, longest), ceil(load) * (u + kStart)) : ceil(load) * longest;
        else
            time = causal ? fmax(mean, longest * fmax(0.5, fmin(0.75, 0.75 * load))) : (floor(load) + (part > 0.0 ? fmax(0.5, part) : 0.0)) * longest;
        if (time < best_time) {
            best = kg;
            best_time = time;
        }
    }
    return best;
}

// A form of the fp32 entry point by number: 1, 2 and 4 are fwd_f32_kernel with that many wavefronts per workgroup, -1 and -2 the split products with that
// many key groups.
template <int D>
static int form_of(int BH, int N, bool causal) {
    const int key_groups = key_groups_of_pieces<D>(BH, N, causal);
    return key_groups ? -key_groups : wavefronts_per_workgroup<D>(BH, N, causal);
}

template <int D, bool CAUSAL>
static hipError_t launch_form(int form, const float* Q, const float* K, const float* V, float* O, int BH, int N, float scale, hipStream_t stream) {
    switch (form) {
        case -2: return launch_fwd_f32_pieces<D, 2, CAUSAL>(Q, K, V, O, BH, N, scale, stream);
        case -1: return launch_fwd_f32_pieces<D, 1, CAUSAL>(Q, K, V, O, BH, N, scale, stream);
        case 1: return launch_shape<D, 1, CAUSAL>(Q, K, V, O, BH, N, scale, stream);
        case 2: return launch_shape<D, 2, CAUSAL>(Q, K, V, O, BH, N, scale, stream);
        case 4: return launch_shape<D, 4, CAUSAL>(Q, K, V, O, BH, N, scale, stream);
        default: return hipErrorInvalidValue;
    }
}

int f32_form(int BH, int N, int d, int causal) { return d == 64 ? form_of<64>(BH, N, causal) : form_of<128>(BH, N, causal); }

hipError_t launch_fwd_f32_form(const float* Q, const float* K, const float* V, float* O, int BH, int N, int d, float scale, int causal, int form,
                               hipStream_t stream) {
    if (d == 64)
        return causal ? launch_form<64, true>(form, Q, K, V, O, BH, N, scale, stream) : launch_form<64, false>(form, Q, K, V, O, BH, N, scale, stream);
    return causal ? launch_form<128, true>(form, Q, K, V, O, BH, N, scale, stream) : launch_form<128, false>(form, Q, K, V, O, BH, N, scale, stream);
}

hipError_t launch_fwd_f32(const float* Q, const float* K, const float* V, float* O, int BH, int N, int d, float scale, int causal, hipStream_t stream) {
    return launch_fwd_f32_form(Q, K, V, O, BH, N, d, scale, causal, f32_form(BH, N, d, causal), stream);
}

}  // namespace flat

// For tests, which have to reach every form at its edges: the form a problem takes, and a call with a given one (d 64 or 128, device pointers as
// flat_attn_fwd_f32 takes them; nothing is checked).  Not part of the interface.
extern "C" int flat_internal_f32_form(int BH, int N, int d, int causal) { return flat::f32_form(BH, N, d, causal); }
extern "C" int flat_internal_fwd_f32_form(const float* Q, const float* K, const float* V, float* O, int BH, int N, int d, float scale, int causal, int form,
                                          void* stream) {
    return (int)flat::launch_fwd_f32_form(Q, K, V, O, BH, N, d, scale, causal, form, static_cast<hipStream_t>(stream));
}
