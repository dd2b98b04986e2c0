// Table of the tile shapes the fused bf16 kernel is built for, and the dispatch by index.  Index 0 of each head
// dimension is the shape flat_attn_fwd uses; the others exist so that the choice can be re-measured (the
// paper's map-space exploration, section 6.1, done by timing instead of a cost model; the trade-off being
// explored is the row granularity of section 5.3: fewer rows per workgroup re-fetch K and V more often and
// fill the matrix units less, more rows need more on-chip state).
#include "flat_launch.hpp"

namespace flat {

namespace {

using LaunchFn = hipError_t (*)(const void*, const void*, const void*, void*, int, const Bf16Problem&, float, int, hipStream_t);
using OccupancyFn = hipError_t (*)(int*);

struct Entry {
    TileShape shape;
    LaunchFn launch;
    OccupancyFn occupancy;
};

template <int D, int QB, int NW, int STAGES, int BCX = 0>
constexpr Entry entry() {
    constexpr int DP = D == 96 ? 128 : D, BC = BCX ? BCX : (D == 256 ? 32 : 64);  // as in Bf16Cfg: padded row length, keys per tile
    return Entry{TileShape{D, 32 * QB * NW, BC, NW, 32 * QB, STAGES, STAGES * 2 * BC * DP * 2},
                 &launch_fwd_bf16_shape<D, QB, NW, STAGES, BCX>, &fwd_bf16_shape_occupancy<D, QB, NW, STAGES, BCX>};
}

const Entry kD64[] = {entry<64, 2, 4, 4>(), entry<64, 2, 4, 3>(), entry<64, 2, 4, 6>(), entry<64, 2, 8, 4>(),
                      entry<64, 1, 8, 4>(), entry<64, 1, 4, 4>(), entry<64, 2, 2, 4>(), entry<64, 1, 4, 3>(),
                      // the key-tile axis: 128 keys per tile (512-row and 256-row workgroups), 32 keys per tile
                      entry<64, 2, 8, 3, 128>(), entry<64, 2, 8, 4, 128>(), entry<64, 2, 4, 3, 128>(), entry<64, 2, 4, 6, 32>()};
const Entry kD128[] = {entry<128, 1, 8, 3>(), entry<128, 1, 8, 4>(), entry<128, 1, 4, 3>(), entry<128, 2, 4, 3>()};
const Entry kD32[] = {entry<32, 2, 4, 4>(), entry<32, 1, 4, 4>()};
const Entry kD96[] = {entry<96, 1, 8, 3>(), entry<96, 1, 4, 3>()};
const Entry kD256[] = {entry<256, 1, 4, 4>()};

const Entry* table(int d) {
    switch (d) {
        case 32: return kD32;
        case 64: return kD64;
        case 96: return kD96;
        case 128: return kD128;
        case 256: return kD256;
        default: return nullptr;
    }
}

const Entry* find(int d, int index) {
    if (index < 0 || index >= tile_shape_count(d)) return nullptr;
    return &table(d)[index];
}

}  // namespace

int tile_shape_count(int d) {
    if (d == 64) return (int)(sizeof(kD64) / sizeof(kD64[0]));
    if (d == 128) return (int)(sizeof(kD128) / sizeof(kD128[0]));
    if (d == 32) return (int)(sizeof(kD32) / sizeof(kD32[0]));
    if (d == 96) return (int)(sizeof(kD96) / sizeof(kD96[0]));
    if (d == 256) return (int)(sizeof(kD256) / sizeof(kD256[0]));
    return 0;
}

bool tile_shape(int d, int index, TileShape* out) {
    const Entry* e = find(d, index);
    if (!e) return false;
    *out = e->shape;
    return true;
}

hipError_t tile_shape_occupancy(int d, int index, int* workgroups_per_cu) {
    const Entry* e = find(d, index);
    return e ? e->occupancy(workgroups_per_cu) : hipErrorInvalidValue;
}

// The 128-row shape of a head size, for launches of few query rows (0: there is none).
int small_launch_shape(int d) { return d == 64 ? 7 : d == 128 ? 2 : d == 32 || d == 96 ? 1 : 0; }

// The shape flat_attn_fwd / flat_attn_fwd_cross run: index 0, except where a measured sweep (python -m
// paper_2107_06419_amd.tile_sweep --small: 1 to 512 heads of 128 to 8192 positions, both masks, several machines)
// shows the 128-row shape of the head dimension ahead:
//   * launches too small to give every compute unit a 256-row workgroup - at most 128 blocks of 256 query rows (causal:
//     256 at d = 32 / 64, 192 at d = 96 / 128): 1.3-1.5 times faster, simply because twice as many compute units work;
//   * d = 64 with the causal mask, up to 4096 positions and 1024 row blocks: ahead by up to 15 %, never behind;
//   * d = 32 (the vector side is the longer pole there and three workgroups per compute unit hide more of it): with
//     the causal mask up to 8192 positions (4-18 %), without it up to 4096 positions and 1024 row blocks (6 %).
// Beyond these ranges the 128-row shapes lose 1-15 %.  No other shape is ahead of index 0 by more than the
// run-to-run spread (the 512-row shape leads by 3 % for d = 64, causal, when B*H*ceil(N/512) is exactly 512, and
// trails by 2-15 % with more or fewer row blocks: no rule is built on that).
//   * up to 128 query rows, where half of a 256-row workgroup or more would be padding (256 heads of 16 rows over 1024
//     keys, d = 64: 23 us on 256 rows, 16 on 128; 2048 heads of 100 rows: 162 and 119 us).
int default_tile_shape(int BH, int Nq, int d, int causal) {
    const long long blocks = (long long)BH * (((long long)Nq + 255) / 256);  // 256-row blocks in the launch
    if (Nq <= 128 && d != 256) return small_launch_shape(d);  // a 256-row workgroup would be at least half padding
    switch (d) {
        case 32:
            if (causal) return Nq <= 8192 ? 1 : 0;
            return (Nq > 512 && ((Nq <= 4096 && blocks <= 1024) || blocks <= 128)) ? 1 : 0;
        case 64:
            if (causal) return (Nq > 256 && blocks <= (Nq <= 4096 ? 1024 : 256)) ? 7 : 0;
            return (Nq > 256 && blocks <= 128) ? 7 : 0;
        case 96: return blocks <= (causal ? 192 : 128) ? 1 : 0;
        case 128: return blocks <= (causal ? 192 : 128) ? 2 : 0;
        default: return 0;
    }
}

// ---- Key-group forms.  A launch of few query rows leaves most of the chip idle on the shapes above, whatever their rows per
// workgroup, because each workgroup walks all keys alone.  In these forms the wavefronts of a workgroup share the keys of
// the same 32, 64 or 128 rows (kernel parameter KG) and merge through LDS at the end; nothing else changes.  They re-read K
// and V from L2 more often per flop, so large launches keep the shapes above.  Each holds a step of K and V per wavefront in
// a ring of two stages (K runs one tile ahead of V); deeper rings measured 3-25 % slower, as fewer workgroups fit.
// Measured, us, best of the shapes above -> form: 12 heads x 512, d = 64, 9.8 -> 6.5; 4 x 4096, d = 64, 47.6 -> 26.4; 2 causal
// x 8192, d = 64, 86.7 -> 39.2; 8 x 1024, d = 128, 22.2 -> 13.3; 4 x 4096, d = 256, 175 -> 109; 64 x 16 rows over 4096 keys,
// d = 64, 46 -> 24.
//
// The choice is by predicted time.  A form (and each shape above) has a measured cost: us to launch, start and drain (`start`),
// us per tile and per workgroup when a workgroup runs alone (`step`, `fixed`), us per tile when the compute unit holds as
// many workgroups as fit (`busy`), and the share of its longest workgroup that a causal launch ends late (`skew`).  Fitted
// to 1750 timings: 1 to 2048 heads, 16 to 300 query rows over 300 to 4096 keys and 64 to 16384 positions, both masks, five
// head sizes.  The choice is within 1-3 % of the fastest on average, where the shapes above alone are 12-28 % behind it, and
// on none of the timings more than 10 % behind the shape it replaces.
namespace {

struct Cost {
    float start, step, fixed, busy, skew;
};
struct Form {
    int rows, keys_per_tile, per_cu;  // query rows per workgroup, keys per tile, workgroups that fit a compute unit
    Cost cost;
    LaunchFn launch;
};
template <int D, int QB, int NW, int STAGES, int BC, int KG>
constexpr Form form(int per_cu, Cost cost) {
    return Form{32 * QB * (NW / KG), BC, per_cu, cost, &launch_fwd_bf16_groups<D, QB, NW, STAGES, BC, KG>};
}

// Per head size: the shapes launch_fwd_bf16 runs (index 0, small_launch_shape), then the key-group forms.
struct Choice {
    int d, n_forms;
    Form base[2];
    Form forms[4];
};
const Choice kChoices[] = {
    {32, 3, {{256, 64, 2, {2.51f, 0.854f, 1.55f, 0.685f, 0.38f}, nullptr}, {128, 64, 3, {2.95f, 0.530f, 0.80f, 0.362f, 0.18f}, nullptr}},
     {form<32, 1, 4, 4, 128, 4>(2, {1.67f, 0.379f, 2.00f, 0.233f, 0.30f}), form<32, 1, 8, 4, 128, 4>(1, {2.95f, 0.378f, 1.48f, 0.378f, 0.29f}),
      form<32, 1, 4, 4, 64, 2>(3, {2.74f, 0.327f, 1.19f, 0.194f, 0.08f})}},
    {64, 3, {{256, 64, 2, {3.88f, 1.031f, 1.67f, 0.995f, 0.35f}, nullptr}, {128, 64, 3, {3.03f, 0.666f, 1.59f, 0.532f, 0.22f}, nullptr}},
     {form<64, 1, 4, 2, 128, 4>(2, {2.05f, 0.520f, 2.43f, 0.367f, 0.21f}), form<64, 1, 8, 2, 128, 4>(1, {1.30f, 0.611f, 4.37f, 0.611f, 0.21f}),
      form<64, 1, 4, 2, 64, 2>(3, {1.61f, 0.421f, 3.01f, 0.294f, 0.17f})}},
    {96, 4, {{256, 64, 1, {0.27f, 1.325f, 5.38f, 1.325f, 0.30f}, nullptr}, {128, 64, 1, {0.57f, 0.857f, 4.69f, 0.857f, 0.19f}, nullptr}},
     {form<96, 1, 4, 2, 128, 4>(1, {1.19f, 0.756f, 3.51f, 0.756f, 0.17f}), form<96, 1, 8, 2, 128, 4>(1, {0.70f, 0.899f, 5.60f, 0.899f, 0.18f}),
      form<96, 1, 4, 2, 64, 2>(2, {1.37f, 0.548f, 3.60f, 0.420f, 0.17f}), form<96, 1, 8, 2, 64, 2>(1, {0.34f, 0.693f, 6.15f, 0.693f, 0.22f})}},
    {128, 4, {{256, 64, 1, {0.33f, 1.609f, 7.00f, 1.609f, 0.29f}, nullptr}, {128, 64, 1, {0.42f, 1.003f, 6.14f, 1.003f, 0.20f}, nullptr}},
     {form<128, 1, 4, 2, 128, 4>(1, {1.17f, 0.861f, 4.64f, 0.861f, 0.17f}), form<128, 1, 8, 2, 128, 4>(1, {0.67f, 1.038f, 7.67f, 1.038f, 0.19f}),
      form<128, 1, 4, 2, 64, 2>(2, {1.82f, 0.588f, 4.40f, 0.489f, 0.23f}), form<128, 1, 8, 2, 64, 2>(1, {0.40f, 0.831f, 8.27f, 0.831f, 0.24f})}},
    {256, 1, {{128, 32, 1, {0.35f, 1.291f, 10.68f, 1.291f, 0.22f}, nullptr}, {128, 32, 1, {0.35f, 1.291f, 10.68f, 1.291f, 0.22f}, nullptr}},
     {form<256, 1, 4, 2, 64, 2>(1, {0.34f, 1.459f, 10.02f, 1.459f, 0.15f})}},
};

float predicted_us(const Form& f, int BH, const Bf16Problem& prob, int d, int causal) {
    const long long wgs = (long long)BH * ((prob.Nq + (long long)f.rows - 1) / f.rows), per_cu = (wgs + 255) / 256;
    const float tiles = (float)((prob.Nk + (long long)f.keys_per_tile - 1) / f.keys_per_tile);
    const float alone = tiles * f.cost.step + f.cost.fixed;             // one workgroup, start to end
    const float fixed_busy = f.cost.fixed * f.cost.busy / f.cost.step;  // its fixed part on a full compute unit
    const float memory = (float)BH * ((float)prob.Nq + (float)prob.Nk) * (float)d * 4.0f / 5.5e6f;  // K, V, Q, O once at 5.5 TB/s
    float work;
    if (!causal) {
        const float rounds = (float)((per_cu + f.per_cu - 1) / f.per_cu) * alone, full = (float)per_cu * (tiles * f.cost.busy + fixed_busy);
        work = rounds > full ? rounds : full;
    } else {  // the longest workgroup, or an even share of the work and what the longest one sticks out
        float seen = ((float)prob.causal_offset + 0.5f * (float)prob.Nq + 0.5f * (float)f.rows) / (float)f.keys_per_tile + 0.5f;
        if (seen > tiles) seen = tiles;
        const float spread = (float)wgs / 256.0f * (seen * f.cost.busy + fixed_busy) + f.cost.skew * alone;
        work = alone > spread ? alone : spread;
    }
    return f.cost.start + (work > memory ? work : memory);
}

// The key-group form for this problem, or null where the shape `index` is predicted to take no more than 1.1 times as long
// (what the prediction is worth) or there is one tile, and so nothing to divide.  Up to 512 keys index 0 also keeps launches of
// more than 512 blocks of 32 rows (forms gain 20 % at most there: 128 heads x 256, d = 64, 10.2 -> 8.0 us) and all of
// d = 32 (16 x 512, 9.7 -> 4.9 us): a caller may hold flat_attn_fwd to flat_attn_fwd_tile 0 bit for bit, and so do the tests.
const Form* key_group_form(int BH, const Bf16Problem& prob, int d, int causal, int index) {
    if (prob.Nk <= 64) return nullptr;
    if (index == 0 && prob.Nk <= 512 && (d == 32 || (long long)BH * ((prob.Nq + 31LL) / 32) > 512)) return nullptr;
    for (const Choice& c : kChoices) {
        if (c.d != d) continue;
        const Form* best = nullptr;
        float limit = predicted_us(c.base[index == 0 ? 0 : 1], BH, prob, d, causal) / 1.1f;
        for (int i = 0; i < c.n_forms; ++i) {
            const float t = predicted_us(c.forms[i], BH, prob, d, causal);
            if (t < limit) limit = t, best = &c.forms[i];
        }
        return best;
    }
    return nullptr;
}

}  // namespace

// A caller's tile shape is run as it is, except that the shape for small launches includes its key-group forms: what
// flat_attn_fwd does with an index is what flat_attn_fwd_tile does with it.
hipError_t launch_fwd_bf16_tile(const void* Q, const void* K, const void* V, void* O, int BH, const Bf16Problem& prob, int d,
                                float scale, int causal, int index, hipStream_t stream) {
    const Entry* e = find(d, index);
    if (!e) return hipErrorInvalidValue;
    const Form* f = index != 0 && index == small_launch_shape(d) ? key_group_form(BH, prob, d, causal, index) : nullptr;
    return (f ? f->launch : e->launch)(Q, K, V, O, BH, prob, scale, causal, stream);
}

hipError_t launch_fwd_bf16(const void* Q, const void* K, const void* V, void* O, int BH, const Bf16Problem& prob, int d,
                           float scale, int causal, hipStream_t stream) {
    const int index = default_tile_shape(BH, prob.Nq, d, causal);
    const Form* f = key_group_form(BH, prob, d, causal, index);
    return (f ? f->launch : table(d)[index].launch)(Q, K, V, O, BH, prob, scale, causal, stream);
}

}  // namespace flat
