// Table of the tile shapes the fused bf16 kernel is built for, and the dispatch by index.  Index 0 of each head dimension is
// the shape large launches use; flat_plan.hip chooses the index of a launch, and the others are here so that the choice can
// be re-measured (the paper's map-space exploration, section 6.1, done by timing instead of a cost model; the trade-off being
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
    return Entry{TileShape{D, 32 * QB * NW, BCX ? BCX : bf16_keys_per_tile(D), NW, 32 * QB, STAGES, bf16_lds_bytes(D, QB, NW, STAGES, BCX, 1)},
                 &launch_fwd_bf16_shape<D, QB, NW, STAGES, BCX>, &fwd_bf16_shape_occupancy<D, QB, NW, STAGES, BCX>};
}

// Key-group form: KG groups of wavefronts share the keys of the same rows (flat_fwd_bf16_groups_*.hip).
template <int D, int QB, int NW, int STAGES, int BC, int KG>
constexpr Entry form() {
    return Entry{TileShape{D, 32 * QB * NW / KG, BC, NW, 32 * QB, STAGES, bf16_lds_bytes(D, QB, NW, STAGES, BC, KG)},
                 &launch_fwd_bf16_groups<D, QB, NW, STAGES, BC, KG>, &fwd_bf16_shape_occupancy<D, QB, NW, STAGES, BC, KG>};
}

const Entry kD64[] = {entry<64, 2, 4, 4>(), entry<64, 2, 4, 3>(), entry<64, 2, 4, 6>(), entry<64, 2, 8, 4>(),
                      entry<64, 1, 8, 4>(), entry<64, 1, 4, 4>(), entry<64, 2, 2, 4>(), entry<64, 1, 4, 3>(),
                      // the key-tile axis: 128 keys per tile (512-row and 256-row workgroups), 32 keys per tile
                      entry<64, 2, 8, 3, 128>(), entry<64, 2, 8, 4, 128>(), entry<64, 2, 4, 3, 128>(), entry<64, 2, 4, 6, 32>(),
                      form<64, 1, 4, 2, 128, 4>(), form<64, 1, 8, 2, 128, 4>(), form<64, 1, 4, 2, 64, 2>()};
const Entry kD128[] = {entry<128, 1, 8, 3>(), entry<128, 1, 8, 4>(), entry<128, 1, 4, 3>(), entry<128, 2, 4, 3>(),
                       form<128, 1, 4, 2, 128, 4>(), form<128, 1, 8, 2, 128, 4>(), form<128, 1, 4, 2, 64, 2>(), form<128, 1, 8, 2, 64, 2>()};
const Entry kD32[] = {entry<32, 2, 4, 4>(), entry<32, 1, 4, 4>(),
                      form<32, 1, 4, 4, 128, 4>(), form<32, 1, 8, 4, 128, 4>(), form<32, 1, 4, 4, 64, 2>()};
const Entry kD96[] = {entry<96, 1, 8, 3>(), entry<96, 1, 4, 3>(),
                      form<96, 1, 4, 2, 128, 4>(), form<96, 1, 8, 2, 128, 4>(), form<96, 1, 4, 2, 64, 2>(), form<96, 1, 8, 2, 64, 2>()};
const Entry kD256[] = {entry<256, 1, 4, 4>(), form<256, 1, 4, 2, 64, 2>()};
template <int N>
constexpr int length(const Entry (&)[N]) { return N; }
static_assert(length(kD32) == first_key_group_form(32) + 3 && length(kD64) == first_key_group_form(64) + 3 && length(kD96) == first_key_group_form(96) + 4 &&
              length(kD128) == first_key_group_form(128) + 4 && length(kD256) == first_key_group_form(256) + 1, "the forms end each table");

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
    if (d == 64) return length(kD64);
    if (d == 128) return length(kD128);
    if (d == 32) return length(kD32);
    if (d == 96) return length(kD96);
    if (d == 256) return length(kD256);
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

hipError_t launch_fwd_bf16_tile(const void* Q, const void* K, const void* V, void* O, int BH, const Bf16Problem& prob, int d,
                                float scale, int causal, int index, hipStream_t stream) {
    const Entry* e = find(d, index);
    return e ? e->launch(Q, K, V, O, BH, prob, scale, causal, stream) : hipErrorInvalidValue;
}

int default_tile_shape(int BH, int Nq, int d, int causal) {
    return chosen_tile_shape(BH, Bf16Problem{Nq, Nq, 0, 1, nullptr, nullptr, nullptr, 0}, d, causal);
}

hipError_t launch_fwd_bf16(const void* Q, const void* K, const void* V, void* O, int BH, const Bf16Problem& prob, int d,
                           float scale, int causal, hipStream_t stream) {
    return launch_fwd_bf16_tile(Q, K, V, O, BH, prob, d, scale, causal, chosen_tile_shape(BH, prob, d, causal), stream);
}

}  // namespace flat
