// Host-side planning (no device code): which key-group form a launch takes, and for a split-keys launch how many workgroups
// share the keys of a row block, how many tiles each takes, and how large the workspace for their partial results is.
#include "flat_launch.hpp"

namespace flat {

namespace {

// The 128-row shape of a head size, for launches of few query rows (0: there is none).
int small_launch_shape(int d) { return d == 64 ? 7 : d == 128 ? 2 : d == 32 || d == 96 ? 1 : 0; }

}  // namespace

// ---- Key-group forms.  A launch of few query rows leaves most of the chip idle on the base shapes, whatever their rows per
// workgroup, because each workgroup walks all keys alone.  In these forms the wavefronts of a workgroup share the keys of
// the same 32, 64 or 128 rows (kernel parameter KG) and merge through LDS at the end; nothing else changes.  They re-read K
// and V from L2 more often per flop, so large launches keep the base shapes.  Each holds a step of K and V per wavefront in
// a ring of two stages (K runs one tile ahead of V); deeper rings measured 3-25 % slower where they cost a workgroup per
// compute unit, so only d = 32, whose tiles are small, has four.
// Measured, us, best base shape -> form: 12 heads x 512, d = 64, 7.8 -> 5.1; 4 x 4096, d = 64, 40.1 -> 24.8, causal 40.0 -> 20.4;
// 4 x 4096, d = 256, 110.7 -> 86.7, causal 109.3 -> 76.1; 64 x 16 rows over 4096 keys, d = 64, 46 -> 22.
//
// The choice is by predicted time.  A form (and each base shape) has five measured costs: us to launch, start and drain (`start`),
// us per tile and per workgroup when a workgroup runs alone (`step`, `fixed`), us per tile when the compute unit holds as
// many workgroups as fit (`busy`), and the share of its longest workgroup that a causal launch ends late (`skew`).  They were
// fitted by hand-run least squares to 1750 timings (1 to 2048 heads, 16 to 300 query rows over 300 to 4096 keys and 64 to 16384
// positions, both masks, five head sizes, inputs that stay in the caches), before the steps, the epilogue and the start of a workgroup
// took their present form.  (Refitted to 21671 timings of the kernels as they are, the choice was no better: 1.0 % behind the fastest on average
// against 0.9 %.)  What it is worth on the kernels as they are, python -m paper_2107_06419_amd.tile_sweep --forms
// says: over 1050 self-attention problems it is 0-2 % behind the fastest on average, 35 % at worst, where the better base
// shape is 9-24 % behind on average, and no form that runs is more than 12 % slower than the base shape it replaces.
namespace {

struct Cost {
    float start, step, fixed, busy, skew;
};
struct Form {
    int rows, keys_per_tile, per_cu;  // query rows per workgroup, keys per tile, workgroups per compute unit the costs were fitted with
    Cost cost;
};
// Per head size: the base shapes (index 0, small_launch_shape), then the key-group forms in the order of the tile table.
struct Choice {
    int d, n_forms;
    Form base[2];
    Form forms[4];
};
const Choice kChoices[] = {
    {32, 3, {{256, 64, 2, {2.51f, 0.854f, 1.55f, 0.685f, 0.38f}}, {128, 64, 3, {2.95f, 0.530f, 0.80f, 0.362f, 0.18f}}},
     {{32, 128, 2, {1.67f, 0.379f, 2.00f, 0.233f, 0.30f}}, {64, 128, 1, {2.95f, 0.378f, 1.48f, 0.378f, 0.29f}},
      {64, 64, 3, {2.74f, 0.327f, 1.19f, 0.194f, 0.08f}}}},
    {64, 3, {{256, 64, 2, {3.88f, 1.031f, 1.67f, 0.995f, 0.35f}}, {128, 64, 3, {3.03f, 0.666f, 1.59f, 0.532f, 0.22f}}},
     {{32, 128, 2, {2.05f, 0.520f, 2.43f, 0.367f, 0.21f}}, {64, 128, 1, {1.30f, 0.611f, 4.37f, 0.611f, 0.21f}},
      {64, 64, 3, {1.61f, 0.421f, 3.01f, 0.294f, 0.17f}}}},
    {96, 4, {{256, 64, 1, {0.27f, 1.325f, 5.38f, 1.325f, 0.30f}}, {128, 64, 1, {0.57f, 0.857f, 4.69f, 0.857f, 0.19f}}},
     {{32, 128, 1, {1.19f, 0.756f, 3.51f, 0.756f, 0.17f}}, {64, 128, 1, {0.70f, 0.899f, 5.60f, 0.899f, 0.18f}},
      {64, 64, 2, {1.37f, 0.548f, 3.60f, 0.420f, 0.17f}}, {128, 64, 1, {0.34f, 0.693f, 6.15f, 0.693f, 0.22f}}}},
    {128, 4, {{256, 64, 1, {0.33f, 1.609f, 7.00f, 1.609f, 0.29f}}, {128, 64, 1, {0.42f, 1.003f, 6.14f, 1.003f, 0.20f}}},
     {{32, 128, 1, {1.17f, 0.861f, 4.64f, 0.861f, 0.17f}}, {64, 128, 1, {0.67f, 1.038f, 7.67f, 1.038f, 0.19f}},
      {64, 64, 2, {1.82f, 0.588f, 4.40f, 0.489f, 0.23f}}, {128, 64, 1, {0.40f, 0.831f, 8.27f, 0.831f, 0.24f}}}},
    {256, 1, {{128, 32, 1, {0.35f, 1.291f, 10.68f, 1.291f, 0.22f}}, {128, 32, 1, {0.35f, 1.291f, 10.68f, 1.291f, 0.22f}}},
     {{64, 64, 1, {0.34f, 1.459f, 10.02f, 1.459f, 0.15f}}}},
};

const Choice* choice_of(int d) {
    for (const Choice& c : kChoices)
        if (c.d == d) return &c;
    return nullptr;
}

float predicted_us(const Form& f, int BH, const Bf16Problem& prob, int d, int causal) {
    const long long wgs = (long long)BH * ((prob.Nq + (long long)f.rows - 1) / f.rows), per_cu = (wgs + 255) / 256;
    const float tiles = (float)((prob.Nk + (long long)f.keys_per_tile - 1) / f.keys_per_tile);
    const float alone = tiles * f.cost.step + f.cost.fixed;             // one workgroup, start to end
    const float fixed_busy = f.cost.fixed * f.cost.busy / f.cost.step;  // its fixed part on a full compute unit
    // K, V, Q, O once at 5.9 TB/s; one workgroup per unit leaves that rate with the units that have nothing in the last round
    float memory = (float)BH * ((float)prob.Nq + (float)prob.Nk) * (float)d * 4.0f / 5.9e6f;
    if (f.per_cu == 1) memory *= (float)per_cu * 256.0f / (float)wgs;
    if (wgs < 256) memory = 0.0f;  // and few workgroups never reach it: `step` holds their rate
    float work;
    if (!causal) {
        const float rounds = (float)((per_cu + f.per_cu - 1) / f.per_cu) * alone, full = (float)per_cu * (tiles * f.cost.busy + fixed_busy);
        work = rounds > full ? rounds : full;
    } else {  // the longest workgroup, or an even share of the work and what the longest one sticks out
        float seen = ((float)prob.causal_offset + 0.5f * (float)prob.Nq + 0.5f * (float)f.rows) / (float)f.keys_per_tile + 0.5f;
        if (seen > tiles) seen = tiles;
        const float spread = (float)wgs / 256.0f * (seen * f.cost.busy + fixed_busy) + f.cost.skew * alone;
        work = alone > spread ? alone : spread;
        // No less than whole rounds of the shortest workgroup: the rows of a short segment behind many keys all see nearly the
        // same number of them, and then a workgroup too many costs a round (86 heads, 142 rows over 5726 keys, d = 256: 351 us in
        // 258 workgroups of 64 rows, 243 in 172 of 128).
        float least = ((float)prob.causal_offset + (float)f.rows) / (float)f.keys_per_tile;
        if (least > tiles) least = tiles;
        const float rounds = (float)((per_cu + f.per_cu - 1) / f.per_cu) * (least * f.cost.step + f.cost.fixed);
        const float full = (float)per_cu * (least * f.cost.busy + fixed_busy), even = rounds > full ? rounds : full;
        if (even > work) work = even;
        // Causal launches deal a head's row blocks over the XCDs, so the first few of them fetch its keys each for itself, at 6.5 TB/s
        // (162 heads, 194 rows over 5060 keys, d = 64: 142 us in 64-row workgroups, 90 in 128-row ones).
        const long long blocks = wgs / BH;
        const float fetched = (float)BH * (float)(blocks < 8 ? blocks : 8) * seen * (float)f.keys_per_tile * (float)d * 4.0f / 6.5e6f;
        if (blocks > 1 && fetched > memory) memory = fetched;
    }
    return f.cost.start + (work > memory ? work : memory);
}

// The shape a launch takes if none of its key-group forms is faster: index 0, except where a measured sweep (python -m
// paper_2107_06419_amd.tile_sweep --small: 1 to 512 heads of 128 to 8192 positions, both masks, several machines)
// shows the 128-row shape of the head dimension ahead:
//   * launches too small to give every compute unit a 256-row workgroup - at most 128 blocks of 256 query rows (causal:
//     256 at d = 32 / 64, 192 at d = 96 / 128): 1.3-1.5 times faster, simply because twice as many compute units work;
//   * d = 64 with the causal mask, up to 4096 positions and 1024 row blocks: ahead by up to 15 %, never behind;
//   * d = 32 with the causal mask up to 8192 positions (4-18 %: the vector side is the longer pole there and three workgroups per
//     compute unit hide more of it);
//   * up to 128 query rows, where half of a 256-row workgroup or more would be padding (256 heads of 16 rows over 1024
//     keys, d = 64: 23 us on 256 rows, 16 on 128; 2048 heads of 100 rows: 162 and 119 us).
// At d = 64 and 32 without a mask the predicted times of the two decide, by 3 %.  Half the rows per workgroup and three workgroups per compute
// unit instead of two waste less on the last row block and the last round, and cost 4-8 % where neither counts: 87 heads x 537, d = 64,
// 21.5 us on 256 rows, 14.8 on 128; 143 x 316 14.7 and 10.3; 26 x 3302 96.7 and 86.2; 457 x 849 124 and 111; 16 x 16384 1029 and 1145.
// Over 12200 random problems (profiles/row_shapes_key_counts.md) the shape taken is 1.5 % (d = 64) and 0.2 % (d = 32) behind the faster one on
// average and 14 and 5 % at the 99th percentile; with rules on the number of row blocks it was 8.4 and 5.3 %.
// With key counts, which the host does not know, the 128-row shape is taken up to 5 % behind: the times are predicted for all keys, and where
// entries differ many short workgroups even out better.  Over 13300 random problems: counts from half the keys to all of them, d = 64,
// 0.8 % behind on average and 10 % at the 99th percentile (with 1.03 for 0.95: 2.8 and 28 %), from an eighth 1.5 and 16 % (4.9 and 45 %), all
// keys in every entry 0.6 and 12 % (1.5 and 14 %); d = 32 0.8, 1.0 and 0.5 % (0.8, 1.5 and 0.3 %).
// Heads of exactly 256 or 512 rows keep to the rules on row blocks for no better reason than that their indices were tested as they are (129
// heads x 512: index 0, 128 x 256: a key-group form): the predicted time would serve them as well as other lengths (512 rows, d = 64: 1.9 %
// behind the faster shape on average, 4.6 % as it is; 129 to 192 heads x 512 lose 16-18 %).
int base_tile_shape(int BH, const Bf16Problem& prob, int d, int causal) {
    const int Nq = prob.Nq;
    const long long blocks = (long long)BH * (((long long)Nq + 255) / 256);  // 256-row blocks in the launch
    if (Nq <= 128 && d != 256) return small_launch_shape(d);  // a 256-row workgroup would be at least half padding
    if ((d == 64 || d == 32) && !causal && (Nq > 512 || Nq % 256 != 0)) {
        const Form* base = choice_of(d)->base;
        const float margin = prob.kv_lens ? 0.95f : 1.03f;
        return predicted_us(base[1], BH, prob, d, 0) * margin < predicted_us(base[0], BH, prob, d, 0) ? small_launch_shape(d) : 0;
    }
    switch (d) {
        case 32: return causal && Nq <= 8192 ? 1 : 0;
        case 64:
            if (causal) return (Nq > 256 && blocks <= (Nq <= 4096 ? 1024 : 256)) ? 7 : 0;
            return (Nq > 256 && blocks <= 128) ? 7 : 0;
        case 96: return blocks <= (causal ? 192 : 128) ? 1 : 0;
        case 128: return blocks <= (causal ? 192 : 128) ? 2 : 0;
        default: return 0;
    }
}

// The key-group form for this problem, as its position in the table, or -1 where the shape `index` is predicted to take no more than 1.1
// times as long (what the prediction is worth) or there is one tile, and so nothing to divide.
int key_group_form(int BH, const Bf16Problem& prob, int d, int causal, int index) {
    // At d = 256 three tiles of the base shape are no more work than two of the form's: 8 x 65 without a mask 10.6 us, in the form
    // 12.0, 7 causal heads, 55 rows over 80 keys, 10.8 and 12.1.  In causal self-attention the form wins there too (2 x 75: 10.5 and 11.4).
    const bool triangle = causal && prob.causal_offset == 0;
    if (prob.Nk <= (d == 256 && !triangle ? 96 : 64)) return -1;
    const Choice* c = choice_of(d);
    if (!c) return -1;
    int best = -1;
    float limit = predicted_us(c->base[index == 0 ? 0 : 1], BH, prob, d, causal) / 1.1f;
    for (int i = 0; i < c->n_forms; ++i) {
        const float t = predicted_us(c->forms[i], BH, prob, d, causal);
        if (t < limit) limit = t, best = i;
    }
    return best;
}

}  // namespace

// The index flat_attn_fwd / flat_attn_fwd_cross run: a base shape or its key-group form.
int chosen_tile_shape(int BH, const Bf16Problem& prob, int d, int causal) {
    const int base = base_tile_shape(BH, prob, d, causal), form = key_group_form(BH, prob, d, causal, base);
    return form < 0 ? base : first_key_group_form(d) + form;
}

namespace {
// The tile shape a split-keys launch uses: rows per workgroup, keys per tile, padded head dimension, workgroups wanted per
// compute unit, the keys it takes at least per split, and its measured cost: us to start and drain, us per unit of 64 keys (32 at
// d = 256) of a workgroup alone and with the compute unit full.  Every workgroup multiplies a full tile of `rows` rows whatever Nq
// is, so few query rows take a shape with fewer rows where flat_splitkv.hip builds one.
struct Geometry { int rows, keys, dp, per_cu, min_keys; float start, step, busy; };
bool geometry(int d, int Nq, Geometry* g) {
    switch (d) {
        case 32:
            if (Nq <= 32) *g = {32, 64, 32, 6, 128, 3.2f, 0.40f, 0.10f};
            else if (Nq <= 64) *g = {64, 64, 32, 4, 256, 5.0f, 0.50f, 0.20f};
            else if (Nq <= 128) *g = {128, 64, 32, 2, 512, 6.0f, 0.53f, 0.45f};
            else *g = {256, 64, 32, 2, 512, 7.0f, 0.85f, 0.75f};
            return true;
        case 64:
            if (Nq <= 32) *g = {32, 64, 64, 3, 128, 3.0f, 0.45f, 0.20f};
            else if (Nq <= 64) *g = {64, 64, 64, 2, 256, 5.5f, 0.65f, 0.40f};
            else if (Nq <= 128) *g = {128, 64, 64, 2, 512, 6.0f, 0.66f, 0.60f};
            else *g = {256, 64, 64, 2, 512, 8.0f, 1.00f, 1.00f};
            return true;
        case 96:
            if (Nq <= 32) *g = {32, 32, 128, 4, 64, 2.8f, 1.00f, 0.30f};
            else if (Nq <= 128) *g = {128, 64, 128, 1, 256, 6.5f, 0.86f, 0.86f};
            else *g = {256, 64, 128, 1, 512, 9.0f, 1.20f, 1.20f};
            return true;
        case 128:
            if (Nq <= 32) *g = {32, 32, 128, 4, 64, 2.8f, 1.20f, 0.40f};
            else if (Nq <= 128) *g = {128, 64, 128, 1, 256, 7.0f, 0.94f, 0.94f};
            else *g = {256, 64, 128, 1, 512, 9.0f, 1.36f, 1.36f};
            return true;
        case 256:
            if (Nq <= 64) *g = {64, 32, 256, 2, 64, 4.0f, 1.22f, 0.70f};
            else *g = {128, 32, 256, 1, 256, 10.0f, 1.29f, 1.29f};
            return true;
        default: return false;
    }
}
// Predicted time of the launch without splits, and of partial pass and merge: the longer of the chain of one workgroup, the
// work of a compute unit and one read of K and V, then the merge (4.3 us and 1.2 ns a row) and the partial results' round trip.
// The former is that of the fastest shape or form, without a mask, which the plan does not know; the launch may take another
// one.  (Predicting the one that is launched moved 125 of 28900 plans; of 96 timed, 62 got slower, by up to 15 %.)
float unsplit_us(int BH, int Nq, int Nk, int d) {
    const Bf16Problem prob{Nq, Nk, 0, 1, nullptr, nullptr, nullptr, 0};
    float best = 1e30f;
    for (const Choice& c : kChoices) {
        if (c.d != d) continue;
        for (int i = -2; i < c.n_forms; ++i) {
            const float t = predicted_us(i < 0 ? c.base[i + 2] : c.forms[i], BH, prob, d, 0);
            if (t < best) best = t;
        }
    }
    return best;
}
float split_us(const Geometry& g, long long blocks, int BH, int Nq, int Nk, int d, long long splits, int n_units) {
    const float units = (float)((n_units + splits - 1) / splits), per_cu = (float)((blocks * splits + 255) / 256);
    const float alone = g.step * units, full = g.busy * units * per_cu, memory = (float)BH * (float)Nk * (float)d * 4.0f / 5.9e6f;
    float t = alone > full ? alone : full;
    if (memory > t) t = memory;
    return g.start + t + 4.3f + 0.0012f * (float)BH * (float)Nq + (float)BH * (float)Nq * (float)splits * (float)(g.dp + 2) * 8.0f / 4.0e6f;
}
constexpr int kComputeUnits = 256;
constexpr int kMaxSplits = 256;        // of one row block: its merge is one workgroup's work
}  // namespace

bool split_plan(int BH, int Nq, int Nk, int d, int n_splits_wanted, SplitPlan* out) {
    Geometry g;
    if (BH <= 0 || Nq <= 0 || Nk <= 0 || !geometry(d, Nq, &g)) return false;
    SplitPlan p;
    p.rows_per_block = g.rows;
    p.padded_d = g.dp;
    p.n_row_blocks = (int)(((long long)Nq + g.rows - 1) / g.rows);
    // splits are counted in units of 64 keys (32 at d = 256), whatever the tile of the shape
    const int unit = d == 256 ? 32 : 64, tiles_per_unit = unit / g.keys;
    const int n_units = (int)(((long long)Nk + unit - 1) / unit);
    long long s = n_splits_wanted, reserved = 0;
    if (s <= 0) {
        // One workgroup per wanted slot of the chip and no more: a workgroup beyond them only adds partial results to write
        // and merge (and a second round), one split fewer leaves some slots empty.  Every split stays long enough to pay for itself.
        const long long blocks = (long long)BH * p.n_row_blocks;
        s = kComputeUnits * g.per_cu / blocks;
        const long long longest = ((long long)Nk + g.min_keys - 1) / g.min_keys;
        if (s < 2) s = 2;  // more heads than slots: still twice as many workgroups, as the last round is half empty otherwise
        if (s > longest) s = longest;
        if (s > kMaxSplits) s = kMaxSplits;
        reserved = s < n_units ? s : n_units;
        // No split where one launch does it in less (many heads over short keys, or enough rows to fill the chip: 64 heads x 200
        // rows over 2048 keys, d = 64, 37.7 -> 17.1 us, 256 x 1 over 512 keys 11.7 -> 8.2) by a clear margin: key counts of different
        // length favour the many short workgroups of a split launch, and over many keys that no cache holds the few long
        // workgroups of one launch take longer than predicted (12 heads x 250 rows over 5597 keys, d = 64, in one launch 42.8 us,
        // 27.4 predicted; 11 splits 25.5, 28.3 predicted).  Margins by the keys, on 1817 random problems: 31 calls are more than
        // 3 % slower than with the rule before key-group forms (every slot, at least 8 tiles per split), 58 with margins of 1.12
        // up to 64 rows and none above.
        const float margin = Nk < 2048 ? 1.12f : Nk < 4096 ? 1.25f : 1.6f;
        if (s > 1 && unsplit_us(BH, Nq, Nk, d) * margin <= split_us(g, blocks, BH, Nq, Nk, d, s, n_units)) s = 1;
    }
    if (s > n_units) s = n_units;
    if (s < 1) s = 1;
    const int units_per_split = (int)((n_units + s - 1) / s);
    p.n_splits = (n_units + units_per_split - 1) / units_per_split;  // no split is left without a unit
    p.tiles_per_split = units_per_split * tiles_per_unit;
    const unsigned __int128 bytes = (unsigned __int128)BH * p.n_row_blocks * p.n_splits * g.rows * (g.dp + 2) * sizeof(float);
    if (bytes >= ((unsigned __int128)1 << 62) || (long long)BH * p.n_row_blocks * p.n_splits > 0x7fffffffLL) return false;
    if ((long long)BH * Nq > 0x7fffffffLL) return false;  // the merge launches one workgroup per (head, row)
    p.used_bytes = (size_t)bytes;
    // The number of splits falls and rises with the keys, by rounding and by the choice of one launch; what the caller is asked to
    // hold never falls, so that a workspace for the longest cache serves every shorter one.
    p.workspace_bytes = reserved > p.n_splits ? p.used_bytes / p.n_splits * reserved : p.used_bytes;
    *out = p;
    return true;
}

}  // namespace flat
