// How a support launch covers its rows and units: the kernel's forms, the sizes of their LDS buffers
// and the choice among them (host code, but for the constants; k_support.hip has the kernels).
#pragma once

#include <initializer_list>

#include "bcpnn_internal.h"

namespace bcpnn {

constexpr int kRows = 16;          // batch rows per row tile
constexpr int kMaxWaves = 16;
constexpr int kCus = 256;                 // compute units
constexpr int64_t kL2Bytes = 32 << 20;    // of all XCDs
constexpr int kXcds = 8;
constexpr int kFewUnits = 16;             // with so few units a launch costs its workgroups, not its work
constexpr int kMinSplit = 16;             // least workgroups for the input's split
constexpr int kOneUnits = 1024;           // unit table of the one-chunk variants
constexpr int kOneBytes = 120 * 1024;     // their panels and table
constexpr int kManyTiles = 4;             // row tiles per workgroup of the many-rows variant
// Bytes of a stage buffer: with one row tile a launch of few workgroups takes most of a CU's LDS (the
// chunks are then few); kManyTiles row tiles, and the form of two workgroups per CU (`pair`), leave
// room for a second workgroup.
constexpr int stage_bytes(int rows, bool pair) {
    return rows > 1 ? 26 * 1024 : pair ? 37 * 1024 : 73 * 1024;
}
// Column tiles per wave: a stride takes at most sixteen waves.
constexpr int tiles_per_wave(int stride) { return stride <= 256 ? 1 : stride / 256; }
constexpr int kXRegs = 12;                // input elements a thread holds per chunk

struct SupportLayout {
    int n_tiles;                   // 16-column tiles of a hidden HCU
    int groups;                    // waves that share the column tiles (tile t: wave t mod groups)
    int parts;                     // waves that share a tile's k-steps; groups * parts waves
    int kc;                        // units per chunk
    int n_chunks;
    int k_alloc;                   // unit table: win chunks, the last in whole runs of 64 units
    int max_k;                     // largest number of active units of a hidden HCU
    uint32_t mcu_magic;            // ceil(2^32 / in_mcu) (0 for in_mcu = 1)
    int per;                       // k-steps of a share in a whole chunk
    int vec4;                      // weight rows move 16 bytes per lane
    int rw, x_slots;               // input rows per wave, loads per thread and chunk
    int xstride, mpad;             // LDS row strides of the input panel and the support tile
    int n_split;                   // workgroups that split the input
    int sum_order;                 // of the input's column sums
    int n_row_groups;              // groups of kR row tiles
    int row_major;                 // workgroup order: hidden HCUs of a row group together
    int n_main;                    // support workgroups; those past it split the input
    int n_row_tiles;
    int win;                       // chunks whose units the table holds at a time
};

constexpr size_t kLdsLimit = 160 * 1024;   // LDS of one gfx950 workgroup

// How a launch covers its rows and units.
enum Shape { kOneChunk, kChunks, kManyRows, kFewOne, kFewChunks, kTwoPerCu, kShapes };

constexpr int shape_rows(int v) { return v == kManyRows ? kManyTiles : 1; }
constexpr bool shape_one(int v) { return v == kOneChunk || v == kFewOne; }

// The weight panel's row stride for M_out columns: 16, 80 (both 16 mod 64, so that the four rows of
// an operand read fall on different banks), then powers of two.  (A stride per 16 columns would
// multiply the kernels; between 16 and 80 the launch bounds such HCUs more than their panel.)
inline int panel_stride(int out_mcu) {
    if (out_mcu <= 80) return out_mcu <= 16 ? 16 : 80;
    int s = 128;
    while (s < out_mcu) s *= 2;
    return s;
}

inline uint32_t magic_of(int d) { return (uint32_t)(((1ull << 32) + (uint64_t)d - 1) / (uint64_t)d); }

inline int input_vec(const Geometry& g) { return g.in_mcu % 2 == 0 ? 2 : 1; }

// Workgroups of a training launch that split the input, beside the support's n_main: a wave per
// task, or on the CUs that the support leaves idle.
inline int64_t split_workgroups(const Geometry& g, const SupportLayout& lay) {
    const int n_waves = lay.groups * lay.parts;
    int64_t n_split = ((int64_t)lay.n_row_tiles * ((g.n_in + 63) / 64) + n_waves - 1) / n_waves;
    if (lay.n_main < kCus && n_split > kCus - lay.n_main)
        n_split = kCus - lay.n_main > kMinSplit ? kCus - lay.n_main : n_split < kMinSplit ? n_split : kMinSplit;
    return n_split;
}

// Whether a launch of this layout keeps below 2^32 work-items (what a grid can have).
inline bool launchable(const Geometry& g, const SupportLayout& lay, bool ops) {
    const int64_t workgroups = lay.n_main + (ops ? split_workgroups(g, lay) : 0);
    return workgroups * lay.groups * lay.parts * 64 < (int64_t)1 << 32;
}

// The most rows of one launch: its inputs have 32-bit byte offsets, and its row tiles x hidden HCUs
// workgroups keep below 2^32 work-items with the waves that the columns need (eight, sixteen above 128
// MCUs).  Layers of more rows than that do not fit the device's memory; a prediction's launches, which
// no batch size bounds, are cut to it.
inline int64_t most_rows(const Geometry& g) {
    const int64_t by_inputs = (int64_t)(UINT32_MAX / 4) / g.n_in;
    const int64_t by_items = (((int64_t)1 << (g.out_mcu > 128 ? 26 : 27)) - 1) / g.out_hcu;
    return (by_inputs < by_items ? by_inputs : by_items) / kRows * kRows;
}

// Layout of a launch in one shape and its dynamic LDS, or false when the shape does not cover the
// sizes.  ops: training.
inline bool make_layout(const Geometry& g, int32_t B, int32_t max_k, int v, bool ops, SupportLayout* out,
                        size_t* dyn_bytes) {
    SupportLayout L{};
    const int kR = shape_rows(v), ps = panel_stride(g.out_mcu);
    const int tpw = tiles_per_wave(ps);
    const bool pair = v == kTwoPerCu;
    if (v != kChunks && ps > (pair ? 256 : 128)) return false;
    if (pair && ps < 128) return false;
    L.n_tiles = (g.out_mcu + 15) / 16;
    L.groups = (L.n_tiles + tpw - 1) / tpw;
    L.max_k = max_k > 0 ? max_k : 1;
    L.mcu_magic = g.in_mcu > 1 ? magic_of(g.in_mcu) : 0;
    L.vec4 = g.out_mcu % 4 == 0 && g.n_out % 4 == 0;
    L.mpad = (g.out_mcu + 15) / 16 * 16 + 4;
    const int xv = input_vec(g);
    const int64_t n_main = ((int64_t)(B + kR * kRows - 1) / (kR * kRows)) * g.out_hcu;
    if (n_main > INT32_MAX / 2) return false;
    L.n_main = (int)n_main;
    L.n_row_tiles = (B + kRows - 1) / kRows;
    const int waves = kR == 1 && !shape_one(v) && !pair ? kMaxWaves : 8;
    L.parts = waves / L.groups > 0 ? waves / L.groups : 1;
    // the chunk; the rows of the input panel lie 4 mod 8 words apart, so that the 16 rows x 4 units
    // of an operand read fall on different banks
    auto stride = [v](int kc) {
        if (shape_one(v)) return (kc + 1) / 2 % 2 ? (kc + 1) / 2 * 2 : (kc + 1) / 2 * 2 + 2;   // fp64
        return (kc + 3) / 4 % 2 ? (kc + 3) / 4 * 4 : (kc + 3) / 4 * 4 + 4;                     // fp32
    };
    const int x_bytes = shape_one(v) ? 8 : 4;              // per element of the input panel
    auto bytes = [&](int kc) { return 4 * kc * ps + x_bytes * kR * kRows * stride(kc); };
    L.rw = (kR * kRows + L.groups * L.parts - 1) / (L.groups * L.parts);
    auto slots = [&](int kc) { return L.rw * ((kc + 64 * xv - 1) / (64 * xv)); };
    const int most_slots = kXRegs / xv;
    if (shape_one(v)) {
        L.kc = (L.max_k + 3) / 4 * 4;
        if (L.kc > kOneUnits || slots(L.kc) > most_slots || bytes(L.kc) + 4 * kOneUnits > kOneBytes) return false;
    } else {
        const int cap = stage_bytes(kR, pair);
        L.kc = cap / (4 * ps + x_bytes * kR * kRows) / 4 * 4;
        while (L.kc > 4 && bytes(L.kc) > cap) L.kc -= 4;
        if (L.kc < 4 || bytes(L.kc) > cap) return false;
        if (L.kc > (L.max_k + 3) / 4 * 4) L.kc = (L.max_k + 3) / 4 * 4;
    }
    L.xstride = stride(L.kc);
    L.n_chunks = (L.max_k + L.kc - 1) / L.kc;
    auto entries = [&](int chunks) { return (L.kc * (chunks - 1) + (L.kc + 63) / 64 * 64 + 63) / 64 * 64; };
    L.win = L.n_chunks;
    L.k_alloc = entries(L.n_chunks);
    const int steps = (L.kc + 3) / 4;                          // no share without a k-step
    if (L.parts > steps) L.parts = steps;
    // the shares' sums, and with one row tile as many shares as leave them room behind the support
    // tile's half in the first stage
    const size_t vals = v == kFewOne || v == kFewChunks ? (size_t)tpw : (size_t)4 * kR * tpw;
    const size_t tile = (size_t)kR * kRows * L.mpad * sizeof(float);
    const size_t stage = shape_one(v) ? 16 : (size_t)stage_bytes(kR, pair);
    auto sums_of = [&](int parts) { return (size_t)(parts - 1) * L.groups * vals * 64 * sizeof(double); };
    if (!shape_one(v) && kR == 1)
        while (L.parts > 1 && tile / 2 + sums_of(L.parts) > stage) --L.parts;
    while (L.parts > 1 && !launchable(g, L, ops)) --L.parts;
    if (!launchable(g, L, ops)) return false;
    L.per = (steps + L.parts - 1) / L.parts;
    L.parts = (steps + L.per - 1) / L.per;
    L.rw = (kR * kRows + L.groups * L.parts - 1) / (L.groups * L.parts);
    L.x_slots = slots(L.kc);
    if (shape_one(v) && L.x_slots > most_slots) return false;
    L.n_row_groups = (L.n_row_tiles + kR - 1) / kR;
    // The row tiles of a hidden HCU one after another: its weights then stay in an XCD's L2, and so do
    // the inputs that every hidden HCU gathers again.  A batch beyond the L2s (32 MiB) and larger than
    // the weights is read once instead: the hidden HCUs of a row tile one after another.  (128 MCUs,
    // 1000 units, 100 HCUs at 128 rows 134 -> 126 us; 10 MCUs, 2764 of 55296 units, 30 HCUs at 1000
    // rows the other way, 305 against 539 us.)  Four row tiles share their weights as it is.
    const int64_t x_bytes_all = (int64_t)B * g.n_in * 4, w_bytes = (int64_t)L.max_k * g.n_out * 4;
    L.row_major = kR > 1 || (!shape_one(v) && x_bytes_all > kL2Bytes && x_bytes_all > w_bytes);
    // A table of every unit may leave no room for the stages (with one row tile, above 3500 units):
    // it then holds as many chunks' as fit (546x10 inputs, 4490 units active, 1x27, 144 rows: 105
    // us; four row tiles per workgroup, whose stages leave room, 269).
    if (!shape_one(v)) {
        const int64_t room = ((int64_t)kLdsLimit / (pair ? 2 : 1) - 16 - 2 * stage_bytes(kR, pair)) / 4;
        if (kR == 1 && L.k_alloc > room) {
            L.win = room - 128 >= L.kc ? (int)((room - 128) / L.kc) : 1;
            L.k_alloc = entries(L.win);
        }
    }
    const size_t table = shape_one(v) ? 0 : (size_t)L.k_alloc * 4;
    const size_t panel = shape_one(v) ? (size_t)bytes(L.kc) : 0;
    const size_t sums = sums_of(L.parts);
    if (!shape_one(v) && tile / 2 + (kR == 1 ? sums : 0) > stage) return false;
    const size_t after = shape_one(v) ? tile + sums : kR > 1 ? sums : 0;
    *dyn_bytes = table + panel > after ? table + panel : after;
    *out = L;
    const size_t fixed = 2 * stage + (shape_one(v) ? 4 * kOneUnits : 16);
    return fixed + *dyn_bytes <= kLdsLimit;
}

// Whether more workgroups than CUs share them in pairs, each with half of the stages, so that one's
// waits pass under the other's products.  It pays where one workgroup's waves load the SIMDs unevenly
// or are few: hidden HCUs of seven to twelve column tiles.  1000 units, 100 MCUs, 100 HCUs at 96 rows:
// 102 us alone, 89 in pairs; 176 MCUs, 156 units, 30 HCUs at 208 rows 33 and 29.  At six tiles a
// workgroup alone is the faster (96 MCUs: 4%), and from thirteen (200 MCUs, 1000 units: 10%).
inline bool two_per_cu(const Geometry& g, int64_t items) {
    return items > kCus && g.out_mcu > 96 && g.out_mcu <= 192;
}

// Time of a launch of more (row tile, hidden HCU) items than CUs, for the choice among its forms, as the
// rounds of workgroups that the CUs run one after another, each weighed with what it takes per row
// tile; the unit is a row tile of four, two workgroups to a CU.  What tells the forms apart: a group of
// row tiles costs four, dead ones too; a last round costs a whole one (less where every CU has one
// workgroup of it); a workgroup alone on its CU waits for its first chunk and at its end, which many
// units outweigh; and its waves may fill the SIMDs better (five column tiles: fifteen waves of a third of
// the k-steps each, with four row tiles five waves).  The weights are fitted to 1046 sizes and tried on
// 2500 (30 to 3000 HCUs, 2 to 128 MCUs, 3 to 3000 units, 2 to 4096 rows).  Against four row tiles from
// 1024 items on, whatever their rows, 17% faster on average: 1100 HCUs x 10 MCUs, 1000 units, 16 rows 157
// -> 62 us; 210 x 100, 80 rows 195 -> 142; 30 x 100 of 156 units, 512 rows 33 -> 26.
inline double launch_cost(const Geometry& g, int32_t B, const SupportLayout& L, int v, size_t lds) {
    const int full = L.n_main / (2 * kCus), rest = L.n_main % (2 * kCus);
    const double rounds = (L.n_main + kCus - 1) / kCus;          // one workgroup to a CU
    const double K = L.max_k;
    switch (v) {
        case kManyRows: {
            const bool shared = 2 * (2 * stage_bytes(kManyTiles, false) + 16 + lds) <= kLdsLimit;
            if (!shared) return 5.2 * rounds;
            return 8.0 * full + (rest == 0 ? 0.0 : rest <= kCus ? 5.2 : 8.0);
        }
        case kTwoPerCu:
            return 1.25 * (2.0 * full + (rest == 0 ? 0.0 : rest <= kCus ? 1.46 : 2.0));
        case kOneChunk:
            // panels that leave a CU a single workgroup; smaller ones, whose workgroups share it, where
            // an XCD's L2 holds the inputs that they gather
            if (2 * (4 * (size_t)kOneUnits + 32 + lds) > kLdsLimit) return 1.7 * rounds;
            if (L.n_tiles > 4) return 1.45 * rounds;
            return rounds * ((int64_t)B * g.n_in * 4 > kL2Bytes / kXcds ? 1.4 : 1.25);
        default: {
            // waves on the fullest SIMD per share of the k-steps
            const int many = 8 / L.n_tiles > 0 ? 8 / L.n_tiles : 1;
            const double here = (double)((L.groups * L.parts + 3) / 4) / L.parts;
            const double there = (double)((L.n_tiles * many + 3) / 4) / many;
            const double fill = L.n_tiles <= 8 ? 0.6 + 0.4 * here / there : 1.0;
            const double alone = (K + 300.0) / (0.85 * K + 30.0);
            return rounds * fill * (alone < 2.0 ? alone : 2.0);
        }
    }
}

// The form and layout of a launch and its dynamic LDS; -1 when no form covers the sizes.  ops:
// training.  One chunk where the units fit, else several; with more items than CUs another form where it
// costs less.
inline int choose_layout(const Geometry& g, int32_t B, int32_t max_k, bool ops, SupportLayout* lay,
                         size_t* lds) {
    const int64_t items = ((int64_t)B + kRows - 1) / kRows * g.out_hcu;
    int shape = -1;
    auto take = [&](int v) {
        if (shape < 0 && make_layout(g, B, max_k, v, ops, lay, lds)) shape = v;
    };
    if (!ops && B == 1) {
        take(kFewOne);
        take(kFewChunks);
    }
    take(kOneChunk);
    if (two_per_cu(g, items)) take(kTwoPerCu);
    take(kChunks);
    if (items <= kCus || shape == kFewOne || shape == kFewChunks) return shape;
    double least = shape < 0 ? 0.0 : launch_cost(g, B, *lay, shape, *lds);
    auto consider = [&](int v) {
        SupportLayout L;
        size_t bytes = 0;
        if (!make_layout(g, B, max_k, v, ops, &L, &bytes)) return;
        const double cost = launch_cost(g, B, L, v, bytes);
        if (shape >= 0 && cost >= least) return;
        shape = v;
        least = cost;
        *lay = L;
        *lds = bytes;
    };
    if (two_per_cu(g, items) && shape == kOneChunk &&
        2 * (4 * (size_t)kOneUnits + 32 + *lds) > kLdsLimit)
        consider(kTwoPerCu);
    if (shape != kOneChunk && max_k <= kFewUnits) least = 1e30;   // (one such workgroup fills a CU's LDS)
    // (one or two row tiles of four: never for their work)
    if (items > 2 * (int64_t)g.out_hcu || least == 1e30) consider(kManyRows);
    return shape;
}

}  // namespace bcpnn
