// Host check of the support's launch layouts (paper_2106_05373_amd/csrc/support_layout.h) over the
// sizes a layer can have: every one has a form that fits the LDS of a workgroup, with its tables,
// panels and sums inside their buffers.
#include <stdint.h>
#include <stdio.h>

#include "support_layout.h"

using namespace bcpnn;

static int failures = 0;
#define CHECK(cond, what)                                                                       \
    do {                                                                                        \
        if (!(cond) && ++failures <= 20)                                                        \
            printf("%s: %dx%d -> %dx%d, %d rows, %d units, %s: form %d\n", what, g.in_hcu,      \
                   g.in_mcu, g.out_hcu, g.out_mcu, B, max_k, ops ? "training" : "forward", v);  \
    } while (0)

static void check(const Geometry& g, int32_t B, int32_t max_k, bool ops) {
    SupportLayout L{};
    size_t lds = 0;
    const int v = choose_layout(g, B, max_k, ops, &L, &lds);
    CHECK(v >= 0, "no form");
    if (v < 0) return;
    const int kR = shape_rows(v), stride = panel_stride(g.out_mcu), tpw = tiles_per_wave(stride);
    const bool one = shape_one(v), few = v == kFewOne || v == kFewChunks;
    const int waves = L.groups * L.parts;
    const bool pair = v == kTwoPerCu;
    const size_t stage = one ? 16 : (size_t)stage_bytes(kR, pair);
    CHECK(2 * stage + (one ? 4 * kOneUnits : 16) + lds <= kLdsLimit, "LDS");
    CHECK(waves >= 1 && waves <= (kR > 1 || one ? 8 : kMaxWaves), "waves");
    CHECK(L.groups * tpw >= L.n_tiles, "columns without a wave");
    CHECK(!few || (B == 1 && !ops), "single-row form");
    // chunks and shares
    CHECK(L.kc % 4 == 0 && L.kc >= 4 && (int64_t)L.n_chunks * L.kc >= max_k, "units without a chunk");
    CHECK(!one || L.n_chunks == 1, "several chunks in the one-chunk form");
    CHECK(L.per * L.parts >= L.kc / 4 && L.per * (L.parts - 1) < L.kc / 4, "k-steps without a share");
    CHECK(L.xstride >= L.kc, "input panel");
    const size_t panel = (size_t)4 * L.kc * stride + (size_t)(one ? 8 : 4) * kR * kRows * L.xstride;
    CHECK(panel <= (one ? lds : stage), "panel");
    CHECK(one || L.win >= 1, "unit table");
    if (one) CHECK((L.kc + 63) / 64 * 64 <= kOneUnits, "unit table");
    else CHECK((int64_t)L.kc * (L.win - 1) + (L.kc + 63) / 64 * 64 <= L.k_alloc && 4 * (size_t)L.k_alloc <= lds,
               "unit table");
    // the support tile and the shares' sums
    const size_t tile = (size_t)kR * kRows * L.mpad * 4;
    const size_t sums = (size_t)(L.parts - 1) * L.groups * (few ? tpw : 4 * kR * tpw) * 512;
    CHECK(L.mpad >= g.out_mcu, "tile row");
    if (one) CHECK(tile + sums <= lds, "tile");
    else if (kR == 1) CHECK(tile / 2 + sums <= stage, "tile");
    else CHECK(tile / 2 <= stage && sums <= lds, "tile");
    const int64_t split = ops ? split_workgroups(g, L) : 0;
    CHECK(((int64_t)L.n_main + split) * 64 * waves < (int64_t)1 << 32, "2^32 work-items");
    // rows: every row tile in a workgroup
    CHECK(L.n_row_tiles == (B + kRows - 1) / kRows && L.n_row_groups * kR >= L.n_row_tiles &&
              (L.n_row_groups - 1) * kR < L.n_row_tiles && L.n_main == L.n_row_groups * g.out_hcu,
          "row tiles");
    CHECK(L.rw * waves >= kR * kRows, "input rows without a wave");
    // a wide hidden HCU's stages take what the launch has: shorter chunks end and drain more often
    if (!one && kR == 1 && L.n_chunks > 1)
        CHECK(panel + 4 * (4 * stride + 4 * kRows) + 512 > (pair ? 36 : 72) * 1024, "part of the LDS idle");
    // row tiles past the batch, which a group computes like the others
    CHECK(5 * L.n_row_groups * kR <= 8 * L.n_row_tiles || max_k <= kFewUnits, "matrix work of absent rows");
    // weights are not read again for every row tile of a batch that the L2s hold
    if (kR == 1 && (int64_t)B * g.n_in * 4 <= kL2Bytes) CHECK(!L.row_major, "order");
    if (pair) CHECK(2 * (2 * stage + 16 + lds) <= kLdsLimit && L.n_main > kCus, "two workgroups per CU");
}

int main() {
    const int mcus[] = {1, 2, 7, 10, 16, 17, 32, 64, 80, 81, 96, 97, 100, 112, 113, 128, 129, 160, 200, 255,
                        256, 257, 300, 400, 511, 512, 513, 700, 1000, 1023, 1024};
    const int units[] = {1, 3, 4, 12, 13, 63, 64, 65, 156, 200, 255, 256, 399, 400, 701, 1000, 1023, 1024,
                         1025, 2764, 3500, 3600, 4100, 8000, 12287, 12288};
    const int hcus[] = {1, 3, 13, 30, 100, 257, 520, 1100, 4096, 100000};
    const int rows[] = {1, 2, 16, 17, 32, 33, 48, 49, 64, 65, 80, 128, 144, 200, 512, 1000, 1024, 5000, 8192};
    for (int m : mcus)
        for (int k : units)
            for (int h : hcus)
                for (int b : rows)
                    for (int in_mcu : {1, 2, 3}) {
                        const int in_hcu = (k + in_mcu - 1) / in_mcu;
                        if (in_hcu * in_mcu > 12288 || (int64_t)h * m > 1 << 22) continue;
                        if ((int64_t)(b + 15) / 16 * h > 1 << 23) continue;
                        const Geometry g{in_hcu + 5, in_mcu, h, m, (int64_t)(in_hcu + 5) * in_mcu, (int64_t)h * m};
                        for (bool ops : {false, true}) check(g, b, in_hcu * in_mcu, ops);
                    }
    // the largest layers, and as many rows as a launch takes or a layer's training operands (96 bytes
    // per row and hidden unit) leave room for on the device
    for (int m : mcus)
        for (int k : {4, 156, 399, 12288})
            for (int h : {(1 << 22) / m, (1 << 21) / m, (1 << 16) / m}) {
                if (h < 1) continue;
                const Geometry g{k + 5, 1, h, m, k + 5, (int64_t)h * m};
                const int64_t most = most_rows(g);
                const int64_t layer = (int64_t)288e9 / 96 / g.n_out;
                for (int64_t b : {most, most - 15, most / 3}) {
                    if (b < 1) continue;
                    check(g, (int32_t)b, k, false);
                    const int64_t t = b < layer ? b : layer;
                    if (t > 0 && (t + 15) / 16 * h <= 1 << 23) check(g, (int32_t)t, k, true);
                }
            }
    printf("%d failures\n", failures);
    return failures != 0;
}
