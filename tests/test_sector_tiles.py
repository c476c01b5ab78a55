"""The tiles of csrc/sectors.h: of a row of any length and phase every column is stored, once, with its own value, and nothing
outside the row.  Tile bounds, loads and stores are plain functions of the tile and the lane, run here on the host; the shift
along the lanes, a DPP move on the GPU, is a move within an array."""
import subprocess


PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "sectors.h"
using namespace approxifer;

constexpr int kGuard = 64;                                       // floats on both sides of the row, a multiple of a sector
static std::vector<float> query;                                 // query[d] = d + 1
static float *memory;                                            // 64-byte aligned
static std::vector<int> stores;

static int check(int64_t D, int phase, int halo) {
    const SectorTiles tiles = sector_tiles(3, D, halo);
    if (tiles.total != 3 * tiles.per_row || tiles.width % 4 != 0) return 1;
    float *base = memory + kGuard + phase;
    stores.assign(D, 0);
    for (int64_t k = 0; k < tiles.per_row; ++k) {
        const RowTile t = row_tile(static_cast<uint32_t>(k), static_cast<uint32_t>(tiles.per_row), tiles.width, halo, D);
        if (t.g != 0 || t.start < 0 || t.left < 1) return 2;
        float held[256];
        for (int lane = 0; lane < 64; ++lane) {
            const int c = t.column(lane);
            const int64_t at = load_column(t, c, D);
            if (at < 0 || at + 4 > D) return 3;
            v4f x = v4f{query[at], query[at + 1], query[at + 2], query[at + 3]};
            if (t.last && D % 4 != 0) x = finish_vector(x, over_the_end(t, c), static_cast<int>(D % 4));
            for (int e = 0; e < 4; ++e) held[4 * lane + e] = x[e];
        }
        float *row = base + t.start;
        const int at = static_cast<int>(reinterpret_cast<uintptr_t>(row) / sizeof(float)) & (kSector - 1);
        const int s = at & 3;
        for (int lane = 0; lane < 64; ++lane) {
            v4f v;
            for (int e = 0; e < 4; ++e) v[e] = 4 * lane + e >= s ? held[4 * lane + e - s] : 0.0f;
            store_lane(row, v, t.column(lane) - s, at, t);
        }
        for (int64_t d = t.start - 32; d < t.start + 256 + 32; ++d) {
            if (d < -kGuard || d >= D + kGuard || base[d] == -1.0f) continue;
            if (d < 0 || d >= D) return 4;
            if (base[d] != query[d]) return 5;
            base[d] = -1.0f;
            ++stores[d];
        }
    }
    for (int64_t d = 0; d < D; ++d)
        if (stores[d] != 1) return 6;
    for (int64_t i = 0; i < 2 * kGuard + 16 + D; ++i)            // no store far from its tile either
        if (memory[i] != -1.0f) return 7;
    return 0;
}

int main() {
    constexpr int64_t kMost = 300100;
    for (int64_t d = 0; d < kMost; ++d) query.push_back(static_cast<float>(d + 1));
    memory = static_cast<float *>(aligned_alloc(64, sizeof(float) * (kMost + 2 * kGuard + 64)));
    for (int64_t i = 0; i < kMost + 2 * kGuard + 64; ++i) memory[i] = -1.0f;
    std::vector<int64_t> lengths;
    for (int64_t d = 17; d <= 2200; ++d) lengths.push_back(d);
    for (int64_t d = 2400; d <= 24000; d += 240)                 // a tile's own columns, and what the rounding up makes of them
        for (int64_t e = -5; e <= 5; ++e) lengths.push_back(d + e);
    for (int64_t d : {47999, 48000, 57599, 57600, 131039, 150528, 268203, 268319, 280000, 299998, 299999, 300000})
        lengths.push_back(d);
    for (int64_t d = 14161; d < 30000; d += 97) lengths.push_back(d);
    for (int64_t d : lengths) {
        for (int phase = 0; phase < 16; ++phase)
            if (int rc = check(d, phase, kTileHalo)) { printf("length %ld phase %d: %d\n", static_cast<long>(d), phase, rc); return 1; }
        if (d % kSector == 0)
            if (int rc = check(d, 0, 0)) { printf("length %ld, whole sectors: %d\n", static_cast<long>(d), rc); return 1; }
    }
    printf("ok\n");
    return 0;
}
"""


def test_tiles_store_every_column_of_a_row_once_and_nothing_else(tmp_path):
    from paper_2109_09868_amd import build
    src = tmp_path / "tiles.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "tiles"
    subprocess.run([build.hipcc_path(), "--offload-host-only", "-O2", "-std=c++17", "-I", build.CSRC, "-I", build.ROOT + "/include",
                    str(src), "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
