// Tiles of 64 vectors (256 floats) of a row whose stores are whole 64-byte sectors, whatever the row's length and address.
#pragma once

#include "common.h"

namespace approxifer {

// ---- rows that do not begin on a 64-byte sector -------------------------------------------------------------------
// A wave whose row segment begins or ends inside a sector writes that sector in part, and its neighbour the rest: the
// memory pays for both as for two.  Where rows are not whole sectors (D % 16 != 0, or a base address that is none) a tile
// therefore writes, of every coded row, the whole sectors that end inside it (tile [start, start + width) writes from the
// sector of column `start` up to the one of column start + width), and loads sixteen columns more on its left for that.
// Lane l of a wave holds columns start - 16 + 4 l .. + 3; a coded row whose phase is not a multiple of four floats is
// shifted along the lanes first, so that every store is one aligned 16-byte piece.  Only a row's own first and last
// sector are written in part, in single floats.  Rows that are whole sectors go by the same tiles without the columns on
// the left.
constexpr int kSector = 16;                               // floats
constexpr int kTileHalo = 4;                              // lanes on the left that a tile shares with its neighbour; the row's
                                                          // last tile leaves one more for what the shift pushes past its end

struct RowTile {
    int64_t g;                                            // group
    int64_t start;                                        // first column, a multiple of four
    int width;                                            // columns of a tile that is not the row's last
    int left;                                             // last tile: columns up to the row's end
    int halo;
    bool first, last;
    // first column of the tile's vector v, relative to start: the row's first tile has no neighbour on the left
    __host__ __device__ __forceinline__ int column(int v) const { return 4 * v - (first ? 0 : 4 * halo); }
};
// tile k of group g's rows, `per_row` tiles to a row; halo: kTileHalo, or 0 where every row is whole sectors
__host__ __device__ __forceinline__ RowTile row_tile(uint32_t g, uint32_t k, uint32_t per_row, int width, int halo, int64_t D) {
    RowTile t;
    t.g = g;
    t.start = static_cast<int64_t>(k) * width;
    t.width = width;
    t.halo = halo;
    t.first = k == 0;
    t.last = k + 1 == per_row;
    t.left = t.last ? static_cast<int>(D - t.start) : width;
    return t;
}
// tile `id` of the batch
__host__ __device__ __forceinline__ RowTile row_tile(uint32_t id, uint32_t per_row, int width, int halo, int64_t D) {
    const uint32_t g = id / per_row;
    return row_tile(g, id - g * per_row, per_row, width, halo, D);
}
// Where lane-vector c (relative to the tile's start) of a query row is loaded from: always inside the row.  The vector over
// the row's end is loaded from its last four columns; finish_vector() then moves its columns to their places.
__host__ __device__ __forceinline__ int64_t load_column(const RowTile &t, int c, int64_t D) {
    const int64_t col = t.start + c;
    if (col < 0) return 0;
    return col + 4 <= D ? col : D - 4;
}
__host__ __device__ __forceinline__ bool over_the_end(const RowTile &t, int c) { return t.last && c < t.left && c + 4 > t.left; }
__host__ __device__ __forceinline__ v4f finish_vector(v4f x, bool over, int tail) {          // tail = D % 4, not 0
    v4f y = x;
    y[0] = tail == 1 ? x[3] : (tail == 2 ? x[2] : x[1]);
    y[1] = tail == 2 ? x[3] : x[2];
    y[2] = x[3];
    return over ? y : x;
}
__device__ __forceinline__ float from_lane_below(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kDppWaveShr1, 0xF, 0xF, true));
}
// Stores what a lane's vector v holds of one coded row of the tile: columns q .. q + 3 relative to the tile's start, row = address
// of column `start`, `at` = floats by which that lies behind a sector's begin, (at + q) % 4 = 0.
__host__ __device__ __forceinline__ void store_lane(float *row, v4f v, int q, int at, const RowTile &t) {
    const int lo = t.first ? 0 : -at;
    const int hi = t.last ? t.left - 3 : t.width - ((at + t.width) & (kSector - 1));
    if (q >= lo && q < hi) __builtin_nontemporal_store(v, reinterpret_cast<v4f *>(row + q));
    if (t.first || t.last) {
        const bool part = (t.first && q < 0 && q > -4) || (t.last && q < t.left && q + 4 > t.left);
        if (part) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (q + e >= lo && (!t.last || q + e < t.left)) __builtin_nontemporal_store(v[e], row + q + e);
        }
    }
}
// One coded row of the tile: v holds the lane's columns c .. c + 3 (c = 4 lane - 16, relative to the tile's start), `at` and row
// as above, the same for all lanes.  Every lane of the wave calls it.
__device__ __forceinline__ void store_sectors(float *row, v4f v, int c, int at, const RowTile &t) {
    const int s = at & 3;
    if (s & 2) {
        const float p2 = from_lane_below(v[2]), p3 = from_lane_below(v[3]);
        v = v4f{p2, p3, v[0], v[1]};
    }
    if (s & 1) {
        const float p3 = from_lane_below(v[3]);
        v = v4f{p3, v[0], v[1], v[2]};
    }
    store_lane(row, v, c - s, at, t);
}

// Tiles of a row: as few as it takes, all of one width.  With columns on the left the last one always leaves its last lane for
// what the shift pushes past the row's end (own vectors + halo + 1 <= 64; a row of one tile has no halo).
struct SectorTiles {
    int64_t per_row, total;
    int width;                              // columns, a multiple of four
};
inline SectorTiles sector_tiles(int64_t G, int64_t D, int halo) {
    const int64_t vecs = (D + 3) / 4;
    const int64_t own = 64 - halo, spill = halo > 0 ? 1 : 0;   // see row_tile
    int64_t per_row = vecs + spill <= 64 ? 1 : (vecs + spill + own - 1) / own;
    int64_t width = (vecs + per_row - 1) / per_row;
    if (halo == 0) width = (width + 7) / 8 * 8;               // whole lines, and with no neighbour's help whole sectors at least
    per_row = (vecs + width - 1) / width;
    if (per_row > 1 && vecs - (per_row - 1) * width > own - spill) {   // rounded up to full tiles, the last one among them
        --width;
        per_row = (vecs + width - 1) / width;
    }
    SectorTiles t;
    t.per_row = per_row;
    t.width = static_cast<int>(4 * width);
    t.total = G * per_row;
    return t;
}
inline bool whole_sectors(const void *p, int64_t D) { return reinterpret_cast<uintptr_t>(p) % (4 * kSector) == 0 && D % kSector == 0; }

}  // namespace approxifer
