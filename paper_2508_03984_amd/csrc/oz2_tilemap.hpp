// Which output tile of a GEMM launch a workgroup works on.  Plain C++, so that the CPU can check that every
// launch covers every tile once.
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define OZ2_HOST_DEVICE __host__ __device__
#else
#define OZ2_HOST_DEVICE
#endif

namespace oz2 {

// x / d for 0 <= x < 2^31 by one multiplication.  mul = 2^(31 + s) / d + e with 2^s >= d and 0 < e <= 1, so that the product
// is off by less than x 2^-(31 + s) < 1 / d.
struct Divisor {
    uint32_t mul, shift;
};
inline Divisor make_divisor(int d) {
    uint32_t s = 0;
    while (((int64_t)1 << s) < d) ++s;
    return Divisor{(uint32_t)(((uint64_t)1 << (31 + s)) / (uint64_t)d + 1), 31 + s};
}
OZ2_HOST_DEVICE inline int divide(int x, Divisor d) { return (int)((uint64_t)(uint32_t)x * d.mul >> d.shift); }

// Workgroup ids are handed to the 8 XCDs round-robin, and 256 workgroups run at a time (one per CU):
// XCD x runs the ids = x (mod 8), 32 at a time.  Those 32 are given 32 consecutive positions of a walk over
// the tiles that covers about 8 x 4 tiles with them, whatever the numbers of tiles, so that an A tile row is fetched
// into that XCD's L2 once for 4 workgroups and a B tile row once for 8.  The walk goes through a slice in
// bands of about 8 tile rows, two bands at a time, 4 columns of the upper and then of the lower one, so that the
// 256 tiles of a round are about 16 x 16 (16384^3: bands one at a time, 8 x 32 tiles, measured 1.7 % slower).  Numbers of
// tiles that are multiples of 16 have the same blocks more simply, dealt so that the upper and the lower half
// of a region belong to four XCDs each (0.4 to 0.6 % faster at 16384^3 and 8192 x 8192 x 512).
// Against ids in row-major order, where e.g. 8 tile columns put 4 slices with 8 A tile rows each and one B tile
// row on an XCD (36 panels for its 32 tiles instead of 12), whole calls repeated in a graph, with 32x32x32 MFMAs, us: 1024^3 N = 15 44.7 -> 42.3,
// 1500 x 1111 x 3001 (A transposed) N = 16 160.5 -> 133.1, 2048^3 FP32 N = 7 97.1 -> 90.4, 1536 x 1000 x 40000 N = 18
// 1665 -> 1643, 5000 x 5000 x 512 N = 15 417 -> 400.
//
// The places are worked out before a workgroup's first loads, so their divisions are multiplications (prepared
// operands, us, tiles in row-major order | this order by integer divisions | by multiplications: 512 x 512 x 1024 FP32
// N = 8 10.75 | 11.1 | 10.95; 64 x 64 x 1024 N = 15 10.25 | 10.5 | 10.37; 2048 x 2048 x 512 N = 15 78.4 | 67.6 | 65.7).
struct TileMap {
    int tiles_m, tiles_n;      // tiles per slice
    int total;                 // tiles in the launch
    int regions_n;             // columns / 16 if both numbers are multiples of 16, else 0
    int bands, band_rows, wide_bands;   // band_rows + 1 tile rows in the first wide_bands bands, band_rows in the others
    Divisor per_slice;         // tiles (regions) of a slice
    Divisor row;               // tiles (regions) of a row
    Divisor narrow, wide;      // band_rows, band_rows + 1
    Divisor group[4];          // tiles of 4 columns of a pair of bands: 2, 1 or no wide ones, the last band alone
};

inline TileMap make_tile_map(int tiles_m, int tiles_n, int total) {
    const int bands = (tiles_m + 7) / 8, rows = tiles_m / bands;
    const bool regions = tiles_m % 16 == 0 && tiles_n % 16 == 0;
    TileMap t{};
    t.tiles_m = tiles_m; t.tiles_n = tiles_n; t.total = total;
    t.regions_n = regions ? tiles_n / 16 : 0;
    t.bands = bands; t.band_rows = rows; t.wide_bands = tiles_m % bands;
    t.per_slice = make_divisor(regions ? tiles_m / 16 * t.regions_n : tiles_m * tiles_n);
    t.row = make_divisor(regions ? t.regions_n : tiles_n);
    t.narrow = make_divisor(rows); t.wide = make_divisor(rows + 1);
    t.group[0] = make_divisor(4 * (2 * rows + 2)); t.group[1] = make_divisor(4 * (2 * rows + 1));
    t.group[2] = make_divisor(4 * 2 * rows); t.group[3] = make_divisor(4 * rows);
    return t;
}

OZ2_HOST_DEVICE inline void map_tile(const TileMap &tm, int id, int &s, int &tr, int &tc) {
    const int xcd = id & 7, local = id >> 3, round0 = id & ~255;
    if (tm.regions_n) {
        const int j = local & 31, region = id >> 8, regions = (tm.tiles_m >> 4) * tm.regions_n;
        s = divide(region, tm.per_slice);
        const int r = region - s * regions, r_row = divide(r, tm.row);
        tr = r_row * 16 + (xcd >> 2) * 8 + (j >> 2);
        tc = (r - r_row * tm.regions_n) * 16 + (xcd & 3) * 4 + (j & 3);
        return;
    }
    const int left = tm.total - round0;                    // tiles from this round on; a last round is dealt evenly
    const int each = left < 256 ? left >> 3 : 32, more = left < 256 ? left & 7 : 0;
    const int pos = round0 + xcd * each + (xcd < more ? xcd : more) + (local & 31);
    s = divide(pos, tm.per_slice);
    int w = pos - s * (tm.tiles_m * tm.tiles_n);
    // the pair of bands: its rows take the positions [first row, last row] * tiles_n
    const int wide_rows = tm.wide_bands * (tm.band_rows + 1), v = divide(w, tm.row);
    const int band = (v < wide_rows ? divide(v, tm.wide) : tm.wide_bands + divide(v - wide_rows, tm.narrow)) & ~1;
    const int row0 = band * tm.band_rows + (band < tm.wide_bands ? band : tm.wide_bands);
    const int upper = tm.band_rows + (band < tm.wide_bands ? 1 : 0);
    const int lower = band + 1 < tm.bands ? tm.band_rows + (band + 1 < tm.wide_bands ? 1 : 0) : 0;
    w -= row0 * tm.tiles_n;
    // (the last band is never a wide one)
    const Divisor by_group = band + 1 >= tm.bands ? tm.group[3] : band + 1 < tm.wide_bands ? tm.group[0]
                                                  : band < tm.wide_bands ? tm.group[1] : tm.group[2];
    const int group = divide(w, by_group), col0 = 4 * group;
    const int cols = tm.tiles_n - col0 < 4 ? tm.tiles_n - col0 : 4;
    w -= group * 4 * (upper + lower);
    const bool low = w >= upper * cols;
    if (low) w -= upper * cols;
    const int row = cols == 3 ? (w * 43691) >> 17 : w >> (cols >> 1);   // w / cols, w < 32; 4 neighbours share an A tile row
    tr = row0 + (low ? upper : 0) + row;
    tc = col0 + w - row * cols;
}

// The work of a launch with one workgroup per tile: the tiles of all slices, each slice once per K range (a `slice` of the map is
// (range, slice), the slices of a range together).  Tiles of 128 x 128 that hold nothing but padding are not among them: they are
// cleared by workgroups of their own, which come last.
struct GemmGrid {
    TileMap map;
    int batch;                 // slices
    Divisor by_batch;
    int k_each, k_more;        // K tiles of a range: k_each, two more in the first k_more ranges
    int padding;               // tiles to clear
    int pad_right, pad_below;  // of a slice: at the right of the rows of tiles; below them
};

struct GemmItem {
    int plane, s;              // where the results go (range * batch + slice); the slice
    int tr, tc;                // tile row and column
    int kb, kt;                // first K tile of the range and how many
};

// rows x cols entries of C, of which valid_rows x valid_cols exist, in tiles of `tile`; rows and cols are multiples of 256 that exceed the
// valid ones by less than 256.  ranges: K ranges of kt_all K tiles in all, an even number in each.
inline GemmGrid make_gemm_grid(int64_t rows, int64_t cols, int64_t valid_rows, int64_t valid_cols, int tile, int batch, int ranges,
                               int kt_all) {
    GemmGrid g{};
    const int tiles_m = (int)((valid_rows + tile - 1) / tile), tiles_n = (int)((valid_cols + tile - 1) / tile);
    g.pad_right = cols / tile > tiles_n ? tiles_m : 0;
    g.pad_below = rows / tile > tiles_m ? (int)(cols / tile) : 0;
    g.padding = (g.pad_right + g.pad_below) * batch;
    g.map = make_tile_map(tiles_m, tiles_n, tiles_m * tiles_n * batch * ranges);
    g.batch = batch;
    g.by_batch = make_divisor(batch);
    g.k_each = kt_all / 2 / ranges * 2; g.k_more = kt_all / 2 % ranges;
    return g;
}

OZ2_HOST_DEVICE inline GemmItem map_item(const GemmGrid &g, int id) {
    GemmItem it;
    map_tile(g.map, id, it.plane, it.tr, it.tc);
    const int range = divide(it.plane, g.by_batch);
    it.s = it.plane - range * g.batch;
    it.kt = g.k_each + (range < g.k_more ? 2 : 0);
    it.kb = range * g.k_each + 2 * (range < g.k_more ? range : g.k_more);
    return it;
}

// Number j of the tiles to clear.
OZ2_HOST_DEVICE inline GemmItem padding_item(const GemmGrid &g, int j) {
    const int each = g.pad_right + g.pad_below, s = j / each, i = j - s * each;
    return i < g.pad_right ? GemmItem{s, s, i, g.map.tiles_n, 0, 0} : GemmItem{s, s, g.map.tiles_m, i - g.pad_right, 0, 0};
}

}  // namespace oz2
