// Which output tile of a GEMM launch a workgroup works on.  Plain C++, so that the CPU can check that every
// launch covers every tile once.
#pragma once
#if defined(__HIPCC__)
#define OZ2_HOST_DEVICE __host__ __device__
#else
#define OZ2_HOST_DEVICE
#endif

namespace oz2 {

// Workgroup ids are handed to the 8 XCDs round-robin, and 256 workgroups run at a time (one per CU):
// XCD x runs the ids = x (mod 8), 32 at a time.  Those 32 are given 32 consecutive positions of a walk over
// the tiles that covers about 8 x 4 tiles with them, whatever the numbers of tiles, so that an A tile row is fetched
// into that XCD's L2 once for 4 workgroups and a B tile row once for 8.  The walk goes through a slice in
// bands of about 8 tile rows, two bands at a time, 4 columns of the upper and then of the lower one, so that the
// 256 tiles of a round are about 16 x 16 (16384^3: bands one at a time, 8 x 32 tiles, measured 1.7 % slower).  Numbers of
// tiles that are multiples of 16 have the same blocks without the divisions, dealt so that the upper and the lower half
// of a region belong to four XCDs each (0.4 to 0.6 % faster at 16384^3 and 8192 x 8192 x 512).
// Against ids in row-major order, where e.g. 8 tile columns put 4 slices with 8 A tile rows each and one B tile
// row on an XCD (36 panels for its 32 tiles instead of 12): 1024^3 N = 15 47.7 -> 40.4 us, 1500 x 1111 x 3001 N = 16
// 180 -> 152 us, 2048^3 FP32 N = 7 99 -> 91 us, 1536 x 1000 x 40000 1670 -> 1643 us.
struct TileMap {
    int tiles_m, tiles_n;      // tiles per slice
    int total;                 // tiles in the launch
    int regions_n;             // columns / 16 if both numbers are multiples of 16, else 0
    int bands, band_rows, wide_bands;   // band_rows + 1 tile rows in the first wide_bands bands, band_rows in the others
};

inline TileMap make_tile_map(int tiles_m, int tiles_n, int total) {
    const int bands = (tiles_m + 7) / 8;
    return TileMap{tiles_m, tiles_n, total, tiles_m % 16 == 0 && tiles_n % 16 == 0 ? tiles_n / 16 : 0, bands, tiles_m / bands, tiles_m % bands};
}

OZ2_HOST_DEVICE inline void map_tile(const TileMap &tm, int id, int &s, int &tr, int &tc) {
    const int xcd = id & 7, local = id >> 3, round0 = id & ~255;
    if (tm.regions_n) {
        const int j = local & 31, region = id >> 8, regions = (tm.tiles_m >> 4) * tm.regions_n;
        s = region / regions;
        const int r = region - s * regions;
        tr = r / tm.regions_n * 16 + (xcd >> 2) * 8 + (j >> 2);
        tc = r % tm.regions_n * 16 + (xcd & 3) * 4 + (j & 3);
        return;
    }
    const int left = tm.total - round0;                    // tiles from this round on; a last round is dealt evenly
    const int each = left < 256 ? left >> 3 : 32, more = left < 256 ? left & 7 : 0;
    const int pos = round0 + xcd * each + (xcd < more ? xcd : more) + (local & 31);
    const int per = tm.tiles_m * tm.tiles_n;
    s = pos / per;
    int w = pos - s * per;
    // the pair of bands: its rows take the positions [first row, last row] * tiles_n
    const int wide_rows = tm.wide_bands * (tm.band_rows + 1), v = w / tm.tiles_n;
    const int band = (v < wide_rows ? v / (tm.band_rows + 1) : tm.wide_bands + (v - wide_rows) / tm.band_rows) & ~1;
    const int row0 = band * tm.band_rows + (band < tm.wide_bands ? band : tm.wide_bands);
    const int upper = tm.band_rows + (band < tm.wide_bands ? 1 : 0);
    const int lower = band + 1 < tm.bands ? tm.band_rows + (band + 1 < tm.wide_bands ? 1 : 0) : 0;
    w -= row0 * tm.tiles_n;
    const int group = w / (4 * (upper + lower)), col0 = 4 * group;
    const int cols = tm.tiles_n - col0 < 4 ? tm.tiles_n - col0 : 4;
    w -= group * 4 * (upper + lower);
    const bool low = w >= upper * cols;
    if (low) w -= upper * cols;
    const int row = w / cols;                              // 4 neighbours share an A tile row
    tr = row0 + (low ? upper : 0) + row;
    tc = col0 + w - row * cols;
}

}  // namespace oz2
