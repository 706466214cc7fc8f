// Algorithm 1 lines 6-12 in one launch for the smallest products: the INT8 GEMMs of all moduli, U_s and
// the accumulation.  A workgroup owns a 16 x 16 or 32 x 32 tile of C; its 16 wavefronts take the moduli in turn, load
// their operands straight from the residue slices (no LDS: nothing is shared between moduli), keep
// U_s in LDS for the accumulation and write it to the product buffer as the general form does.
//
// Bound: a launch, the way of the first operands, and then the loads of a compute unit, 32 Kp N or 64 Kp N bytes at
// about 60 bytes per clock.  tiny_product_applies (oz2_plan.hpp) draws the line and says what it measured.
#include <algorithm>
#include <type_traits>

#include "oz2_bytemod.hpp"
#include "oz2_convert.hpp"
#include "oz2_epilogue.hpp"
#include "oz2_kernels.hpp"
#include "oz2_tilemap.hpp"

namespace oz2 {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kWaves = 16;
constexpr int kChunk = 128;              // elements of k loaded at a time: two MFMA K steps

struct TinyMods {
    ByteMod byte_mod[kMaxModuli];
};

template <typename OutT, int BLOCKS>
__global__ __launch_bounds__(64 * kWaves) void k_tiny_product(const int8_t *__restrict__ A, const int8_t *__restrict__ B,
                                                                 uint8_t *__restrict__ U, int64_t Mp, int64_t Np,
                                                                 int64_t Kp, int64_t m, int64_t n,
                                                                 const int32_t *__restrict__ tA,
                                                                 const int32_t *__restrict__ tB, ModArgs ma, TinyMods tm,
                                                                 double alpha, double beta, OutT *C, int64_t ldc,
                                                                 int tiles_n, Divisor by_tiles_n, int tiles, int tiles_short,
                                                                 Divisor by_short) {
    constexpr int kTile = 16 * BLOCKS;                        // BLOCKS x BLOCKS blocks of 16 x 16
    constexpr int kFlight = 4 / BLOCKS;                       // chunks on the way per wavefront: 16 loads
    __shared__ v4i u_lds[kMaxModuli][kTile][BLOCKS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 15, lquad = lane >> 4;
    // All of the arguments that the way to the first loads needs are requested before any branch: one wait for the
    // argument buffer instead of three (256^3 prepared, N = 14, other operands in
    // each call: 9.0 -> 8.7 us).
    asm volatile("" ::"s"(A), "s"(B), "s"(U), "s"(Mp), "s"(Np), "s"(Kp), "s"(m), "s"(tA), "s"(tB), "s"(ma.n), "s"(tiles_n),
                 "s"(by_short.mul), "s"(by_short.shift), "s"(tiles), "s"(tiles_short));
    const int64_t plane = Mp * Np;
    if ((int)blockIdx.x >= tiles) {
        // Padding of U, zero as from the products of zero residues: 32 rows of a block of 256 columns, all planes.  First
        // the last blocks of the rows of tiles (beside the tiles), then all blocks of the rows below.  (Tiles that clear what
        // lies beside them take longer: 1 x 1 x 64, N = 15, 9.6 us, this way 7.1; padding in 32 x 32 tiles writes partial
        // lines: 8000 x 1 x 64 50 us, this way 13.6.)
        const int id = (int)blockIdx.x - tiles, columns = (int)(Np / kPadMN), live = tiles_n * kTile;
        const int tiles_m = divide(tiles, by_tiles_n), beside = Np > live ? tiles_m : 0;
        const bool right = id < beside;
        const int row = right ? id : tiles_m + (id - beside) / columns, block = right ? columns - 1 : (id - beside) % columns;
        const int64_t col = (int64_t)block * kPadMN + (tid & 15) * 16;
        uint8_t *const u = U + ((int64_t)row * kTile + (tid >> 4) % kTile) * Np + col;
        if (!right || col >= live)
            for (int s = (tid >> 4) / kTile; s < ma.n; s += kWaves * 4 / kTile) *reinterpret_cast<v4i *>(u + s * plane) = v4i{0, 0, 0, 0};
        return;
    }
    // Ids are dealt to the 8 XCDs round-robin: each XCD gets consecutive tiles across the shorter side of C, so that a row of the
    // longer factor is fetched by one XCD (64 x 1000 x 256, N = 15: 14.7 us for the call, 18.2 with tiles along the longer side, 16.0
    // with neighbouring tiles on different XCDs).
    const int xcd = (int)blockIdx.x & 7, more = tiles & 7;
    const int id = xcd * (tiles >> 3) + (xcd < more ? xcd : more) + ((int)blockIdx.x >> 3);
    const int line = divide(id, by_short), at = id - line * tiles_short;
    const int tile_r = tiles_short == tiles_n ? line : at, tile_c = tiles_short == tiles_n ? at : line;
    const int64_t row0 = (int64_t)tile_r * kTile, col0 = (int64_t)tile_c * kTile;
    // Where this lane's 16 bytes (BLOCKS 1: 4 bytes) of a modulus go in the tile: see the exchange below
    const int u_row = BLOCKS == 2 ? 16 * (lquad >> 1) + lrow : lrow, u_col = BLOCKS == 2 ? 16 * (lquad & 1) : 4 * lquad;
    uint8_t *const u_out = U + (row0 + u_row) * Np + col0 + u_col;

    // Chunk number c of this wavefront: modulus wave + 16 (c / chunks), elements 128 (c % chunks) ...  Lane l holds
    // row l % 16 of a block of 16 rows and 16 consecutive k of the K block's 64, number l / 16.
    const int chunks = (int)(Kp / kChunk), total = (ma.n - wave + kWaves - 1) / kWaves * chunks;
    const int8_t *pa = A + (row0 + lrow) * kBlockK + lquad * 16, *pb = B + (col0 + lrow) * kBlockK + lquad * 16;
    v4i fa[kFlight][2][BLOCKS], fb[kFlight][2][BLOCKS];
    auto load = [&](int buf, int c) {
        const int64_t s = wave + (int64_t)kWaves * (c / chunks), kb = 2 * (int64_t)(c % chunks);
        const int8_t *a = pa + (s * (Kp / kBlockK) + kb) * Mp * kBlockK, *b = pb + (s * (Kp / kBlockK) + kb) * Np * kBlockK;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i) {
                fa[buf][h][i] = *reinterpret_cast<const v4i *>(a + (h * Mp + i * 16) * kBlockK);
                fb[buf][h][i] = *reinterpret_cast<const v4i *>(b + (h * Np + i * 16) * kBlockK);
            }
    };
    if (total > 0) {
        // (Chunks beyond the last one are not requested: the last one again in their place, to spare the branches, is what the loads
        // of a compute unit at k = 256 consisted of by half and at 128 by three quarters.  Graph of calls, other operands in each, us: 256^3
        // N = 14 12.9 -> 11.1, prepared 8.7 -> 7.0, 128^3 12.0 -> 9.5, 300 x 300 x 128 N = 15 prepared 9.7 -> 8.0.  Calls one after another from Python, whose pace
        // the host's work for two launches sets, are level: 256^3 11.8 -> 11.9.)
#pragma unroll
        for (int b = 0; b < kFlight; ++b)
            if (b < total) load(b, b);
        const v4i start = {(int)0x80000000, (int)0x80000000, (int)0x80000000, (int)0x80000000};
        v4i acc[BLOCKS][BLOCKS];
        int left = chunks, s = wave;                        // chunks left of the current modulus
        auto restart = [&] {
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
                for (int j = 0; j < BLOCKS; ++j) acc[i][j] = start;
        };
        restart();
        for (int c0 = 0; c0 < total; c0 += kFlight) {
#pragma unroll
            for (int b = 0; b < kFlight; ++b) {
                const int c = c0 + b;
                if (c >= total) break;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
                        for (int j = 0; j < BLOCKS; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[b][h][j], fa[b][h][i], acc[i][j], 0, 0, 0);
                if (c + kFlight < total) load(b, c + kFlight);
                if (--left == 0) {
                    // lane l holds row l % 16 and columns 4 (l / 16) + {0..3} of each block (as in GemmCore::store)
                    const ByteMod bm = tm.byte_mod[s];
                    uint32_t d[4];
#pragma unroll
                    for (int g = 0; g < BLOCKS * BLOCKS; ++g) {
                        const v4i &x = acc[g / BLOCKS][g % BLOCKS];
                        d[g] = byte_mod_pack(x[0], x[1], x[2], x[3], bm);
                    }
                    uint8_t *const u = reinterpret_cast<uint8_t *>(&u_lds[s][u_row][0]) + u_col;
                    if constexpr (BLOCKS == 2) {
                        const v4i q = exchange_quarters(d);
                        *reinterpret_cast<v4i *>(u) = q;
                        *reinterpret_cast<v4i *>(u_out + s * plane) = q;
                    } else {
                        *reinterpret_cast<uint32_t *>(u) = d[0];
                        *reinterpret_cast<uint32_t *>(u_out + s * plane) = d[0];
                    }
                    s += kWaves;
                    left = chunks;
                    restart();
                }
            }
        }
    }
    // what the accumulation needs from memory travels meanwhile
    const int r = tid / kTile, c = tid % kTile;             // (threads beyond the tile's entries: below)
    const int64_t i = row0 + r, j = col0 + c;
    const int shift = (r < kTile && i < m ? tA[i] : 0) + (j < n ? tB[j] : 0);
    __syncthreads();

    // Accumulation: one entry per thread, moduli in ascending order.  Also in the lanes beyond C: FP64 instructions of a
    // wavefront with 16 lanes or fewer at work take longer (128 x 100 x 64, N = 15: 10.6 us with 4 columns' lanes alone
    // in the last tile, 7.3 us with all, as for 128 columns).
    const int wave_row = wave * (64 / kTile);               // its first row
    if (wave_row >= kTile || row0 + wave_row >= m) return;
    const uint8_t *u = reinterpret_cast<const uint8_t *>(&u_lds[0][r][0]) + c;
    double C1 = 0.0, C2 = 0.0;
    for (int s0 = 0; s0 < ma.n; s0 += kModGroup) {          // the constants and bytes of a group requested together
        double s1[kModGroup], s2[kModGroup];
        int v[kModGroup];
#pragma unroll
        for (int g = 0; g < kModGroup; ++g) {
            s1[g] = ma.s1[s0 + g];
            s2[g] = ma.s2[s0 + g];
            v[g] = u[(s0 + g) * kTile * kTile];             // (beyond ma.n: not used)
        }
#pragma unroll
        for (int g = 0; g < kModGroup; ++g)
            if (s0 + g < ma.n) {
                C1 = fma(s1[g], (double)v[g], C1);
                C2 = fma(s2[g], (double)v[g], C2);
            }
    }
    if (i >= m || j >= n) return;
    OutT *dst = C + i * ldc + j;
    *dst = crt_entry<OutT>(C1, C2, shift, ma, alpha, beta, dst);
}

}  // namespace

template <typename OutT>
hipError_t launch_tiny_product(const int8_t *A, const int8_t *B, uint8_t *U, int64_t Mp, int64_t Np, int64_t Kp,
                               int64_t m, int64_t n, const int32_t *tA, const int32_t *tB, const ModArgs &ma,
                               double alpha, double beta, OutT *C, int64_t ldc, hipStream_t stream) {
    TinyMods tm{};
    for (int i = 0; i < ma.n; ++i) tm.byte_mod[i] = make_byte_mod(ma.p[i]);
    auto go = [&](auto blocks, const TinyGrid &g) {
        const int tiles_n = (int)g.tiles_n, tiles = (int)g.tiles(), tiles_short = (int)std::min(g.tiles_m, g.tiles_n);
        hipLaunchKernelGGL((k_tiny_product<OutT, decltype(blocks)::value>), dim3((unsigned)(tiles + g.padding)), dim3(64 * kWaves), 0,
                           stream, A, B, U, Mp, Np, Kp, m, n, tA, tB, ma, tm, alpha, beta, C, ldc, tiles_n, make_divisor(tiles_n),
                           tiles, tiles_short, make_divisor(tiles_short));
        return hipGetLastError();
    };
    // Tiles of 16 x 16 where these and the padding have a compute unit each: four times as many units fetch operands and
    // accumulate (repeated in a graph, other operands in each call, us, 32 x 32 | 16 x 16: 256^3 N = 14 12.8 | 11.9, prepared 8.0 | 7.1; 200^3
    // N = 15 13.5 | 12.9, 8.2 | 7.3; 128^3 N = 14 11.6 | 10.7, 7.7 | 6.9; 256 x 256 x 512 FP32 N = 6 11.4 | 9.7, 6.8 | 5.1).
    if (tiny_small_tiles(m, n)) return go(std::integral_constant<int, 1>{}, tiny_grid(m, n, 16));
    return go(std::integral_constant<int, 2>{}, tiny_grid(m, n, 32));
}

#define OZ2_INSTANTIATE_TINY(T)                                                                                   \
    template hipError_t launch_tiny_product<T>(const int8_t *, const int8_t *, uint8_t *, int64_t, int64_t, int64_t, \
                                               int64_t, int64_t, const int32_t *, const int32_t *, const ModArgs &, \
                                               double, double, T *, int64_t, hipStream_t);
OZ2_INSTANTIATE_TINY(double)
OZ2_INSTANTIATE_TINY(float)

}  // namespace oz2
