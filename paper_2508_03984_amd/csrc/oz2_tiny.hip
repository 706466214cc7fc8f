// Algorithm 1 lines 6-12 in one launch for the smallest products: the INT8 GEMMs of all moduli, U_s and
// the accumulation.  A workgroup owns a 32 x 32 tile of C; its 16 wavefronts take the moduli in turn, load
// their operands straight from the residue slices (no LDS: nothing is shared between moduli), keep
// U_s in LDS for the accumulation and write it to the product buffer as the general form does.
//
// Bound: a launch, the way of the first operands, and then the loads of a compute unit, 64 Kp N bytes at
// about 64 bytes per clock.  tiny_product_applies (oz2_plan.hpp) draws the line and says what it measured.
#include "oz2_bytemod.hpp"
#include "oz2_convert.hpp"
#include "oz2_epilogue.hpp"
#include "oz2_kernels.hpp"
#include "oz2_tilemap.hpp"

namespace oz2 {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kTile = 32, kWaves = 16;
constexpr int kChunk = 128;              // elements of k loaded at a time: four MFMA K steps, 32 registers
constexpr int kFlight = 2;               // chunks on the way per wavefront

struct TinyMods {
    ByteMod byte_mod[kMaxModuli];
};

template <typename OutT>
__global__ __launch_bounds__(64 * kWaves) void k_tiny_product(const int8_t *__restrict__ A, const int8_t *__restrict__ B,
                                                                 uint8_t *__restrict__ U, int64_t Mp, int64_t Np,
                                                                 int64_t Kp, int64_t m, int64_t n,
                                                                 const int32_t *__restrict__ tA,
                                                                 const int32_t *__restrict__ tB, ModArgs ma, TinyMods tm,
                                                                 double alpha, double beta, OutT *C, int64_t ldc,
                                                                 int tiles_n, Divisor by_tiles_n, int tiles) {
    __shared__ v4i u_lds[kMaxModuli][kTile][kTile / 16];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5;
    // All of the arguments that the way to the first loads needs are requested before any branch: one wait for the
    // argument buffer instead of three (256^3 prepared, N = 14, other operands in
    // each call: 9.0 -> 8.7 us).
    asm volatile("" ::"s"(A), "s"(B), "s"(U), "s"(Mp), "s"(Np), "s"(Kp), "s"(m), "s"(tA), "s"(tB), "s"(ma.n), "s"(tiles_n),
                 "s"(by_tiles_n.mul), "s"(by_tiles_n.shift), "s"(tiles));
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
        uint8_t *const u = U + ((int64_t)row * kTile + (tid >> 4 & 31)) * Np + col;
        if (!right || col >= live)
            for (int s = tid >> 9; s < ma.n; s += 2) *reinterpret_cast<v4i *>(u + s * plane) = v4i{0, 0, 0, 0};
        return;
    }
    const int tile_r = divide((int)blockIdx.x, by_tiles_n), tile_c = (int)blockIdx.x - tile_r * tiles_n;
    const int64_t row0 = (int64_t)tile_r * kTile, col0 = (int64_t)tile_c * kTile;
    uint8_t *const u_out = U + (row0 + lrow) * Np + col0 + 16 * lhalf;

    // Chunk number c of this wavefront: modulus wave + 16 (c / chunks), elements 128 (c % chunks) ...
    const int chunks = (int)(Kp / kChunk), total = (ma.n - wave + kWaves - 1) / kWaves * chunks;
    const int8_t *pa = A + (row0 + lrow) * kBlockK + lhalf * 16, *pb = B + (col0 + lrow) * kBlockK + lhalf * 16;
    v4i fa[kFlight][4], fb[kFlight][4];
    auto load = [&](int buf, int c) {
        const int64_t s = wave + (int64_t)kWaves * (c / chunks), kb = 2 * (int64_t)(c % chunks);
        const int8_t *a = pa + (s * (Kp / kBlockK) + kb) * Mp * kBlockK, *b = pb + (s * (Kp / kBlockK) + kb) * Np * kBlockK;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            fa[buf][i] = *reinterpret_cast<const v4i *>(a + (i >> 1) * Mp * kBlockK + (i & 1) * 32);
            fb[buf][i] = *reinterpret_cast<const v4i *>(b + (i >> 1) * Np * kBlockK + (i & 1) * 32);
        }
    };
    if (total > 0) {
        // (indices beyond the last chunk load it again: no branch around a load)
#pragma unroll
        for (int b = 0; b < kFlight; ++b) load(b, b < total ? b : total - 1);
        v16i acc;
        int left = chunks, s = wave;                        // chunks left of the current modulus
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = (int)0x80000000;
        for (int c0 = 0; c0 < total; c0 += kFlight) {
            const bool more = c0 + kFlight < total;
#pragma unroll
            for (int b = 0; b < kFlight; ++b) {
                const int c = c0 + b;
                if (c >= total) break;
#pragma unroll
                for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[b][i], fa[b][i], acc, 0, 0, 0);
                if (more) load(b, c + kFlight < total ? c + kFlight : total - 1);
                if (--left == 0) {
                    // lane l holds row l % 32 and columns 8 g + 4 (l / 32) + {0..3} of the tile (as in GemmCore::store)
                    const ByteMod bm = tm.byte_mod[s];
                    uint32_t d[4];
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        d[g] = byte_mod_pack(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3], bm);
                    const auto s0 = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
                    const v4i q = v4i{(int)s0[0], (int)s0[1], (int)s1[0], (int)s1[1]};
                    u_lds[s][lrow][lhalf] = q;
                    *reinterpret_cast<v4i *>(u_out + s * plane) = q;
                    s += kWaves;
                    left = chunks;
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[r] = (int)0x80000000;
                }
            }
        }
    }
    // what the accumulation needs from memory travels meanwhile
    const int r = tid >> 5, c = tid & 31;
    const int64_t i = row0 + r, j = col0 + c;
    const int shift = (i < m ? tA[i] : 0) + (j < n ? tB[j] : 0);
    __syncthreads();

    // Accumulation: one entry per thread, moduli in ascending order.  Also in the lanes beyond C: FP64 instructions of a
    // wavefront with 16 lanes or fewer at work take longer (128 x 100 x 64, N = 15: 10.6 us with 4 columns' lanes alone
    // in the last tile, 7.3 us with all, as for 128 columns).
    if (row0 + 2 * wave >= m) return;                       // both rows of the wavefront
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
    const int tiles_m = (int)((m + kTile - 1) / kTile), tiles_n = (int)((n + kTile - 1) / kTile), tiles = tiles_m * tiles_n;
    const int64_t padding = (Mp / kTile - tiles_m) * (Np / kPadMN) + (Np > (int64_t)tiles_n * kTile ? tiles_m : 0);
    hipLaunchKernelGGL((k_tiny_product<OutT>), dim3((unsigned)(tiles + padding)), dim3(64 * kWaves), 0, stream, A, B, U, Mp, Np,
                       Kp, m, n, tA, tB, ma, tm, alpha, beta, C, ldc, tiles_n, make_divisor(tiles_n), tiles);
    return hipGetLastError();
}

#define OZ2_INSTANTIATE_TINY(T)                                                                                   \
    template hipError_t launch_tiny_product<T>(const int8_t *, const int8_t *, uint8_t *, int64_t, int64_t, int64_t, \
                                               int64_t, int64_t, const int32_t *, const int32_t *, const ModArgs &, \
                                               double, double, T *, int64_t, hipStream_t);
OZ2_INSTANTIATE_TINY(double)
OZ2_INSTANTIATE_TINY(float)

}  // namespace oz2
