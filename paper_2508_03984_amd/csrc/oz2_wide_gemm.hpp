// The INT8 GEMM of oz2_wide_gemm.hip, which launch_int8_gemm takes where it applies.
#pragma once
#include "oz2_bytemod.hpp"
#include "oz2_kernels.hpp"
#include "oz2_tilemap.hpp"

namespace oz2 {

struct WideMods {
    int32_t p[kMaxModuli];
    ByteMod byte_mod[kMaxModuli];          // of sums that start at -2^30: make_byte_mod(p, kWideFirst)
};
constexpr uint32_t kWideFirst = 0xc0000000u;

// grid: tiles of 256 x 256, every item with an even number of K tiles, at least kWideMinKTiles, launches of at most kWideMaxK
// elements of k.  The other arguments as the kernels of oz2_int8_gemm.hip take them; units: workgroups at most, a multiple of 8.
hipError_t launch_wide_gemm(const int8_t *A, const int8_t *B, uint8_t *C, int64_t Mp, int64_t Np, int64_t KB, int kb0, int64_t c_ld,
                            int64_t c_plane, const GemmGrid &grid, const WideMods &mods, bool fold, int units, hipStream_t stream);

}  // namespace oz2
