// Residues of both factors in one launch for SMALL problems whose shifts are known (accurate mode,
// after its product Cbar): the row-form and column-form workgroups of the general kernels, dealt to the
// two factors by workgroup index.  Below about 2048^3 a launch less is worth more than anything the
// separate launches could do better.
#include <algorithm>

#include "oz2_convert.hpp"
#include "oz2_kernels.hpp"

namespace oz2 {
namespace {

using namespace dev;

// One factor: `vecs` vectors of `len` elements; element h of vector v is X[v * ld + h] (k_contiguous)
// or X[h * ld + v].
template <typename T>
struct SmallSide {
    const T *X;
    int64_t ld, vecs, len;
    const int32_t *t;           // [vecs] shifts
    int8_t *out;                // residue slices [N][len_pad/64][vecs_pad][64]
    int64_t vecs_pad, len_pad;
    int k_contiguous;
    unsigned blocks;            // workgroups of this side in the launch at hand
};

#ifndef OZ2_SPLIT_MODULI_BELOW
#define OZ2_SPLIT_MODULI_BELOW 600
#endif
constexpr unsigned kSplitModuliBelow = OZ2_SPLIT_MODULI_BELOW;   // residue launches with fewer workgroups split the moduli

// gridDim.y > 1: workgroup row y produces the moduli of group y only (groups of kModGroup), so
// that the smallest problems, whose few workgroups would each walk through all N moduli one after
// the other, fill more of the chip; the operand is then read once per group, from the caches.
// COLUMNS: one of the factors has strided vectors.  Two factors of rows have a kernel of their own, without the registers and
// the LDS of the column form (1552 x 1520 x 1061, N = 15, us: 15.7 with them, 14.3 without).  7 workgroups per compute unit, as many as LDS
// has room for, are 72 registers in FP64 instead of 86 (2048^3 N = 15 37.8 -> 35.8 us; 256^3 N = 14 5.2 -> 5.5).
template <typename T, int ROUNDS, bool COLUMNS>
__global__ __launch_bounds__(256, 7) void k_small_residues(SmallSide<T> a, SmallSide<T> b, ModArgs ma) {
    const bool first = blockIdx.x < a.blocks;
    const SmallSide<T> s = first ? a : b;
    const int64_t blk = first ? blockIdx.x : blockIdx.x - a.blocks;
    const int g_lo = gridDim.y > 1 ? (int)blockIdx.y : 0, g_hi = gridDim.y > 1 ? (int)blockIdx.y + 1 : 1 << 30;
    if (!COLUMNS || s.k_contiguous) {
        residues_block<T, ROUNDS, 0>(blk, s.X, s.ld, s.vecs, s.len, s.t, ma, s.out, s.vecs_pad, s.len_pad,
                                     s.vecs_pad, g_lo, g_hi);
    } else if constexpr (COLUMNS) {
        const int64_t strips = s.vecs_pad / kColStrip;
        residues_cols_block<T, ROUNDS, 0, 256, false>(blk % strips, blk / strips, s.X, s.ld, s.len, s.vecs, s.t, ma, s.out,
                                          s.vecs_pad, s.len_pad, s.vecs_pad, g_lo, g_hi);
    }
}

template <typename T>
SmallSide<T> side_of(const T *X, int64_t ld, bool k_contiguous, int64_t vecs, int64_t len, const int32_t *t,
                     int8_t *out, int64_t vecs_pad, int64_t len_pad) {
    return SmallSide<T>{X, ld, vecs, len, t, out, vecs_pad, len_pad, k_contiguous ? 1 : 0, 0u};
}

template <typename T>
unsigned residue_blocks(const SmallSide<T> &s) {
    return (unsigned)(s.k_contiguous ? (s.vecs_pad * (s.len_pad / kResPerThread) + 255) / 256
                                     : (s.vecs_pad / kColStrip) * (s.len_pad / kBlockK));
}

}  // namespace

template <typename T>
hipError_t launch_small_residues(const T *A, int64_t lda, bool a_k_contiguous, const T *B, int64_t ldb,
                                 bool b_k_contiguous, int64_t m, int64_t n, int64_t k, const ModArgs &ma,
                                 const int32_t *tA, const int32_t *tB, int8_t *rA, int8_t *rB, int64_t Mp,
                                 int64_t Np, int64_t Kp, hipStream_t stream) {
    SmallSide<T> a = side_of<T>(A, lda, a_k_contiguous, m, k, tA, rA, Mp, Kp);
    SmallSide<T> b = side_of<T>(B, ldb, b_k_contiguous, n, k, tB, rB, Np, Kp);
    a.blocks = residue_blocks(a);
    b.blocks = residue_blocks(b);
    // few workgroups: one row of workgroups per group of moduli (see k_small_residues)
    const unsigned groups = (unsigned)((ma.n + kModGroup - 1) / kModGroup);
    const unsigned rows = (a.blocks + b.blocks) < kSplitModuliBelow ? groups : 1u;
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(a.blocks + b.blocks, rows), dim3(256), 0, stream, a, b, ma); };
    if (a.k_contiguous && b.k_contiguous) ma.rounds == 1 ? go(k_small_residues<T, 1, false>) : go(k_small_residues<T, 2, false>);
    else ma.rounds == 1 ? go(k_small_residues<T, 1, true>) : go(k_small_residues<T, 2, true>);
    return hipGetLastError();
}

#define OZ2_INSTANTIATE_SMALL(T)                                                                        \
    template hipError_t launch_small_residues<T>(const T *, int64_t, bool, const T *, int64_t, bool,    \
                                                 int64_t, int64_t, int64_t, const ModArgs &,            \
                                                 const int32_t *, const int32_t *, int8_t *, int8_t *,  \
                                                 int64_t, int64_t, int64_t, hipStream_t);
OZ2_INSTANTIATE_SMALL(double)
OZ2_INSTANTIATE_SMALL(float)

}  // namespace oz2
