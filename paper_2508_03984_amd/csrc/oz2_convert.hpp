// Device code of the conversion to INT8 residues (Algorithm 1 lines 2-5) shared by the row
// kernels, the column kernels, the fused conversion and accurate mode's residue launch for small problems: the reduction of an
// integer-valued FP64 number modulo the moduli of Section 4.1, and the work of one workgroup
// of the row form (residues_block) and of the column form (residues_cols_block).
#pragma once
#include "oz2_kernels.hpp"

namespace oz2 {
namespace dev {

constexpr int kWave = 64;
constexpr int kColStrip = 64;        // columns per workgroup of the column form (one per lane)

// The sums of squares behind the shifts are sums of integers of at most 2^32 in FP64: exact up to this many.
constexpr int64_t kMaxSquares = (int64_t)1 << (53 - 32);
static_assert(OZ2_MAX_K_BLOCKED <= kMaxSquares, "sums of squares beyond 2^53 would be rounded");

// 16 bytes of elements for one load at element alignment, which the hardware's global loads take.
template <typename T>
using Vec16 __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T)))) = T;

// f on every element of a contiguous vector by a workgroup of THREADS threads: eight 16-byte loads in
// flight per thread (a loop of single elements reached 2.2 TB/s on rows of 40000).
template <typename T, int THREADS, typename F>
__device__ __forceinline__ void scan_row(const T *__restrict__ x, int64_t len, F f) {
    constexpr int kVec = 16 / sizeof(T), kFlight = 8;
    const Vec16<T> *v = reinterpret_cast<const Vec16<T> *>(x);
    const int64_t n = len / kVec;
    int64_t i = threadIdx.x;
    for (; i + (kFlight - 1) * THREADS < n; i += kFlight * THREADS) {
        Vec16<T> w[kFlight];
#pragma unroll
        for (int j = 0; j < kFlight; ++j) w[j] = v[i + j * THREADS];
#pragma unroll
        for (int j = 0; j < kFlight; ++j)
#pragma unroll
            for (int e = 0; e < kVec; ++e) f((double)w[j][e]);
    }
    for (; i < n; i += THREADS) {
        const Vec16<T> w = v[i];
#pragma unroll
        for (int e = 0; e < kVec; ++e) f((double)w[e]);
    }
    const int64_t h = n * kVec + threadIdx.x;
    if (h < len) f((double)x[h]);
}

__device__ inline uint64_t abs_bits(double x) { return (uint64_t)__double_as_longlong(fabs(x)); }

__device__ inline uint64_t wave_max(uint64_t v) {
    for (int off = kWave / 2; off > 0; off >>= 1) {
        uint64_t o = __shfl_xor(v, off, kWave);
        v = o > v ? o : v;
    }
    return v;
}
__device__ inline uint64_t wave_sum(uint64_t v) {
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// f = f_max - j, j = the number of thresholds below v (the table is sorted and filled up with the largest
// number; at most levels - 1): all comparisons at once instead of a search whose every step waits for a
// scalar load.
__device__ __forceinline__ int shift_exponent(uint64_t v, const ShiftArgs &sa) {
    int j = 0;
#pragma unroll
    for (int i = 0; i < kMaxLevels; ++i) j += v > sa.theta[i] ? 1 : 0;
    return sa.f_max - (j < sa.levels - 1 ? j : sa.levels - 1);
}

// v of another lane: bits 1:0 of the lane number flipped by the quad permutations, the others by
// mirroring groups of 8 or 16 lanes (the callers have made the lanes of a group equal before).
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppMirror8 = 0x141, kDppMirror16 = 0x140;
template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, false);
    return (uint64_t)(uint32_t)lo | ((uint64_t)(uint32_t)hi << 32);
}

// ----------------------------------------------------------------------------------------
// Residues.  x' = trunc(x 2^t) is an integer-valued FP64 number below 2^77.  Its
// symmetric residue modulo p comes from rounds of  y <- fma(-rint(y * (1/p)), p, y),
// the reduction of Section 4.2 kept in FP64 throughout:
//   the first round is exact (the difference is an integer below 2^26 in magnitude) and leaves
//   |y| <= p/2 + 2^-52 |x'|;  for |x'| < 2^46 the quotient estimate is within 2^-13 of
//   x'/p, closer than any integer/p can be to a half-integer for odd p, so rint returns
//   round(x'/p) and y is already the residue in [-(p-1)/2, (p-1)/2];
//   otherwise two rounds.  The first one is shared by up to five moduli: it reduces
//   modulo their product M < 2^40 (group_reduce), which is exact for the same reason (the
//   difference is an integer, |y| <= M/2 + 2^-51 |x'| < 2^45) and y = x' (mod M) implies
//   y = x' (mod p) for every p that divides M; the second round, on |y| < 2^46, is the
//   one-round case above for each of these p.
// p = 256: 1/p is exact, y lands in [-128, 128], and of 128 and -128, which are the same class (Section 4.1),
// only the low byte is kept: 0x80 for both.
// ----------------------------------------------------------------------------------------
__device__ inline double group_reduce(double x, double M, double Minv) {
    return fma(-rint(x * Minv), M, x);
}

// The one-round case for 8 numbers at a time, only the low byte of y - p rint(y/p) being wanted:
// one FP64 FMA leaves 1.5 * 2^52 + rint(y/p), whose low half holds the quotient modulo 2^32, and the rest
// is 16-bit integer arithmetic on two numbers per instruction.  (The FMA rounds y/p once where a
// multiplication followed by rint rounds twice; the quotient is the same, since y/p is further from a
// half-integer than either error for odd p, and p = 256 divides exactly.)  Per number and modulus one FP64 FMA, half a
// packed multiply-add and three quarters of a byte permute, where multiplication, rint, FMA, conversion (all FP64) and the
// insertion of a byte were five and more.
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
constexpr double kRintMagic = 6755399441055744.0;                     // 1.5 * 2^52
__device__ __forceinline__ uint32_t low_word(double x) { return (uint32_t)__double_as_longlong(x); }
__device__ __forceinline__ us2 low_halves(double x0, double x1) {     // the low 16 bits of both
    return __builtin_bit_cast(us2, __builtin_amdgcn_perm(low_word(x1), low_word(x0), 0x05040100u));
}

struct ResidueInput {
    double y[8];                                                      // |y| < 2^46, integers
    us2 low[4];                                                       // their low 16 bits
    __device__ __forceinline__ void set_low() {
#pragma unroll
        for (int i = 0; i < 4; ++i) low[i] = low_halves(y[2 * i] + kRintMagic, y[2 * i + 1] + kRintMagic);
    }
    // the residues modulo p of the 8 numbers as 8 bytes
    __device__ __forceinline__ uint2 residues(int p, double pinv) const {
        const us2 neg_p = {(unsigned short)-p, (unsigned short)-p};
        uint32_t w[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            us2 r[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int e = 4 * h + 2 * i;
                r[i] = low_halves(fma(y[e], pinv, kRintMagic), fma(y[e + 1], pinv, kRintMagic)) * neg_p + low[e / 2];
            }
            w[h] = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, r[1]), __builtin_bit_cast(uint32_t, r[0]),
                                         0x06040200u);
        }
        return make_uint2(w[0], w[1]);
    }
};

constexpr int kResPerThread = 8;     // consecutive elements per thread -> 8-byte stores

// store(s, bytes) for the moduli s0 <= s < n of one group.  The constants of all of them are requested
// together (s0 + 4 < kMaxModuli always): where few wavefronts are resident, one that waits for each
// modulus' own scalar loads takes about twice as long.
template <typename Store>
__device__ __forceinline__ void emit_group(const ResidueInput &in, const ModArgs &ma, int s0, int n, Store store) {
    int p[kModGroup];
    double pinv[kModGroup];
#pragma unroll
    for (int g = 0; g < kModGroup; ++g) { p[g] = ma.p[s0 + g]; pinv[g] = ma.pinv[s0 + g]; }
#pragma unroll
    for (int g = 0; g < kModGroup; ++g)
        if (s0 + g < n) store(s0 + g, in.residues(p[g], pinv[g]));
}
static_assert(kMaxModuli % kModGroup == 0, "emit_group reads the constants of whole groups");

// KIND 0: residues of trunc(x 2^t) for all moduli.  KIND 1 (accurate mode): the single
// 7-bit magnitude matrix ceil(|x| 2^t), written as slice 0.
template <typename T, int ROUNDS, int KIND>
__device__ __forceinline__ void residues_block(int64_t block, const T *__restrict__ X, int64_t ld,
                                               int64_t rows, int64_t len,
                                               const int32_t *__restrict__ t, const ModArgs &ma,
                                               int8_t *__restrict__ out, int64_t rows_pad,
                                               int64_t len_pad, int64_t rows_stride, int group_lo = 0,
                                               int group_hi = 1 << 30) {
    // Only the moduli of the groups [group_lo, group_hi) (groups of kModGroup) are produced: small
    // problems spread the groups over several workgroups (see oz2_small.hip).
    // rows_pad rows are written (zeros beyond `rows`); rows_stride >= rows_pad is the number of
    // rows of the whole slice, of which this launch may fill a block.
    // Thread -> (K block, row, 8-element piece of the 64-wide block), piece fastest: a
    // wavefront writes 8 rows x 64 B = 512 contiguous bytes of the blocked output and reads
    // 512 contiguous bytes of each of 8 input rows.
    constexpr int kPieces = kBlockK / kResPerThread;
    const int64_t idx = block * 256 + threadIdx.x;
    if (idx >= rows_pad * (len_pad / kResPerThread)) return;
    const int64_t kb = idx / (rows_pad * kPieces);
    const int64_t r = (idx / kPieces) % rows_pad;
    const int64_t h0 = kb * kBlockK + (idx % kPieces) * kResPerThread;

    double v[kResPerThread];
    if (r < rows) {
        const int sh = t[r];
        const T *x = X + r * ld + h0;
        T raw[kResPerThread];
        if (h0 + kResPerThread <= len) {
            // whole piece in range: 16-byte loads (1.9 -> 1.3 ms at 16384^2), at any element alignment
            constexpr int kVec = 16 / sizeof(T);
#pragma unroll
            for (int i = 0; i < kResPerThread / kVec; ++i) {
                const Vec16<T> q = reinterpret_cast<const Vec16<T> *>(x)[i];
#pragma unroll
                for (int c = 0; c < kVec; ++c) raw[i * kVec + c] = q[c];
            }
        } else {
#pragma unroll
            for (int i = 0; i < kResPerThread; ++i) raw[i] = (h0 + i < len) ? x[i] : T(0);
        }
#pragma unroll
        for (int i = 0; i < kResPerThread; ++i)
            v[i] = KIND == 0 ? trunc(ldexp((double)raw[i], sh)) : ceil(ldexp(fabs((double)raw[i]), sh));
    } else {
#pragma unroll
        for (int i = 0; i < kResPerThread; ++i) v[i] = 0.0;
    }

    const int64_t plane = rows_stride * len_pad;
    int8_t *o = out + (kb * rows_stride + r) * kBlockK + (h0 - kb * kBlockK);
    if (KIND == 1) {
        uint32_t w[2] = {0u, 0u};
#pragma unroll
        for (int i = 0; i < kResPerThread; ++i) w[i >> 2] |= ((uint32_t)(int)v[i] & 0xffu) << (8 * (i & 3));
        *reinterpret_cast<uint2 *>(o) = make_uint2(w[0], w[1]);
        return;
    }
    const int s_end = group_hi < (ma.n + kModGroup - 1) / kModGroup ? group_hi * kModGroup : ma.n;
    for (int s0 = group_lo * kModGroup; s0 < s_end; s0 += kModGroup) {
        ResidueInput in;
#pragma unroll
        for (int i = 0; i < kResPerThread; ++i)
            in.y[i] = ROUNDS == 2 ? group_reduce(v[i], ma.group_mod[s0 / kModGroup], ma.group_inv[s0 / kModGroup]) : v[i];
        in.set_low();
        emit_group(in, ma, s0, ma.n, [&](int s, uint2 w) { *reinterpret_cast<uint2 *>(o + (int64_t)s * plane) = w; });
    }
}

// KIND as in the row kernel: 0 = residues for all moduli, 1 = the 7-bit magnitudes (slice 0).
// THREADS: 512 (one piece of 8 elements per thread) or 256 (two).
// LARGE: the launches of large factors (k_residues_cols); otherwise those of accurate mode's small ones (oz2_small.hip).
template <typename T, int ROUNDS, int KIND, int THREADS, bool LARGE>
__device__ __forceinline__ void residues_cols_block(int64_t block_x, int64_t block_y,
                                                    const T *__restrict__ X, int64_t ld, int64_t rows,
                                                    int64_t cols, const int32_t *__restrict__ t,
                                                    const ModArgs &ma, int8_t *__restrict__ out,
                                                    int64_t cols_pad, int64_t rows_pad,
                                                    int64_t cols_stride, int group_lo = 0,
                                                    int group_hi = 1 << 30) {
    // Only the moduli of the groups [group_lo, group_hi) are produced (as in residues_block).
    // cols_pad columns are written (the grid covers them); cols_stride >= cols_pad is the number
    // of rows of the whole transposed slice, of which this launch may fill a block.
    // LDS: per modulus 8 pieces x 64 columns x 8 bytes, piece-major so that the writes of a
    // wavefront (one piece, 64 columns) are contiguous; 8 bytes of padding per piece row.
    // Moduli are processed kGroup at a time to keep the LDS footprint (and so the number of
    // resident workgroups) independent of N; a group is also what shares the first reduction
    // round when two are needed.
    constexpr int kGroup = kModGroup;
    constexpr int kWaves = THREADS / kWave, kHalves = 8 / kWaves;     // pieces wave, wave + kWaves
    // Two of them in turn, so that one barrier per group is enough, in the large launches (in accurate mode's launch for small residues
    // one: 2048^3 N = 15 196.6 us a call, two 199.7).
    constexpr int kStages = LARGE ? 2 : 1;
    __shared__ uint2 stages[kStages][kGroup][8][65];
    int turn = 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c = block_x * kColStrip + lane;                     // column of X = row of the output
    const int64_t kb = block_y;                                       // K block
    const int sh = c < cols ? t[c] : 0;

    // All loads first, from places that exist (a number beyond the end is not used).  Ordinary ones: past the L2 the
    // kernel is 5 to 8 % faster where rows are whole 128-byte lines, but 10 to 30 % slower where they are not (strips share lines
    // then), and what follows finds less of the operand in the memory-side cache.  The kernel | a whole call with 64 rows of A, us, masked loads in
    // order of use and two barriers per group; this; past the L2: 8192 x 8192 FP32 N = 8 165 | 404; 129 | 342; 121 | 346,
    // 1000 columns of 40000 FP64 N = 15 181 | 563; 165 | 444; 161 | 454, 1057 of 5182 26 | 96; 25 | 71; 34 | 80, 33 of 50000 FP32 25 | 202; 20 | 85; 31 | 96,
    // 4096 of 5000 FP32 45 | 130; 41 | 108; 39 | 104, 12001 of 12000 FP64 610 | 1497; 602 | 1287; 642 | 1341.
    T raw[kHalves][8];
    const T *x = X + (c < cols ? c : cols - 1);
#pragma unroll
    for (int half = 0; half < kHalves; ++half) {
        const int64_t h0 = kb * kBlockK + (wave + kWaves * half) * 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) raw[half][i] = x[(h0 + i < rows ? h0 + i : rows - 1) * ld];
    }
    double v[kHalves][8];
#pragma unroll
    for (int half = 0; half < kHalves; ++half) {
        const int64_t h0 = kb * kBlockK + (wave + kWaves * half) * 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const double y = c < cols && h0 + i < rows ? (double)raw[half][i] : 0.0;
            v[half][i] = KIND == 0 ? trunc(ldexp(y, sh)) : ceil(ldexp(fabs(y), sh));
        }
    }

    // Write-out: per modulus the 64 columns x 64 bytes of this tile are contiguous in
    // out[s][kb][c0 .. c0+63][64]; thread -> (column, 16-byte quarter).
    const int64_t plane = cols_stride * rows_pad;
    const int part = threadIdx.x & 255, col = part >> 2, quarter = part & 3;
    const int g0 = threadIdx.x >> 8;                                  // 512 threads: two moduli at a time
    int8_t *dst = out + (kb * cols_stride + block_x * kColStrip) * kBlockK + part * 16;

    const int n_all = KIND == 0 ? ma.n : 1;
    const int n_slices = group_hi < (n_all + kGroup - 1) / kGroup ? group_hi * kGroup : n_all;
    for (int s0 = group_lo * kGroup; s0 < n_slices; s0 += kGroup) {
        const int ns = n_slices - s0 < kGroup ? n_slices - s0 : kGroup;
        uint2 (*const stage)[8][65] = stages[turn];
        turn ^= kStages - 1;
        if (KIND == 1) {
#pragma unroll
            for (int half = 0; half < kHalves; ++half) {
                uint32_t w[2] = {0u, 0u};
#pragma unroll
                for (int i = 0; i < 8; ++i) w[i >> 2] |= ((uint32_t)(int)v[half][i] & 0xffu) << (8 * (i & 3));
                stage[0][wave + kWaves * half][lane] = make_uint2(w[0], w[1]);
            }
        } else {
            ResidueInput in[kHalves];
#pragma unroll
            for (int half = 0; half < kHalves; ++half) {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    in[half].y[i] = ROUNDS == 2 ? group_reduce(v[half][i], ma.group_mod[s0 / kGroup], ma.group_inv[s0 / kGroup])
                                                : v[half][i];
                in[half].set_low();
            }
#pragma unroll
            for (int half = 0; half < kHalves; ++half)
                emit_group(in[half], ma, s0, s0 + ns,
                           [&](int s, uint2 w) { stage[s - s0][wave + kWaves * half][lane] = w; });
        }
        __syncthreads();
        for (int g = g0; g < ns; g += THREADS / 256) {
            const uint2 lo = stage[g][2 * quarter][col];
            const uint2 hi = stage[g][2 * quarter + 1][col];
            *reinterpret_cast<uint4 *>(dst + (int64_t)(s0 + g) * plane) = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
        if (!LARGE) __syncthreads();
    }
}

}  // namespace dev
}  // namespace oz2
