// Column-side kernels: B is row-major k x n, its scale vector runs over COLUMNS
// (Algorithm 1 line 1: nu in F^n) and its residue slices are wanted K-contiguous
// (transposed).  These kernels read B in place, coalesced along its rows, so no transposed
// copy of B is ever written:
//   k_col_sums, k_col_shift, k_col_again  -- the fast-mode shift of Section 4.2 per column;
//   k_col_max  -- the maximum of each column (accurate mode): partial maxima per (column strip, row
//       chunk) combined with 64-bit integer atomics, which is exact and order-independent;
//   k_residues_cols -- Algorithm 1 lines 3 and 5 for B: a 64 x 64 tile of B is read row-wise,
//       each thread reduces 8 consecutive k of one column modulo all N moduli, and the int8
//       results go through LDS so that every modulus' 4 KiB piece of the K-blocked output
//       [Kp/64][Np][64] is written as one contiguous run.
#include <algorithm>

#include "oz2_convert.hpp"
#include "oz2_kernels.hpp"

namespace oz2 {
namespace {

using namespace dev;

constexpr int kRowChunk = 512;       // rows per workgroup of k_col_max

__global__ __launch_bounds__(256) void k_fill_u64(uint64_t *p, int64_t count, uint64_t v) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = v;
}

// colmax[c] = max_h bits(|X[h][c]|)
template <typename T>
__global__ __launch_bounds__(256) void k_col_max(const T *__restrict__ X, int64_t ld, int64_t rows,
                                                 int64_t cols, unsigned long long *colmax) {
    __shared__ uint64_t part[4][kColStrip];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * kColStrip + lane;
    const int64_t r0 = (int64_t)blockIdx.y * kRowChunk;
    const int64_t r1 = r0 + kRowChunk < rows ? r0 + kRowChunk : rows;
    uint64_t mx = 0;
    if (c < cols) {
#pragma unroll 8
        for (int64_t r = r0 + wave; r < r1; r += 4) {
            uint64_t b = (uint64_t)__double_as_longlong(fabs((double)X[r * ld + c]));
            mx = b > mx ? b : mx;
        }
    }
    part[wave][lane] = mx;
    __syncthreads();
    if (wave == 0 && c < cols) {
        for (int w = 1; w < 4; ++w) mx = part[w][lane] > mx ? part[w][lane] : mx;
        if (mx) atomicMax(&colmax[c], (unsigned long long)mx);
    }
}

// The fast-mode shift in one read of X.  The exponent e of a column's maximum is known only once all of it has been
// read, so each workgroup keeps a tile of kSumRows x 64 elements in registers, takes the exponent e_c of
// each column of the tile, and stores with it the sums of squares
//   S_d = sum ceil(|x| 2^(15 - e_c - d))^2,  d = 0 .. kSumLevels - 1,
// of which k_col_shift picks the one with e_c + d = e.  Where the whole column's maximum is further
// above the tile's, it brackets the tile's sum (see there).  HBM bound.  Both kernels against four launches (clearing, maxima,
// squares from a second read, shifts), us: 40000 x 1000 FP64 119 -> 66, 16384 x 16384 FP64 688 -> 379, 8192 x 8192 FP32 117 -> 75,
// 5000 x 2000 FP64 45 -> 24.  A workgroup's loads all precede its arithmetic, so others have to be
// resident beside it: 512 threads with 32 rows each 74 at 40000 x 1000 (256: 58), 512 with 16 72.  Pairs of FP32 columns
// per lane gain 6 of 69 at 8192 x 8192 and cost as much for few columns.
// A word holds S_d <= 2^39 and, for d = 0, e_c + kExpBias above it (0: the tile's column is zero).
constexpr int kSumThreads = 256, kSumPer = 32;
constexpr int kSumRows = kSumThreads / kWave * kSumPer, kSumLevels = 3;
constexpr int kExpBias = 2048, kExpShift = 48;
constexpr uint64_t kSumMask = ((uint64_t)1 << kExpShift) - 1;
static_assert(kSumRows <= 1 << (39 - 32), "S_d and the exponent share a word");
// The words of all tiles, and behind them what k_col_shift leaves to k_col_again (five words per column, or fewer), lie where the residue slices
// of the same factor go afterwards: N >= 2 bytes per element.
static_assert((kSumLevels * ((kPadK + kSumRows - 1) / kSumRows) + 5) * sizeof(uint64_t) <= OZ2_MIN_MODULI * kPadK, "words beyond the slices");
static_assert(kSumThreads / kWave > kSumLevels, "a wavefront clears what k_col_shift adds to");

// Columns to read again, in strips of kAgainCols: the sum of a column's known tiles; of a strip, which columns and how many workgroups are
// done with it; the strips that have any, and how many these are.
constexpr int kAgainCols = 16;
struct Again {
    unsigned long long *sum, *mask, *done, *list, *count;
    __host__ __device__ Again(uint64_t *words, int64_t tiles, int64_t cols) {
        sum = reinterpret_cast<unsigned long long *>(words + tiles * kSumLevels * cols);
        mask = sum + cols; done = mask + cols; list = done + cols; count = list + cols;
    }
};

// (3 workgroups per compute unit: 168 registers in FP64; two more cost a third of them and 5 to 10 %.)
template <typename T>
__global__ __launch_bounds__(kSumThreads, 3) void k_col_sums(const T *__restrict__ X, int64_t ld, int64_t rows,
                                                          int64_t cols, uint64_t *__restrict__ words) {
    constexpr int kWaves = kSumThreads / kWave;
    __shared__ uint64_t part[kSumLevels][kWaves][kColStrip];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * kColStrip + lane;
    const int64_t r0 = (int64_t)blockIdx.y * kSumRows + wave;
    const T *x = X + (c < cols ? c : cols - 1);
    T v[kSumPer];
#pragma unroll
    for (int i = 0; i < kSumPer; ++i) {
        const int64_t r = r0 + i * kWaves;
        v[i] = x[(r < rows ? r : rows - 1) * ld];                     // beyond the end: a number that is not counted
    }
    uint64_t mx = 0;
#pragma unroll
    for (int i = 0; i < kSumPer; ++i) {
        if (r0 + i * kWaves >= rows) v[i] = T(0);
        const uint64_t b = abs_bits((double)v[i]);
        mx = b > mx ? b : mx;
    }
    part[0][wave][lane] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mx = part[0][w][lane] > mx ? part[0][w][lane] : mx;
    __syncthreads();                                                  // part is reused
    const int e = floor_log2_of_bits(mx);
    uint64_t sum[kSumLevels];
    if (e < 1024) {
        double s[kSumLevels] = {};                                    // exact: see kMaxSquares
#pragma unroll
        for (int i = 0; i < kSumPer; ++i)
#pragma unroll
            for (int d = 0; d < kSumLevels; ++d) {
                const double q = ceil(ldexp(fabs((double)v[i]), 15 - e - d));
                s[d] = fma(q, q, s[d]);
            }
#pragma unroll
        for (int d = 0; d < kSumLevels; ++d) sum[d] = (uint64_t)s[d];
    } else {                                                          // an infinity or NaN: no finite column has this e
        sum[0] = 0;
        for (int i = 0; i < kSumPer; ++i) {
            const uint64_t q = (uint64_t)ceil(ldexp(fabs((double)v[i]), 15 - e));
            sum[0] += q * q;
        }
#pragma unroll
        for (int d = 1; d < kSumLevels; ++d) sum[d] = 0;
    }
#pragma unroll
    for (int d = 0; d < kSumLevels; ++d) part[d][wave][lane] = sum[d];
    __syncthreads();
    if (wave == kSumLevels && c < cols && c % kAgainCols == 0 && blockIdx.y == 0) {
        const Again a(words, gridDim.y, cols);
        a.mask[c / kAgainCols] = a.done[c / kAgainCols] = 0;
        if (c == 0) *a.count = 0;
    }
    if (wave < kSumLevels && c < cols) {                              // wavefront d writes S_d
        uint64_t t = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) t += part[wave][w][lane];
        t &= kSumMask;
        if (wave == 0 && mx) t |= (uint64_t)(e + kExpBias) << kExpShift;
        words[((int64_t)blockIdx.y * kSumLevels + wave) * cols + c] = t;
    }
}

// t[c] from the words of all tiles.  With d = e - e_c < kSumLevels for every tile of the column (random data: the
// maxima of 128 numbers and of 2^17 differ by less than a factor of 8) the sum T is exact.  A tile further below
// adds an interval: q' = ceil(y / 2^d') for the y behind its last sum S (n numbers q = ceil(y)), hence
// q / 2^d' <= q' < q / 2^d' + 1, and with Cauchy's sum q <= sqrt(n S)
//   S / 4^d' - n <= sum q'^2 <= S / 4^d' + 2 sqrt(n S) / 2^d' + n
// (the n below is for numbers that the scaling takes to zero).  If both ends of T's interval give the same
// shift, that is the shift; otherwise the tiles with an interval are read again.  The thresholds are a
// factor of 4 apart, T is at least 2^30 and the interval is narrow (2^-6 to 2^-10 of T), so this is rare.  A compute unit reads 0.5 to 0.6 rows of
// a column per ns, so those of long columns (LATER) go to a launch of their own, k_col_again.
//
// THREADS / COLS threads go through the words of a column, the first kHeld tiles of each from registers.
constexpr int kHeld = 8;

// v combined over the lanes of a wavefront with the same lane % COLS
template <int COLS, typename V, typename F>
__device__ __forceinline__ V over_column(V v, F f) {
#pragma unroll
    for (int off = COLS; off < kWave; off <<= 1) v = f(v, __shfl_xor(v, off, kWave));
    return v;
}

template <typename T, int THREADS, int COLS, bool LATER>
__global__ __launch_bounds__(THREADS) void k_col_shift(const T *__restrict__ X, int64_t ld, int64_t rows, int64_t cols,
                                                       const uint64_t *__restrict__ words, Again later,
                                                       ShiftArgs sa, int32_t *__restrict__ t) {
    constexpr int kWaves = THREADS / kWave, kGroups = THREADS / COLS;
    __shared__ uint64_t part[kWaves][COLS];
    __shared__ double low[kWaves][COLS], high[kWaves][COLS];
    __shared__ uint64_t again, known[COLS];
    __shared__ int exponent[COLS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = threadIdx.x % COLS, group = threadIdx.x / COLS;
    const int64_t c0 = (int64_t)blockIdx.x * COLS, c = c0 + col;
    const int tiles = (int)((rows + kSumRows - 1) / kSumRows);
    const uint64_t *w = words + (c < cols ? c : cols - 1);
    const auto larger = [](uint64_t x, uint64_t y) { return x > y ? x : y; };
    const auto plus = [](auto x, auto y) { return x + y; };

    uint64_t held[kHeld], top = 0;                                    // top: the word of the largest exponent
#pragma unroll
    for (int j = 0; j < kHeld; ++j) {
        const int i = group + j * kGroups;
        held[j] = i < tiles ? w[(int64_t)i * kSumLevels * cols] : 0;
    }
#pragma unroll 8
    for (int i = group + kHeld * kGroups; i < tiles; i += kGroups) top = larger(top, w[(int64_t)i * kSumLevels * cols]);
#pragma unroll
    for (int j = 0; j < kHeld; ++j) top = larger(top, held[j]);
    top = over_column<COLS>(top, larger);
    if (lane < COLS) part[wave][col] = top;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kWaves; ++i) top = larger(top, part[i][col]);
    __syncthreads();                                                  // part is reused
    const int code = (int)(top >> kExpShift);
    uint64_t sum = 0;
    double lo = 0.0, hi = 0.0;
    const auto below = [&](uint64_t u0) { return code - (int)(u0 >> kExpShift); };
    const auto level = [&](uint64_t u0) { return below(u0) < kSumLevels ? below(u0) : kSumLevels - 1; };
    const auto add = [&](uint64_t u0, uint64_t s) {
        s &= kSumMask;
        const int d = below(u0);
        if (d < kSumLevels) {
            sum += s;
        } else if (u0) {
            const double n = kSumRows, a = ldexp((double)s, -2 * (d - (kSumLevels - 1)));
            lo += a - n;
            hi += a + 2.0 * sqrt(n * a) + n;
        }
    };
    uint64_t s[kHeld];
#pragma unroll
    for (int j = 0; j < kHeld; ++j) {
        const int i = group + j * kGroups;
        s[j] = i < tiles ? w[((int64_t)i * kSumLevels + level(held[j])) * cols] : 0;
    }
#pragma unroll
    for (int j = 0; j < kHeld; ++j) add(held[j], s[j]);
#pragma unroll 8
    for (int i = group + kHeld * kGroups; i < tiles; i += kGroups) {
        const uint64_t *u = w + (int64_t)i * kSumLevels * cols;
        const uint64_t u0 = u[0];
        add(u0, u[(int64_t)level(u0) * cols]);
    }
    sum = over_column<COLS>(sum, plus);
    lo = over_column<COLS>(lo, plus);
    hi = over_column<COLS>(hi, plus);
    if (lane < COLS) { part[wave][col] = sum; low[wave][col] = lo; high[wave][col] = hi; }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int i = 1; i < kWaves; ++i) { sum += part[i][col]; lo += low[i][col]; hi += high[i][col]; }
        const int e = code - kExpBias;
        bool open = false;
        if (lane < COLS && c < cols) {
            exponent[col] = e;
            known[col] = sum;
            // 2^-40 and 1 cover the rounding of lo and hi
            const double a = (double)sum + lo * (1.0 - 0x1p-40) - 1.0, b = (double)sum + hi * (1.0 + 0x1p-40) + 1.0;
            const bool exact = hi == 0.0;
            const int f = shift_exponent(exact ? sum : a > 0.0 ? (uint64_t)a : 0, sa);
            open = !exact && f != shift_exponent((uint64_t)b, sa);
            t[c] = open ? e : top ? f - e : 0;                        // 0: an all-zero column; e: for k_col_again
            if (LATER && open) {
                later.sum[c] = sum;
                const int64_t strip = c / kAgainCols;
                if (atomicOr(&later.mask[strip], 1ull << (c % kAgainCols)) == 0) later.list[atomicAdd(later.count, 1ull)] = strip;
            }
        }
        const uint64_t mask = __ballot(open);
        if (lane == 0) again = mask;
    }
    if (LATER) return;
    __syncthreads();
    for (uint64_t m = again; m; m &= m - 1) {                         // the same in every thread
        const int j = __ffsll((unsigned long long)m) - 1;
        const int e = exponent[j];
        sum = 0;
        // A wavefront's 64 rows lie in one tile.
        constexpr int kFlight = 8;
        for (int64_t r0 = wave * kWave; r0 < rows; r0 += kFlight * THREADS) {
            T x[kFlight];
            uint64_t u0[kFlight];
#pragma unroll
            for (int i = 0; i < kFlight; ++i) {
                const int64_t r = r0 + i * THREADS;
                u0[i] = words[(r < rows ? r : r0) / kSumRows * kSumLevels * cols + c0 + j];
            }
#pragma unroll
            for (int i = 0; i < kFlight; ++i) {
                const int64_t r = r0 + i * THREADS + lane;
                x[i] = T(0);
                if (u0[i] && e + kExpBias - (int)(u0[i] >> kExpShift) >= kSumLevels && r < rows) x[i] = X[r * ld + c0 + j];
            }
#pragma unroll
            for (int i = 0; i < kFlight; ++i) {
                const uint64_t q = (uint64_t)ceil(ldexp(fabs((double)x[i]), 15 - e));
                sum += q * q;
            }
        }
        sum = wave_sum(sum);
        __syncthreads();                                              // part is reused
        if (lane == 0) part[wave][0] = sum;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int i = 1; i < kWaves; ++i) sum += part[i][0];
            t[c0 + j] = shift_exponent(known[j] + sum, sa) - e;
        }
    }
}

// The second read of long columns: workgroups in teams, a strip of columns for each team at a time, of which a wavefront reads
// 32 rows of a tile that has to be read, 4 rows at a time (t holds the exponents).  The last member of a team to add its sums computes the shifts.
// Bound: memory latency.  Whole calls with 64 rows of A, us, everything read twice (no words) | read again in k_col_shift, by at most 256 workgroups
// for all columns | this: 200000 x 400 FP32 with one row 1000 times the others 1425 | 1540 | 1340, 300000 x 300 FP32 exp(2 normal) 2099 | 2144 | 1946, 70000 x 2000
// FP64 exp(4 normal) 1772 | 1517 | 1390, 70000 x 8192 5725 | 5131 | 5020; nothing to read again: 66000 x 64 552 | 289 | 291, 300000 x 300 2763 | 2558 | 2556.
// Up to 65536 rows a column costs at most 0.13 ms in k_col_shift, and two launches of sums and words are what the calls of a few columns consist of.
constexpr int kAgainThreads = 1024, kAgainGrid = 256;

template <typename T>
__global__ __launch_bounds__(kAgainThreads) void k_col_again(const T *__restrict__ X, int64_t ld, int64_t rows, int64_t cols,
                                                             const uint64_t *__restrict__ words, Again a, ShiftArgs sa, int32_t *t) {
    constexpr int kWaves = kAgainThreads / kWave, kRows = kWave / kAgainCols, kFlight = 8, kUnit = kRows * kFlight;
    static_assert(kSumRows % kUnit == 0, "a unit's rows lie in one tile");
    __shared__ uint64_t part[kWaves][kAgainCols];
    __shared__ bool last;
    const int strips = (int)*a.count;
    if (strips == 0) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane % kAgainCols, row = lane / kAgainCols;
    const int teams = strips < (int)gridDim.x ? strips : (int)gridDim.x, members = (int)gridDim.x / teams;
    const int team = (int)blockIdx.x / members, member = (int)blockIdx.x % members;
    if (team >= teams) return;
    const int64_t units = (rows + kUnit - 1) / kUnit;
    for (int i = team; i < strips; i += teams) {                      // the same in every thread of a workgroup
        const int64_t strip = (int64_t)a.list[i], c = strip * kAgainCols + col;
        const bool open = a.mask[strip] >> col & 1;
        const int e = open ? t[c] : 0;
        const auto word = [&](int64_t u) { return open && u < units ? words[u * kUnit / kSumRows * kSumLevels * cols + c] : 0; };
        uint64_t sum = 0, u0 = word(member * kWaves + wave);
        for (int64_t u = member * kWaves + wave; u < units; u += members * kWaves) {
            const uint64_t next = word(u + members * kWaves);
            if (u0 && e + kExpBias - (int)(u0 >> kExpShift) >= kSumLevels) {
                T x[kFlight];
#pragma unroll
                for (int j = 0; j < kFlight; ++j) {
                    const int64_t r = u * kUnit + j * kRows + row;
                    x[j] = r < rows ? X[r * ld + c] : T(0);
                }
#pragma unroll
                for (int j = 0; j < kFlight; ++j) {
                    const uint64_t q = (uint64_t)ceil(ldexp(fabs((double)x[j]), 15 - e));
                    sum += q * q;
                }
            }
            u0 = next;
        }
        sum = over_column<kAgainCols>(sum, [](uint64_t x, uint64_t y) { return x + y; });
        if (lane < kAgainCols) part[wave][col] = sum;
        __syncthreads();
        if (threadIdx.x < kAgainCols && open) {
            for (int w = 1; w < kWaves; ++w) sum += part[w][col];
            atomicAdd(&a.sum[c], (unsigned long long)sum);
            __threadfence();
        }
        __syncthreads();
        if (threadIdx.x == 0) last = atomicAdd(&a.done[strip], 1ull) == (unsigned long long)members - 1;
        __syncthreads();
        if (last && threadIdx.x < kAgainCols && open) {
            __threadfence();
            t[c] = shift_exponent(atomicAdd(&a.sum[c], 0ull), sa) - e;
        }
    }
}

constexpr int kResColThreads = 512;   // 16384^2, 16 moduli: 256 threads with two pieces each 1.42 ms, 1.20 ms with one

template <typename T, int ROUNDS, int KIND>
__global__ __launch_bounds__(kResColThreads) void k_residues_cols(const T *__restrict__ X, int64_t ld,
                                                       int64_t rows, int64_t cols,
                                                       const int32_t *__restrict__ t, ModArgs ma,
                                                       int8_t *__restrict__ out, int64_t cols_pad,
                                                       int64_t rows_pad, int64_t cols_stride) {
    residues_cols_block<T, ROUNDS, KIND, kResColThreads, true>(blockIdx.x, blockIdx.y, X, ld, rows, cols, t, ma, out, cols_pad,
                                         rows_pad, cols_stride);
}

}  // namespace

template <typename T>
hipError_t launch_shifts_cols(const T *X, int64_t ld, int64_t rows, int64_t cols,
                              const ShiftArgs &sa, void *scratch, int32_t *t, hipStream_t stream) {
    uint64_t *words = static_cast<uint64_t *>(scratch);
    const unsigned strips = (unsigned)((cols + kColStrip - 1) / kColStrip);
    hipLaunchKernelGGL((k_col_sums<T>), dim3(strips, (unsigned)((rows + kSumRows - 1) / kSumRows)), dim3(kSumThreads), 0,
                       stream, X, ld, rows, cols, words);
    const int64_t tiles = (rows + kSumRows - 1) / kSumRows;
    const Again later(words, tiles, cols);
    const auto shift = [&](auto kernel, int threads, int per) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((cols + per - 1) / per)), dim3(threads), 0, stream, X, ld, rows, cols, words, later, sa, t);
    };
    // The fewest threads per column (16, 64 or 256) whose registers hold all its words; of long columns, which are often few,
    // fewer per workgroup.  us for 16 | 64 | 256: 16384 x 16384 10.5 | 28 | 69, 40000 x 1000 16 | 7.6 | 8.3, 10^6 x 100 383 | 110 | 44.
    if (tiles <= 16 * kHeld) shift(k_col_shift<T, 256, 16, false>, 256, 16);
    else if (tiles <= 64 * kHeld) shift(k_col_shift<T, 256, 4, false>, 256, 4);
    else {
        shift(k_col_shift<T, 1024, 4, true>, 1024, 4);
        hipLaunchKernelGGL((k_col_again<T>), dim3(kAgainGrid), dim3(kAgainThreads), 0, stream, X, ld, rows, cols, words, later, sa, t);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_residues_cols(const T *X, int64_t ld, int64_t rows, int64_t cols, const int32_t *t,
                                const ModArgs &ma, int8_t *out, int64_t cols_pad, int64_t rows_pad,
                                hipStream_t stream, int64_t cols_stride) {
    if (cols_stride == 0) cols_stride = cols_pad;
    dim3 grid((unsigned)(cols_pad / kColStrip), (unsigned)(rows_pad / kBlockK));
    if (ma.rounds == 1)
        hipLaunchKernelGGL((k_residues_cols<T, 1, 0>), grid, dim3(kResColThreads), 0, stream, X, ld, rows, cols, t,
                           ma, out, cols_pad, rows_pad, cols_stride);
    else
        hipLaunchKernelGGL((k_residues_cols<T, 2, 0>), grid, dim3(kResColThreads), 0, stream, X, ld, rows, cols, t,
                           ma, out, cols_pad, rows_pad, cols_stride);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_magnitudes_cols(const T *X, int64_t ld, int64_t rows, int64_t cols,
                                  const int32_t *pre, int8_t *out, int64_t cols_pad,
                                  int64_t rows_pad, hipStream_t stream) {
    dim3 grid((unsigned)(cols_pad / kColStrip), (unsigned)(rows_pad / kBlockK));
    ModArgs none{};
    hipLaunchKernelGGL((k_residues_cols<T, 1, 1>), grid, dim3(kResColThreads), 0, stream, X, ld, rows, cols, pre,
                       none, out, cols_pad, rows_pad, cols_pad);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_col_maxbits(const T *X, int64_t ld, int64_t rows, int64_t cols,
                              unsigned long long *colmax, hipStream_t stream) {
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)((cols + 255) / 256)), dim3(256), 0, stream,
                       reinterpret_cast<uint64_t *>(colmax), cols, 0ull);
    dim3 grid((unsigned)((cols + kColStrip - 1) / kColStrip), (unsigned)((rows + kRowChunk - 1) / kRowChunk));
    hipLaunchKernelGGL((k_col_max<T>), grid, dim3(256), 0, stream, X, ld, rows, cols, colmax);
    return hipGetLastError();
}

#define OZ2_INSTANTIATE_COLS(T)                                                                   \
    template hipError_t launch_shifts_cols<T>(const T *, int64_t, int64_t, int64_t,               \
                                              const ShiftArgs &, void *, int32_t *, hipStream_t); \
    template hipError_t launch_magnitudes_cols<T>(const T *, int64_t, int64_t, int64_t,           \
                                                  const int32_t *, int8_t *, int64_t, int64_t,    \
                                                  hipStream_t);                                   \
    template hipError_t launch_col_maxbits<T>(const T *, int64_t, int64_t, int64_t,               \
                                              unsigned long long *, hipStream_t);                 \
    template hipError_t launch_residues_cols<T>(const T *, int64_t, int64_t, int64_t,             \
                                                const int32_t *, const ModArgs &, int8_t *,       \
                                                int64_t, int64_t, hipStream_t, int64_t);
OZ2_INSTANTIATE_COLS(double)
OZ2_INSTANTIATE_COLS(float)

}  // namespace oz2
