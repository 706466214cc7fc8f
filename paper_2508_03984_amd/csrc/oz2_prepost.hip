// Bandwidth-bound kernels of the emulation for gfx950 (row side: A, and the output):
// fast-mode shifts (Algorithm 1 line 1), residue slices (lines 2-5) and the fused
// mod-reduce + CRT + unscale epilogue (lines 7-12).  64-wide wavefronts throughout.
#include <algorithm>
#include <type_traits>

#include "oz2_convert.hpp"
#include "oz2_epilogue.hpp"
#include "oz2_kernels.hpp"
#include "oz2_tilemap.hpp"

namespace oz2 {

int residue_rounds(const Table &t, bool accurate) {
    // One reduction round gives the canonical residue while |x'| < 2^46 (see ResidueInput).
    // Fast mode: |x| < 2^(e+1) and t = f - e with f <= f_max, so |x'| < 2^(f_max+1).
    // Accurate mode: mu' brings |x| below 2^6 and the second factor is at most 2^accu_f_max
    // (reached when the maximum of Cbar is 0 or 1), so |x'| < 2^(accu_f_max+6).
    const int bits = accurate ? t.accu_f_max + 6 : t.f_max + 1;
    return bits <= 46 ? 1 : 2;
}

ModArgs make_mod_args(const Table &t, bool accurate) {
    ModArgs a{};
    a.n = t.n;
    a.rounds = residue_rounds(t, accurate);
    for (int i = 0; i < t.n; ++i) {
        a.p[i] = t.p[i];
        a.pinv_prime[i] = t.pinv_prime[i];
        a.pinv[i] = t.pinv[i];
        a.s1[i] = t.s1[i];
        a.s2[i] = t.s2[i];
    }
    for (int g = 0; g * kModGroup < t.n; ++g) {
        double M = 1.0;                                  // exact: an integer below 2^40
        for (int i = g * kModGroup; i < t.n && i < (g + 1) * kModGroup; ++i) M *= (double)t.p[i];
        a.group_mod[g] = M;
        a.group_inv[g] = 1.0 / M;
    }
    a.P1 = t.P1; a.P2 = t.P2; a.Pinv = t.Pinv;
    return a;
}

ShiftArgs make_shift_args(const Table &t) {
    ShiftArgs s{};
    s.f_max = t.f_max;
    s.levels = t.levels;
    for (int j = 0; j < kMaxLevels; ++j) s.theta[j] = j < t.levels ? t.theta[j] : ~0ull;
    return s;
}

ShiftArgs make_accu_shift_args(const Table &t) {
    ShiftArgs s{};
    s.f_max = t.accu_f_max;
    s.levels = t.accu_levels;
    for (int j = 0; j < kMaxLevels; ++j) s.theta[j] = j < t.accu_levels ? t.accu_theta[j] : ~0ull;
    return s;
}

namespace {

using namespace dev;

// ----------------------------------------------------------------------------------------
// Shifts.  One workgroup per row: pass 1 finds max|x| (as an integer compare of the FP64
// bit patterns), pass 2 sums q^2 with q = ceil(|x| 2^(15-e)) <= 2^16 by FP64 FMA: integers whose sum
// stays within 2^53 (kMaxSquares), so the sum is exact and independent of the order.  f comes from the threshold table,
// t = f - e.  k_shifts re-reads the row for pass 2 (rows of any length); k_shifts_cached
// further down keeps rows of up to 49152 elements in registers between the passes.
// ----------------------------------------------------------------------------------------
constexpr int kShiftThreads = 512;

template <typename T>
__global__ __launch_bounds__(kShiftThreads) void k_shifts(const T *__restrict__ X, int64_t ld, int64_t len,
                                                          ShiftArgs sa, int32_t *__restrict__ t) {
    constexpr int kWaves = kShiftThreads / kWave;
    __shared__ uint64_t part_max[kWaves], part_sum[kWaves];
    const T *x = X + (int64_t)blockIdx.x * ld;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    uint64_t mx = 0;
    scan_row<T, kShiftThreads>(x, len, [&](double v) {
        const uint64_t b = abs_bits(v);
        mx = b > mx ? b : mx;
    });
    mx = wave_max(mx);
    if (lane == 0) part_max[wave] = mx;
    __syncthreads();
    for (int w = 0; w < kWaves; ++w) mx = part_max[w] > mx ? part_max[w] : mx;
    if (mx == 0) {                                                    // all-zero row
        if (threadIdx.x == 0) t[blockIdx.x] = 0;
        return;
    }
    const int e = floor_log2_of_bits(mx);

    double sum = 0.0;                                                 // exact: see kMaxSquares
    scan_row<T, kShiftThreads>(x, len, [&](double v) {
        const double q = ceil(ldexp(fabs(v), 15 - e));
        sum = fma(q, q, sum);
    });
    const uint64_t s = wave_sum((uint64_t)sum);
    if (lane == 0) part_sum[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t T_ = 0;
        for (int w = 0; w < kWaves; ++w) T_ += part_sum[w];
        t[blockIdx.x] = shift_exponent(T_, sa) - e;
    }
}

template <typename T, int ROUNDS, int KIND>
__global__ __launch_bounds__(256) void k_residues(const T *__restrict__ X, int64_t ld,
                                                  int64_t rows, int64_t len,
                                                  const int32_t *__restrict__ t, ModArgs ma,
                                                  int8_t *__restrict__ out, int64_t rows_pad,
                                                  int64_t len_pad, int64_t rows_stride) {
    residues_block<T, ROUNDS, KIND>(blockIdx.x, X, ld, rows, len, t, ma, out, rows_pad, len_pad, rows_stride);
}

// ----------------------------------------------------------------------------------------
// Shifts of rows of up to 49152 elements, reading each row once: the row is held in registers
// (CH pieces of 8 elements per thread, 8 threads per 64 elements), its maximum and then its
// integer sum of squares come from two workgroup reductions.  Same result as k_shifts, half
// its memory traffic (0.34 against 0.67 ms at 16384^2 FP64; 0.105 against 0.226 ms for 1536 rows of 40000).  (Rows of up to 16384 elements get their
// residues from the same registers, oz2_fused.hip; a workgroup that owns a single longer row would
// write them in 64-byte pieces, which is slower than a kernel of its own.)
// ----------------------------------------------------------------------------------------
template <typename T, int THREADS, int CH>
__global__ __launch_bounds__(THREADS) void k_shifts_cached(const T *__restrict__ X, int64_t ld,
                                                           int64_t len, ShiftArgs sa,
                                                           int32_t *__restrict__ t_out) {
    constexpr int kPer = 8;                                           // elements per piece
    constexpr int kWaves = THREADS / kWave;
    __shared__ uint64_t part[kWaves];
    __shared__ uint64_t bcast;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const T *x = X + (int64_t)blockIdx.x * ld;

    // all loads first (pieces beyond the row's end read its first elements, or nothing if it has no 8)
    constexpr int kVec = 16 / sizeof(T);
    Vec16<T> w[CH][kPer / kVec];
    if (len >= kPer) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int64_t h0 = ((int64_t)c * THREADS + threadIdx.x) * kPer;
            const T *src = h0 + kPer <= len ? x + h0 : x;
#pragma unroll
            for (int i = 0; i < kPer / kVec; ++i) w[c][i] = reinterpret_cast<const Vec16<T> *>(src)[i];
        }
    }
    double v[CH][kPer];
    uint64_t mx = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int64_t h0 = ((int64_t)c * THREADS + threadIdx.x) * kPer;
        const bool whole = h0 + kPer <= len;
#pragma unroll
        for (int i = 0; i < kPer; ++i) v[c][i] = whole ? (double)w[c][i / kVec][i % kVec] : 0.0;
        if (!whole && h0 < len) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) v[c][i] = h0 + i < len ? (double)x[h0 + i] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint64_t bits = abs_bits(v[c][i]);
            mx = bits > mx ? bits : mx;
        }
    }
    mx = wave_max(mx);
    if (lane == 0) part[wave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t m = part[0];
        for (int w = 1; w < kWaves; ++w) m = part[w] > m ? part[w] : m;
        bcast = m;
    }
    __syncthreads();
    mx = bcast;
    if (mx == 0) {                                                    // all-zero row
        if (threadIdx.x == 0) t_out[blockIdx.x] = 0;
        return;
    }
    const int e = floor_log2_of_bits(mx);
    double sum = 0.0;                                                 // exact: see kMaxSquares
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const double q = ceil(ldexp(fabs(v[c][i]), 15 - e));
            sum = fma(q, q, sum);
        }
    const uint64_t s = wave_sum((uint64_t)sum);
    __syncthreads();                                                  // part[] is reused
    if (lane == 0) part[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t T_ = 0;
        for (int w = 0; w < kWaves; ++w) T_ += part[w];
        t_out[blockIdx.x] = shift_exponent(T_, sa) - e;
    }
}

// ----------------------------------------------------------------------------------------
// Epilogue: for each (i, j) read U_s once (or the N int32 products, U_s = mod(C'_s, p_s) by the
// mulhi reduction of Section 4.3), C1 += s_s1 U_s, C2 += s_s2 U_s (s = 1..N, one FMA each),
// Q = rint(P_inv C1), C'' = fma(-P2, Q, fma(-P1, Q, C1) + C2), c = C'' 2^-(tA_i + tB_j).
// One thread per 4 consecutive columns: one 4-byte (uint8 input) or 16-byte (int32 input) load
// per modulus; 8 columns per thread measured slower (2.4 against 1.9 ms at 16384^2, N = 16).
// ----------------------------------------------------------------------------------------
// A thread's place: row i of C and its first column, by a 32-bit division that is a multiplication: a 64-bit
// division and its remainder took about a quarter of a thread's vector instructions.
struct EpiloguePlace {
    int64_t i, j0;
    bool valid;
    __device__ __forceinline__ EpiloguePlace(int64_t m, int groups, Divisor by_groups) {
        const int idx = (int)(blockIdx.x * kEpilogueThreads + threadIdx.x), row = divide(idx, by_groups);
        i = row; j0 = (int64_t)(idx - row * groups) * kEpilogueColumns;
        valid = row < m;
    }
};

// The end of an entry for the four columns of a thread; `old`: C before the call if `beta` needs it and it was
// loaded as 16-byte pieces (whole, aligned groups of columns).
template <typename OutT>
struct EpilogueTail {
    static constexpr int W = kEpilogueColumns, kVec = 16 / sizeof(OutT);
    typedef OutT vec_t __attribute__((ext_vector_type(kVec)));
    OutT *dst;
    int shift[W], columns;
    bool vector;
    vec_t old[W / kVec];
    __device__ __forceinline__ EpilogueTail(const EpiloguePlace &at, int64_t n, const int32_t *tA, const int32_t *tB, double beta,
                                            OutT *C, int64_t ldc) {
        dst = C + at.i * ldc + at.j0;
        columns = n - at.j0 < W ? (int)(n - at.j0) : W;
        vector = columns == W && (reinterpret_cast<uintptr_t>(dst) & 15) == 0;
        const int ta = tA[at.i];
#pragma unroll
        for (int c = 0; c < W; ++c) shift[c] = ta + (c < columns ? tB[at.j0 + c] : 0);
        if (vector && beta != 0.0) {
#pragma unroll
            for (int q = 0; q < W / kVec; ++q) old[q] = reinterpret_cast<const vec_t *>(dst)[q];
        }
    }
    __device__ __forceinline__ void store(const double (&C1)[W], const double (&C2)[W], const ModArgs &ma, double alpha, double beta) {
        if (vector) {
#pragma unroll
            for (int c = 0; c < W; ++c) {
                const OutT before = beta != 0.0 ? old[c / kVec][c % kVec] : OutT(0);
                old[c / kVec][c % kVec] = crt_entry<OutT>(C1[c], C2[c], shift[c], ma, alpha, beta, &before);
            }
#pragma unroll
            for (int q = 0; q < W / kVec; ++q) reinterpret_cast<vec_t *>(dst)[q] = old[q];
        } else {
#pragma unroll
            for (int c = 0; c < W; ++c)
                if (c < columns) dst[c] = crt_entry<OutT>(C1[c], C2[c], shift[c], ma, alpha, beta, dst + c);
        }
    }
};

// The uint8 form for N moduli: everything it reads, C for beta != 0 included, is requested before anything is used.  Bound: HBM
// for large C (8192^2, N = 15, beta = 1: 389 us, 5.3 TB/s).  With groups of 8, 4, 2 and 1 moduli that waited for their loads, C
// read at the end and 64-bit divisions it took 450 us; 4096^2, N = 14, 76 -> 68; 2048^2, N = 15, 20.8 -> 18.8; 1024^2 8.5 -> 7.2.
template <typename OutT, int N>
__global__ __launch_bounds__(kEpilogueThreads) void k_epilogue(const uint8_t *__restrict__ U, int64_t plane, int64_t Np, int64_t m, int64_t n,
                                                  const int32_t *__restrict__ tA, const int32_t *__restrict__ tB, ModArgs ma,
                                                  double alpha, double beta, OutT *C, int64_t ldc, int groups, Divisor by_groups) {
    constexpr int W = kEpilogueColumns;
    const EpiloguePlace at(m, groups, by_groups);
    if (!at.valid) return;
    const uint8_t *u = U + at.i * Np + at.j0;                 // Np is a multiple of 256: aligned, and within the row
    uint32_t x[N];
#pragma unroll
    for (int s = 0; s < N; ++s) { x[s] = *reinterpret_cast<const uint32_t *>(u); u += plane; }
    EpilogueTail<OutT> tail(at, n, tA, tB, beta, C, ldc);
    double C1[W], C2[W];
#pragma unroll
    for (int c = 0; c < W; ++c) C1[c] = C2[c] = 0.0;
    // ascending order of s, in which the accumulation of C'(2) is defined
#pragma unroll
    for (int s = 0; s < N; ++s) {
        const double s1 = ma.s1[s], s2 = ma.s2[s];
#pragma unroll
        for (int c = 0; c < W; ++c) {
            const double v = (double)(int)((x[s] >> (8 * c)) & 0xffu);
            C1[c] = fma(s1, v, C1[c]);
            C2[c] = fma(s2, v, C2[c]);
        }
    }
    tail.store(C1, C2, ma, alpha, beta);
}

// The form for residues of K ranges (launch_int8_gemm), ranges x n planes: U_s is the sum of the ranges' residues modulo p_s, which
// replaces those of the first.  A workgroup owns 256 columns of a row: a thread adds up 16 bytes of a modulus, all ranges requested at
// once, and U_s goes to memory and through LDS to the threads that accumulate, one entry each.
constexpr int kRangeColumns = 256;
template <typename OutT>
__global__ __launch_bounds__(256) void k_epilogue_ranges(uint8_t *U, int64_t plane, int ranges, int64_t Np, int64_t n,
                                                         const int32_t *__restrict__ tA, const int32_t *__restrict__ tB, ModArgs ma,
                                                         double alpha, double beta, OutT *C, int64_t ldc) {
    constexpr int kFlight = 8;
    __shared__ uint4 sum_lds[kMaxModuli][kRangeColumns / 16];
    const int tid = threadIdx.x;
    const int64_t i = blockIdx.y, j0 = (int64_t)blockIdx.x * kRangeColumns, j = j0 + tid;
    uint8_t *const row = U + i * Np + j0;
    const int64_t step = ma.n * plane;
    const int shift = tA[i] + (j < n ? tB[j] : 0);
    for (int q = tid; q < ma.n * (kRangeColumns / 16); q += 256) {
        const int s = q / (kRangeColumns / 16), c = q % (kRangeColumns / 16);
        if (j0 + 16 * c >= n) continue;                       // padding: zero in the first range, not written in the others
        uint8_t *const u = row + s * plane + 16 * c;
        uint4 x = *reinterpret_cast<const uint4 *>(u);
        const int p = ma.p[s];
        for (int z0 = 1; z0 < ranges; z0 += kFlight) {
            uint4 y[kFlight];
#pragma unroll
            for (int z = 0; z < kFlight; ++z)                 // (beyond the last range: it again, not used)
                y[z] = *reinterpret_cast<const uint4 *>(u + (z0 + z < ranges ? z0 + z : ranges - 1) * step);
#pragma unroll
            for (int z = 0; z < kFlight; ++z)
                if (z0 + z < ranges)
                    x = make_uint4(add_mod_bytes(x.x, y[z].x, p), add_mod_bytes(x.y, y[z].y, p), add_mod_bytes(x.z, y[z].z, p),
                                   add_mod_bytes(x.w, y[z].w, p));
        }
        *reinterpret_cast<uint4 *>(u) = x;
        sum_lds[s][c] = x;
    }
    __syncthreads();
    if (j >= n) return;
    const uint8_t *const mine = reinterpret_cast<const uint8_t *>(&sum_lds[0][0]) + tid;
    double C1 = 0.0, C2 = 0.0;
    for (int s = 0; s < ma.n; ++s) {                          // ascending, as everywhere
        const double v = (double)(int)mine[s * kRangeColumns];
        C1 = fma(ma.s1[s], v, C1);
        C2 = fma(ma.s2[s], v, C2);
    }
    OutT *dst = C + i * ldc + j;
    *dst = crt_entry<OutT>(C1, C2, shift, ma, alpha, beta, dst);
}

// The form for int32 sums (possibly folded partial sums), which are reduced here.  Bound: HBM.  Moduli in groups of 8, then 4, 2
// and 1, a group's loads first.  Planes beyond the memory-side cache are read better by fewer wavefronts: LDS that nobody uses keeps
// them to 4 per SIMD there.  us, loops of 4 moduli and single ones at the end | groups | groups, 4 wavefronts: 8192^2 N = 16 980 |
// 972 | 954, 4096^2 N = 14 242 | 241 | 233, with beta = 1 264 | 262 | 255, FP32 N = 8 145 | 144 | 136; from the cache 2048^2 N = 15
// 51 | 52 | 54, 1024^2 15.8 | 15.9 | 15.9.
constexpr int64_t kMemorySideCache = (int64_t)256 << 20;
constexpr unsigned kLdsFor4Waves = 40 * 1024;             // a quarter of a compute unit's, per workgroup of 4 wavefronts
template <typename OutT>
__global__ __launch_bounds__(kEpilogueThreads) void k_epilogue_i32(const int32_t *__restrict__ prod, int64_t plane, int64_t Np, int64_t m,
                                                      int64_t n, const int32_t *__restrict__ tA,
                                                      const int32_t *__restrict__ tB, ModArgs ma, double alpha, double beta,
                                                      OutT *C, int64_t ldc, int groups, Divisor by_groups) {
    constexpr int W = kEpilogueColumns;
    const EpiloguePlace at(m, groups, by_groups);
    if (!at.valid) return;
    const int32_t *u = prod + at.i * Np + at.j0;
    double C1[W], C2[W];
#pragma unroll
    for (int c = 0; c < W; ++c) C1[c] = C2[c] = 0.0;
    // moduli s0 .. s0 + CNT - 1, the FMAs in ascending order of s
    auto group = [&](int s0, auto cnt) {
        constexpr int CNT = decltype(cnt)::value;
        int4 x[CNT];
#pragma unroll
        for (int g = 0; g < CNT; ++g) x[g] = *reinterpret_cast<const int4 *>(u + (s0 + g) * plane);
#pragma unroll
        for (int g = 0; g < CNT; ++g) {
            const int p = ma.p[s0 + g], pv = (int)ma.pinv_prime[s0 + g];
            const int us[W] = {mod_small(x[g].x, p, pv), mod_small(x[g].y, p, pv), mod_small(x[g].z, p, pv), mod_small(x[g].w, p, pv)};
            const double s1 = ma.s1[s0 + g], s2 = ma.s2[s0 + g];
#pragma unroll
            for (int c = 0; c < W; ++c) {
                C1[c] = fma(s1, (double)us[c], C1[c]);
                C2[c] = fma(s2, (double)us[c], C2[c]);
            }
        }
    };
    int s = 0;
    for (; s + 8 <= ma.n; s += 8) group(s, std::integral_constant<int, 8>{});
    if (s + 4 <= ma.n) { group(s, std::integral_constant<int, 4>{}); s += 4; }
    if (s + 2 <= ma.n) { group(s, std::integral_constant<int, 2>{}); s += 2; }
    if (s < ma.n) group(s, std::integral_constant<int, 1>{});
    EpilogueTail<OutT>(at, n, tA, tB, beta, C, ldc).store(C1, C2, ma, alpha, beta);
}

template <typename OutT, int N>
hipError_t launch_epilogue_u8(const uint8_t *U, int64_t plane, int64_t Np, int64_t m, int64_t n, const int32_t *tA,
                              const int32_t *tB, const ModArgs &ma, double alpha, double beta, OutT *C, int64_t ldc, int groups,
                              unsigned blocks, hipStream_t stream) {
    if constexpr (N <= kMaxModuli) {
        if (ma.n != N)
            return launch_epilogue_u8<OutT, N + 1>(U, plane, Np, m, n, tA, tB, ma, alpha, beta, C, ldc, groups, blocks, stream);
        hipLaunchKernelGGL((k_epilogue<OutT, N>), dim3(blocks), dim3(kEpilogueThreads), 0, stream, U, plane, Np, m, n, tA, tB, ma, alpha, beta, C,
                           ldc, groups, make_divisor(groups));
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

template <typename OutT>
__global__ __launch_bounds__(256) void k_scale_c(OutT *C, int64_t ldc, int64_t m, int64_t n,
                                                 double beta) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= m * n) return;
    OutT *dst = C + (idx / n) * ldc + idx % n;
    *dst = (beta == 0.0) ? OutT(0) : (OutT)(beta * (double)*dst);
}

inline unsigned blocks_for(int64_t threads) { return (unsigned)((threads + 255) / 256); }

}  // namespace

template <typename T>
hipError_t launch_shifts(const T *X, int64_t ld, int64_t rows, int64_t len, const ShiftArgs &sa,
                         int32_t *t, hipStream_t stream) {
    // rows of up to 49152 elements are read once (pieces of 8 elements: 128 threads hold 1024
    // elements per piece, 512 threads 4096, 1024 threads 8192); longer rows are read twice
    auto cached = [&](auto threads, auto ch) {
        hipLaunchKernelGGL((k_shifts_cached<T, decltype(threads)::value, decltype(ch)::value>), dim3((unsigned)rows),
                           dim3(decltype(threads)::value), 0, stream, X, ld, len, sa, t);
    };
    using std::integral_constant;
    if (len <= 1024) cached(integral_constant<int, 128>{}, integral_constant<int, 1>{});
    else if (len <= 2048) cached(integral_constant<int, 128>{}, integral_constant<int, 2>{});
    else if (len <= 4096) cached(integral_constant<int, 512>{}, integral_constant<int, 1>{});
    else if (len <= 8192) cached(integral_constant<int, 512>{}, integral_constant<int, 2>{});
    else if (len <= 12288) cached(integral_constant<int, 512>{}, integral_constant<int, 3>{});
    else if (len <= 16384) cached(integral_constant<int, 512>{}, integral_constant<int, 4>{});
    else if (len <= 24576) cached(integral_constant<int, 1024>{}, integral_constant<int, 3>{});
    else if (len <= 32768) cached(integral_constant<int, 1024>{}, integral_constant<int, 4>{});
    else if (len <= 40960) cached(integral_constant<int, 1024>{}, integral_constant<int, 5>{});
    else if (len <= 49152) cached(integral_constant<int, 1024>{}, integral_constant<int, 6>{});
    else hipLaunchKernelGGL((k_shifts<T>), dim3((unsigned)rows), dim3(kShiftThreads), 0, stream, X, ld, len, sa, t);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_residues(const T *X, int64_t ld, int64_t rows, int64_t len, const int32_t *t,
                           const ModArgs &ma, int8_t *out, int64_t rows_pad, int64_t len_pad,
                           hipStream_t stream, int64_t rows_stride) {
    if (rows_stride == 0) rows_stride = rows_pad;
    const int64_t threads = rows_pad * (len_pad / kResPerThread);
    if (ma.rounds == 1)
        hipLaunchKernelGGL((k_residues<T, 1, 0>), dim3(blocks_for(threads)), dim3(256), 0, stream, X,
                           ld, rows, len, t, ma, out, rows_pad, len_pad, rows_stride);
    else
        hipLaunchKernelGGL((k_residues<T, 2, 0>), dim3(blocks_for(threads)), dim3(256), 0, stream, X,
                           ld, rows, len, t, ma, out, rows_pad, len_pad, rows_stride);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_magnitudes(const T *X, int64_t ld, int64_t rows, int64_t len, const int32_t *pre,
                             int8_t *out, int64_t rows_pad, int64_t len_pad, hipStream_t stream) {
    const int64_t threads = rows_pad * (len_pad / kResPerThread);
    ModArgs none{};
    hipLaunchKernelGGL((k_residues<T, 1, 1>), dim3(blocks_for(threads)), dim3(256), 0, stream, X, ld,
                       rows, len, pre, none, out, rows_pad, len_pad, rows_pad);
    return hipGetLastError();
}

template <typename OutT>
hipError_t launch_epilogue(void *prod, bool prod_is_u8, int64_t Mp, int64_t Np, int64_t m,
                           int64_t n, const int32_t *tA, const int32_t *tB, const ModArgs &ma,
                           double alpha, double beta, OutT *C, int64_t ldc, hipStream_t stream, int ranges) {
    const int64_t groups = epilogue_groups(n), plane = Mp * Np, rows = epilogue_rows(groups);
    if (rows < 1) return hipErrorInvalidValue;
    for (int64_t r = 0; r < m; r += rows) {
        const int64_t count = std::min(rows, m - r);
        const unsigned blocks = (unsigned)((count * groups + kEpilogueThreads - 1) / kEpilogueThreads);
        hipError_t e;
        if (ranges > 1) {
            const int64_t most = 65535;                       // rows of a grid
            e = hipSuccess;
            for (int64_t q = 0; q < count && e == hipSuccess; q += most) {
                hipLaunchKernelGGL((k_epilogue_ranges<OutT>), dim3((unsigned)((n + kRangeColumns - 1) / kRangeColumns), (unsigned)std::min(most, count - q)),
                                   dim3(256), 0, stream, static_cast<uint8_t *>(prod) + (r + q) * Np, plane, ranges, Np, n, tA + r + q, tB, ma,
                                   alpha, beta, C + (r + q) * ldc, ldc);
                e = hipGetLastError();
            }
        } else if (prod_is_u8) {
            e = launch_epilogue_u8<OutT, OZ2_MIN_MODULI>(static_cast<const uint8_t *>(prod) + r * Np, plane, Np, count, n, tA + r, tB, ma,
                                                         alpha, beta, C + r * ldc, ldc, (int)groups, blocks, stream);
        } else {
            const unsigned lds_bytes = 4 * ma.n * plane > kMemorySideCache ? kLdsFor4Waves : 0;
            hipLaunchKernelGGL((k_epilogue_i32<OutT>), dim3(blocks), dim3(kEpilogueThreads), lds_bytes, stream,
                               static_cast<const int32_t *>(prod) + r * Np, plane, Np, count, n, tA + r, tB, ma, alpha, beta,
                               C + r * ldc, ldc, (int)groups, make_divisor((int)groups));
            e = hipGetLastError();
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename OutT>
hipError_t launch_scale_c(OutT *C, int64_t ldc, int64_t m, int64_t n, double beta,
                          hipStream_t stream) {
    hipLaunchKernelGGL((k_scale_c<OutT>), dim3(blocks_for(m * n)), dim3(256), 0, stream, C, ldc, m,
                       n, beta);
    return hipGetLastError();
}

#define OZ2_INSTANTIATE(T)                                                                        \
    template hipError_t launch_shifts<T>(const T *, int64_t, int64_t, int64_t, const ShiftArgs &, \
                                         int32_t *, hipStream_t);                                 \
    template hipError_t launch_magnitudes<T>(const T *, int64_t, int64_t, int64_t,               \
                                             const int32_t *, int8_t *, int64_t, int64_t,        \
                                             hipStream_t);                                        \
    template hipError_t launch_residues<T>(const T *, int64_t, int64_t, int64_t, const int32_t *, \
                                           const ModArgs &, int8_t *, int64_t, int64_t,           \
                                           hipStream_t, int64_t);                                 \
    template hipError_t launch_epilogue<T>(void *, bool, int64_t, int64_t, int64_t,              \
                                           int64_t, const int32_t *, const int32_t *,             \
                                           const ModArgs &, double, double, T *, int64_t,         \
                                           hipStream_t, int);                                          \
    template hipError_t launch_scale_c<T>(T *, int64_t, int64_t, int64_t, double, hipStream_t);
OZ2_INSTANTIATE(double)
OZ2_INSTANTIATE(float)

}  // namespace oz2
