// Accurate mode of Section 4.2: the scale vectors come from the row and column maxima of
// Cbar = Abar * Bbar, where Abar = ceil(mu' |A|) and Bbar = ceil(|B| nu') are 7-bit
// matrices (mu'_i = 2^(5 - floor(log2 max_h |a_ih|)), likewise nu'_j) and the product runs
// on the INT8 matrix cores like every other slice.  Everything here is integer or exact
// power-of-two arithmetic, so the shifts are bit-reproducible; the floor(P'_accu - 0.51 log2 c)
// of the paper is a table lookup on the integer maximum c (built on the host from that
// formula, see oz2_constants.cpp).
#include "oz2_convert.hpp"
#include "oz2_kernels.hpp"

namespace oz2 {
namespace {

// rowmax[r] = max_h bits(|X[r][h]|): one workgroup per row.
constexpr int kRowThreads = 512;
template <typename T>
__global__ __launch_bounds__(kRowThreads) void k_row_maxbits(const T *__restrict__ X, int64_t ld,
                                                             int64_t len, unsigned long long *rowmax) {
    __shared__ uint64_t part[kRowThreads / dev::kWave];
    uint64_t mx = 0;
    dev::scan_row<T, kRowThreads>(X + (int64_t)blockIdx.x * ld, len, [&](double v) {
        const uint64_t b = dev::abs_bits(v);
        mx = b > mx ? b : mx;
    });
    mx = dev::wave_max(mx);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kRowThreads / dev::kWave; ++w) mx = part[w] > mx ? part[w] : mx;
        rowmax[blockIdx.x] = mx;
    }
}

// pre[v] = 5 - floor(log2 max) (0 for an all-zero vector: its magnitudes are all 0 anyway), for
// the vectors of one factor; also clears their maxima of Cbar for every K range, `stride` apart (a
// kernel, not a memset: the call may be captured into a HIP graph).
__global__ __launch_bounds__(256) void k_preshift(const unsigned long long *__restrict__ maxbits,
                                                  int64_t vecs, int64_t stride, int ranges,
                                                  int32_t *__restrict__ pre, int32_t *__restrict__ cmax) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= vecs) return;
    const uint64_t b = maxbits[i];
    pre[i] = b ? 5 - floor_log2_of_bits(b) : 0;
    for (int r = 0; r < ranges; ++r) cmax[r * stride + i] = 0;
}

// t[v] = (5 - e_v) + floor(P'_accu - 0.51 log2 max(c_v, 1)) with c_v the sum over the K ranges of
// the maxima of Cbar_r (Section 4.2; for a contraction of more than 2^17 the sum bounds the
// maximum of the whole Cbar from above, Section 4.3); an all-zero vector gets 0.
// Entries [0, m) are the rows of A, [m, count) the columns of B (the arrays adjoin).
__global__ __launch_bounds__(256) void k_accu_finish(const unsigned long long *__restrict__ maxbits,
                                                     const int32_t *__restrict__ cmax, int64_t m,
                                                     int64_t count, int ranges, ShiftArgs sa,
                                                     int32_t *__restrict__ tA, int32_t *__restrict__ tB) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    int32_t *t = i < m ? tA + i : tB + (i - m);
    const uint64_t b = maxbits[i];
    if (b == 0) { *t = 0; return; }
    uint64_t c = 0;
    for (int r = 0; r < ranges; ++r) c += (uint64_t)cmax[r * count + i];   // each in [0, 2^29]
    if (c == 0) c = 1;
    int j = 0;
    while (j < sa.levels - 1 && c > sa.theta[j]) ++j;
    *t = (5 - floor_log2_of_bits(b)) + (sa.f_max - j);
}

struct Scratch {
    unsigned long long *amax, *bmax;     // bits of max |.| per row of A / column of B
    int32_t *preA, *preB;                // 5 - e
    int32_t *cmax;                       // maxima of Cbar_r: [range][m row maxima | n column maxima]
};

Scratch carve(void *scratch, int64_t m, int64_t n) {
    Scratch s;
    s.amax = static_cast<unsigned long long *>(scratch);
    s.bmax = s.amax + m;
    s.preA = reinterpret_cast<int32_t *>(s.bmax + n);
    s.preB = s.preA + m;
    s.cmax = s.preB + n;
    return s;
}

inline unsigned blocks_for(int64_t threads) { return (unsigned)((threads + 255) / 256); }

}  // namespace

template <typename T>
hipError_t launch_accurate_prescale(const T *A, int64_t lda, bool a_k_contiguous, const T *B,
                                    int64_t ldb, bool b_k_contiguous, int64_t m, int64_t n,
                                    int64_t k, int ranges, void *scratch, int8_t *Abar, int8_t *Bbar,
                                    int64_t Mp, int64_t Np, int64_t Kp, bool fused, hipStream_t stream) {
    if (ranges < 1 || ranges > kMaxKRanges) return hipErrorInvalidValue;
    const Scratch s = carve(scratch, m, n);
    // Factors whose vectors fit a workgroup: everything in one launch for both.
    const bool use[2] = {fused && fused_applies(Kp, a_k_contiguous), fused && fused_applies(Kp, b_k_contiguous)};
    if (use[0] || use[1]) {
        const FusedFactor<T> fa{use[0] ? A : nullptr, lda, a_k_contiguous, m, k, s.preA, Abar, Mp, Kp, s.amax, s.cmax, m + n, ranges};
        const FusedFactor<T> fb{use[1] ? B : nullptr, ldb, b_k_contiguous, n, k, s.preB, Bbar, Np, Kp, s.bmax, s.cmax + m, m + n, ranges};
        if (hipError_t e = launch_fused_magnitudes<T>(fa, fb, stream)) return e;
    }
    // The others: maxima, then pre-shifts (and the cleared maxima of Cbar), then magnitudes.  A vector of
    // the product (a row of op(A), a column of op(B)) is either contiguous in memory (one workgroup per
    // vector) or strided by the leading dimension (column kernels).
    auto general = [&](const T *X, int64_t ld, bool k_contiguous, int64_t vecs, unsigned long long *maxbits, int32_t *pre,
                       int32_t *cmax, int8_t *out, int64_t vecs_pad) -> hipError_t {
        if (k_contiguous)
            hipLaunchKernelGGL((k_row_maxbits<T>), dim3((unsigned)vecs), dim3(kRowThreads), 0, stream, X, ld, k,
                               maxbits);
        else if (hipError_t e = launch_col_maxbits<T>(X, ld, k, vecs, maxbits, stream)) return e;
        hipLaunchKernelGGL(k_preshift, dim3(blocks_for(vecs)), dim3(256), 0, stream, maxbits, vecs, m + n, ranges, pre, cmax);
        return k_contiguous ? launch_magnitudes<T>(X, ld, vecs, k, pre, out, vecs_pad, Kp, stream)
                            : launch_magnitudes_cols<T>(X, ld, k, vecs, pre, out, vecs_pad, Kp, stream);
    };
    if (!use[0])
        if (hipError_t e = general(A, lda, a_k_contiguous, m, s.amax, s.preA, s.cmax, Abar, Mp)) return e;
    return use[1] ? hipSuccess : general(B, ldb, b_k_contiguous, n, s.bmax, s.preB, s.cmax + m, Bbar, Np);
}

void accurate_maxima(void *scratch, int64_t m, int64_t n, int range, int **row_max, int **col_max) {
    const Scratch s = carve(scratch, m, n);
    *row_max = s.cmax + (int64_t)range * (m + n);
    *col_max = *row_max + m;
}

hipError_t launch_accurate_finish(int64_t m, int64_t n, int ranges, const ShiftArgs &sa, void *scratch,
                                  int32_t *tA, int32_t *tB, hipStream_t stream) {
    if (ranges < 1 || ranges > kMaxKRanges) return hipErrorInvalidValue;
    const Scratch s = carve(scratch, m, n);
    hipLaunchKernelGGL(k_accu_finish, dim3(blocks_for(m + n)), dim3(256), 0, stream, s.amax, s.cmax, m, m + n,
                       ranges, sa, tA, tB);
    return hipGetLastError();
}

template hipError_t launch_accurate_prescale<double>(const double *, int64_t, bool, const double *, int64_t,
                                                     bool, int64_t, int64_t, int64_t, int, void *, int8_t *,
                                                     int8_t *, int64_t, int64_t, int64_t, bool, hipStream_t);
template hipError_t launch_accurate_prescale<float>(const float *, int64_t, bool, const float *, int64_t,
                                                    bool, int64_t, int64_t, int64_t, int, void *, int8_t *,
                                                    int8_t *, int64_t, int64_t, int64_t, bool, hipStream_t);

}  // namespace oz2
