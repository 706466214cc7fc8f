// Algorithm 1 lines 1-5 in one launch and one read of the operands: scale vector and residues.
// A workgroup owns whole vectors (V rows, or a strip of V columns, of a factor) and keeps them in
// registers between the three things that are done to them: the maximum of |x|, the exact sum of
// squares behind the shift (fast mode of Section 4.2), and the reduction modulo all N moduli.  The
// general kernels (oz2_prepost.hip, oz2_columns.hip) do these in two or three launches and two or three
// reads; their results are the same bit for bit.  fused_plan (oz2_plan.hpp) says which vectors fit.
//
// Layout: after the load, thread `tid` holds in piece c the 8 consecutive elements of number
//   q = c THREADS + tid = ((kb V + vec) 8 + piece),  element h = 64 kb + 8 piece + {0..7} of vector vec,
// so that the 8-byte pieces of residues which a wavefront stores are 512 contiguous bytes of the K-blocked
// slice (for V >= 8).  Rows are loaded that way directly.  A strip of columns is loaded along its rows
// (64-byte segments for V = 8 in FP64) and exchanged through LDS, once per element and not once per
// modulus.
//
// KIND 1 is the first half of accurate mode: the maximum, the pre-shift 5 - e and the 7-bit magnitudes
// ceil(|x| 2^(5-e)) (slice 0); the maxima of Cbar are cleared on the way.
//
// Bound: HBM (reads and N bytes per element written) for large vectors, launch and load latency for
// small ones.
#include <algorithm>

#include "oz2_convert.hpp"
#include "oz2_kernels.hpp"

namespace oz2 {
namespace {

using namespace dev;

constexpr int kMaxLogV = 5;

template <typename T>
struct Side {
    const T *X;
    int64_t ld, vecs, len;      // `vecs` vectors of `len` elements: X[v ld + h] (k_contiguous) or X[h ld + v]
    int32_t *t;                 // [vecs] shifts (KIND 1: pre-shifts)
    unsigned long long *maxbits;   // KIND 1: [vecs] bits of max |x|
    int32_t *cmax;              // KIND 1: [ranges][cmax_stride], cleared
    int64_t cmax_stride;
    int8_t *out;                // slices [N][len_pad/64][vecs_pad][64]
    int64_t vecs_pad, len_pad;
    int ranges;
    int k_contiguous, log_v;    // vectors per workgroup = 2^log_v
    unsigned blocks;            // workgroups of this side
};

// SPLIT: workgroup row y of the launch produces the moduli of group y only.
template <typename T, int THREADS, int CH, int ROUNDS, int KIND, bool SPLIT>
__global__ __launch_bounds__(THREADS) void k_convert(Side<T> a, Side<T> b, ShiftArgs sa, ModArgs ma) {
    __shared__ T tile[THREADS * 9];                                   // one piece per thread, padded (columns only)
    __shared__ unsigned long long red_max[1 << kMaxLogV], red_sum[1 << kMaxLogV];
    const bool first = blockIdx.x < a.blocks;
    const Side<T> s = first ? a : b;
    unsigned blk = first ? blockIdx.x : blockIdx.x - a.blocks;
    // Workgroups go to the 8 XCDs round-robin: neighbouring vectors, which share 128-byte lines of the
    // operand (strips of columns) or of the slices (single rows), are given to one XCD.
    if ((s.blocks & 7u) == 0) blk = (blk & 7u) * (s.blocks >> 3) + (blk >> 3);
    const int tid = threadIdx.x, lane = tid & 63, lv = s.log_v, V = 1 << lv;
    const int64_t v0 = (int64_t)blk << lv;
    const int vec = (tid >> 3) & (V - 1), piece = tid & 7;
    const bool valid = v0 + vec < s.vecs;
    if (tid < V) { red_max[tid] = 0; red_sum[tid] = 0; }

    double x[CH][8];
    const int kb0 = tid >> (3 + lv), kb_step = THREADS >> (3 + lv);   // K block of piece c: kb0 + c kb_step
    if (s.k_contiguous) {
        // All whole pieces are requested before anything is done with them: no branch around a load (pieces
        // that are not whole read the first row instead, whose first 8 elements exist if len >= 8), and
        // 16-byte loads at element alignment, which the hardware takes.  The piece that holds a row's end
        // follows, element by element; a masked load per element cost eight waits for memory per
        // wavefront (500 x 300 x 777 in FP32: 10.5 us of conversion, 9.5 us this way).
        constexpr int kVec = 16 / sizeof(T);
        const T *row = s.X + (valid ? v0 + vec : 0) * s.ld;
        Vec16<T> w[CH][8 / kVec];
        if (s.len >= 8) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int64_t h0 = (int64_t)(kb0 + c * kb_step) * kBlockK + piece * 8;
                const T *src = h0 + 8 <= s.len ? row + h0 : s.X;
#pragma unroll
                for (int i = 0; i < 8 / kVec; ++i) w[c][i] = reinterpret_cast<const Vec16<T> *>(src)[i];
            }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int64_t h0 = (int64_t)(kb0 + c * kb_step) * kBlockK + piece * 8;
            const bool whole = valid && h0 + 8 <= s.len;
#pragma unroll
            for (int i = 0; i < 8; ++i) x[c][i] = whole ? (double)w[c][i / kVec][i % kVec] : 0.0;
            if (valid && h0 < s.len && !whole) {
                T last[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) last[i] = row[h0 + i < s.len ? h0 + i : h0];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[c][i] = h0 + i < s.len ? (double)last[i] : 0.0;
            }
        }
    } else {
        // thread -> column tid & (V - 1) and, a constant stride apart, the rows (tid >> lv) + j (THREADS >> lv)
        const int col = tid & (V - 1), step = THREADS >> lv;
        const T *src = s.X + v0 + col + (int64_t)(tid >> lv) * s.ld;
        const int64_t src_step = step * s.ld;
        T raw[CH][8];
        int left = v0 + col < s.vecs ? (int)s.len - (tid >> lv) : 0;  // rows from this thread's to the last
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                raw[c][i] = left > 0 ? *src : T(0);
                src += src_step;
                left -= step;
            }
        const int group = 9 * V;                                      // 8 rows of V elements, and V of padding
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int r = (i * THREADS + tid) >> lv;
                tile[(r >> 3) * group + (r & 7) * V + col] = raw[c][i];
            }
            __syncthreads();
            const T *mine = tile + (kb0 * 8 + piece) * group + vec;
#pragma unroll
            for (int i = 0; i < 8; ++i) x[c][i] = (double)mine[i * V];
        }
    }

    // maximum of |x| per vector
    uint64_t mx = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint64_t bits = abs_bits(x[c][i]);
            mx = bits > mx ? bits : mx;
        }
    auto over_lanes = [&](auto op, uint64_t v) {                      // lanes of this wavefront with the same vector
        v = op(v, dpp64<kDppXor1>(v));
        v = op(v, dpp64<kDppXor2>(v));
        v = op(v, dpp64<kDppMirror8>(v));
        if (lv < 1) v = op(v, dpp64<kDppMirror16>(v));
        if (lv < 2) v = op(v, (uint64_t)__shfl_xor(v, 16, kWave));
        if (lv < 3) v = op(v, (uint64_t)__shfl_xor(v, 32, kWave));
        return v;
    };
    const bool leader = piece == 0 && (lane >> (3 + lv)) == 0;        // one lane per wavefront and vector
    mx = over_lanes([](uint64_t p, uint64_t q) { return p > q ? p : q; }, mx);
    __syncthreads();                                                  // red_max is cleared
    if (leader) atomicMax(&red_max[vec], (unsigned long long)mx);
    __syncthreads();
    mx = red_max[vec];
    const int e = mx ? floor_log2_of_bits(mx) : 0;
    const bool writes = tid < 8 * V && piece == 0 && valid;           // one thread per vector

    if (KIND == 1) {
        const int pre = mx ? 5 - e : 0;
        if (writes) {
            s.maxbits[v0 + vec] = mx;
            s.t[v0 + vec] = pre;
            for (int r = 0; r < s.ranges; ++r) s.cmax[r * s.cmax_stride + v0 + vec] = 0;
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int64_t kb = kb0 + c * kb_step;
            if (kb * kBlockK >= s.len_pad) continue;
            uint32_t w[2] = {0u, 0u};
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w[i >> 2] |= ((uint32_t)(int)ceil(ldexp(fabs(x[c][i]), pre)) & 0xffu) << (8 * (i & 3));
            *reinterpret_cast<uint2 *>(s.out + (kb * s.vecs_pad + v0 + vec) * kBlockK + piece * 8) = make_uint2(w[0], w[1]);
        }
        return;
    }

    // T = sum of ceil(|x| 2^(15-e))^2: integers of at most 2^32, whose sum FP64 holds exactly (kMaxSquares)
    double sum = 0.0;
    if (mx) {
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const double q = ceil(ldexp(fabs(x[c][i]), 15 - e));
                sum = fma(q, q, sum);
            }
    }
    const uint64_t part = over_lanes([](uint64_t p, uint64_t q) { return p + q; }, (uint64_t)sum);
    if (leader) atomicAdd(&red_sum[vec], (unsigned long long)part);
    __syncthreads();
    const int t = mx ? shift_exponent(red_sum[vec], sa) - e : 0;
    if (writes && (!SPLIT || blockIdx.y == 0)) s.t[v0 + vec] = t;

    const int64_t plane = s.vecs_pad * s.len_pad;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int64_t kb = kb0 + c * kb_step;
        if (kb * kBlockK >= s.len_pad) continue;
        int8_t *o = s.out + (kb * s.vecs_pad + v0 + vec) * kBlockK + piece * 8;
        double v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = trunc(ldexp(x[c][i], t));
        const int first = SPLIT ? (int)blockIdx.y * kModGroup : 0, end = SPLIT ? first + 1 : ma.n;
        for (int s0 = first; s0 < end; s0 += kModGroup) {
            ResidueInput in;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                in.y[i] = ROUNDS == 2 ? group_reduce(v[i], ma.group_mod[s0 / kModGroup], ma.group_inv[s0 / kModGroup]) : v[i];
            in.set_low();
            emit_group(in, ma, s0, ma.n, [&](int m, uint2 w) { *reinterpret_cast<uint2 *>(o + (int64_t)m * plane) = w; });
        }
    }
}

template <typename T>
Side<T> side_of(const FusedFactor<T> &f, const FusedPlan &plan) {
    Side<T> s{};
    if (!f.X) return s;                                               // no workgroups
    s.X = f.X; s.ld = f.ld; s.vecs = f.vecs; s.len = f.len; s.t = f.t; s.maxbits = f.maxbits;
    s.cmax = f.cmax; s.cmax_stride = f.cmax_stride; s.ranges = f.ranges;
    s.out = f.out; s.vecs_pad = f.vecs_pad; s.len_pad = f.len_pad;
    s.k_contiguous = f.k_contiguous ? 1 : 0;
    s.log_v = plan.log_v;
    s.blocks = (unsigned)(f.vecs_pad >> s.log_v);
    return s;
}

template <typename T, int ROUNDS, int KIND>
hipError_t launch_kind(const FusedFactor<T> &A, const FusedFactor<T> &B, const ShiftArgs &sa, const ModArgs &ma,
                       hipStream_t stream) {
    const int64_t Kp = A.X ? A.len_pad : B.len_pad;
    const bool strips = (A.X && !A.k_contiguous) || (B.X && !B.k_contiguous);
    if (A.X && B.X && A.k_contiguous != B.k_contiguous && Kp > kFusedShareLaunch) {
        const FusedFactor<T> none{};
        if (hipError_t e = launch_kind<T, ROUNDS, KIND>(A, none, sa, ma, stream)) return e;
        return launch_kind<T, ROUNDS, KIND>(none, B, sa, ma, stream);
    }
    const FusedPlan plan = fused_plan(Kp, strips, (A.X ? A.vecs_pad : 0) + (B.X ? B.vecs_pad : 0), sizeof(T));
    const Side<T> a = side_of(A, plan), b = side_of(B, plan);
    // The smallest launches leave compute units idle while each thread walks through all moduli: where there is one for
    // each, every group of moduli gets workgroups of its own, which read the operands again, from the caches (whole calls
    // repeated in a graph, other operands in each, us, all else as it is: 256^3 N = 14 12.9 -> 11.9, 64^3 N = 15 11.5 -> 10.7, 200^3
    // N = 15 13.6 -> 12.9, 100 x 90 x 200 N = 18 13.4 -> 12.2, 128^3 FP32 N = 8 8.9 -> 8.7).
    const unsigned blocks = a.blocks + b.blocks, groups = (unsigned)((ma.n + kModGroup - 1) / kModGroup);
    if constexpr (KIND == 0) {
        if (fused_split_applies(plan, blocks, groups)) {
            hipLaunchKernelGGL((k_convert<T, kFusedSplitThreads, kFusedSplitPieces, ROUNDS, KIND, true>), dim3(blocks, groups),
                               dim3(kFusedSplitThreads), 0, stream, a, b, sa, ma);
            return hipGetLastError();
        }
    }
    const dim3 grid(blocks);
#define OZ2_CONVERT(THREADS, CH)                                                                              \
    if (plan.threads == THREADS && plan.pieces == CH) {                                                       \
        hipLaunchKernelGGL((k_convert<T, THREADS, CH, ROUNDS, KIND, false>), grid, dim3(THREADS), 0, stream, a, b, sa, ma); \
        return hipGetLastError();                                                                             \
    }
    OZ2_CONVERT(256, 1) OZ2_CONVERT(512, 1) OZ2_CONVERT(512, 2) OZ2_CONVERT(512, 3) OZ2_CONVERT(512, 4)
    OZ2_CONVERT(1024, 3) OZ2_CONVERT(1024, 4)
#undef OZ2_CONVERT
    return hipErrorInvalidValue;
}

}  // namespace

template <typename T>
hipError_t launch_fused_conversion(const FusedFactor<T> &A, const FusedFactor<T> &B, const ShiftArgs &sa,
                                   const ModArgs &ma, hipStream_t stream) {
    return ma.rounds == 1 ? launch_kind<T, 1, 0>(A, B, sa, ma, stream) : launch_kind<T, 2, 0>(A, B, sa, ma, stream);
}

template <typename T>
hipError_t launch_fused_magnitudes(const FusedFactor<T> &A, const FusedFactor<T> &B, hipStream_t stream) {
    return launch_kind<T, 1, 1>(A, B, ShiftArgs{}, ModArgs{}, stream);
}

#define OZ2_INSTANTIATE_FUSED(T)                                                                              \
    template hipError_t launch_fused_conversion<T>(const FusedFactor<T> &, const FusedFactor<T> &,            \
                                                   const ShiftArgs &, const ModArgs &, hipStream_t);          \
    template hipError_t launch_fused_magnitudes<T>(const FusedFactor<T> &, const FusedFactor<T> &, hipStream_t);
OZ2_INSTANTIATE_FUSED(double)
OZ2_INSTANTIATE_FUSED(float)

}  // namespace oz2
