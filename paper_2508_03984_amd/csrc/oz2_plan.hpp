// Host-side planning of a product call: argument checks, the workspace layout, how C is cut
// into panels when the workspace is bounded, and the rules that pick a form of the call.
// Plain C++ with no dependency on the HIP runtime, so that it can be built and exercised on the
// CPU (also under sanitizers); the entry points in oz2_api.hip apply it unchanged.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "../../include/oz2.h"

namespace oz2 {

// Tile granularity the INT8 GEMM assumes for its padded operands.
constexpr int64_t kPadMN = 256;   // rows of the A slices, rows of the B^T slices
constexpr int64_t kPadK = 128;    // contraction length
constexpr int kBlockK = 64;       // K block of the residue-slice layout [Kp/64][rows][64]
// K ranges of a blocked contraction (Section 4.3, last sentence): at most this many of OZ2_MAX_K.
constexpr int kMaxKRanges = OZ2_MAX_K_BLOCKED / OZ2_MAX_K;

inline int64_t round_up(int64_t x, int64_t to) { return (x + to - 1) / to * to; }
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Scratch of accurate mode: per row of A and column of B the bits of max |.| (8 bytes), the
// pre-shift (4) and one maximum of Cbar per K range (4 each).
inline size_t accurate_scratch_bytes(int64_t m, int64_t n) { return (size_t)(m + n) * (12 + 4 * kMaxKRanges); }

// Shapes whose residues of both factors come from one launch once the shifts are known (accurate mode, oz2_small.hip):
// both operands within 2 x 2048^2 elements, so that they and their slices sit in the caches.
inline bool small_conversion_applies(int64_t m, int64_t n, int64_t k) {
    return k <= 4096 && m <= 8192 && n <= 8192 && (m + n) * k <= (int64_t)2 * 2048 * 2048;
}

// The fused conversion (oz2_fused.hip): a workgroup of `threads` threads holds 8 `pieces` elements per
// thread, i.e. 2^log_v whole vectors of Kp elements.
struct FusedPlan {
    int threads, pieces, log_v;
};
constexpr int64_t kFusedElements = 32768;  // 1024 threads, 4 pieces
constexpr int64_t kFusedMaxRow = kFusedElements / 2, kFusedMaxColumn = kFusedElements / 8;

// Rows of up to 16384 elements (two per workgroup: 128-byte lines of the slices; one per workgroup measured
// 1.8 ms for 2^28 elements and 15 moduli against 1.6 ms for the general kernels) and columns of up to
// 4096 (eight per workgroup: 64-byte segments of the operand in FP64).
inline bool fused_applies(int64_t Kp, bool k_contiguous) { return Kp <= (k_contiguous ? kFusedMaxRow : kFusedMaxColumn); }

// For many vectors the smallest workgroup with room for two rows (four of up to 1024 elements) or eight columns; strips of
// columns of more than 1024 elements take 16 where they fit.  Measured (us, both factors, N = 15 in FP64): rows of 4096, 4096^2
// each, 512 threads and 2 rows 148, 1024 threads and 8 rows 171 (several workgroups per compute
// unit overlap one's loads with another's stores); columns of 2048, 2048^2 each, 16 per workgroup 42, 8 52;
// columns of 1024, 1024^2 each, 8 per workgroup 16.8, 16 21.4.  Columns of up to 1024 in FP64 go by 4 while the launch has
// few workgroups, two of which then overlap on a compute unit (conversion stage, N = 15, us, by 8 | by 4: 1024 x 1024 x 1024 21.7 |
// 20.4, 1500 x 1500 x 1000 25.2 | 23.7, 2500 x 2500 x 1024 41.2 | 37.8; 4096 x 4096 x 1024 53.0 | 54.1, 8192 x 8192 x 512 46.4 | 47.6;
// FP32, whose segments would be 16 bytes, 1024 x 1024 x 1024 N = 8 21.8 | 22.4).
// Beyond 2048 a strip of 8 columns fills a compute unit, and the launch runs in rounds of 256 strips; of strips of
// 4 two or three are resident.  Those are read less well, so they are taken where they save more than their price in the last
// round (1500 + 1111 columns of 3001: 71 -> 40 us).  The prices, 1.1 in FP64 and 1.3 in FP32, are on the safe side of what long
// launches show (strips of 4 against 8, us, 16384 columns of 2100 | 3072 | 4096: FP64 N = 15 206 : 189 | 274 : 270 | 384 : 369,
// FP32 N = 8 130 : 130 | 196 : 179 | 266 : 225; 8192 columns 111 : 96 | 146 : 133 | 203 : 185 and 45 : 54 | 97 : 84 | 132 : 108).
// Where operand and slices stay in the caches strips of 4 would also win with whole rounds of 8: FP32, 5120 columns of 3072 41 : 49.
// Few vectors: narrower workgroups until there is one per compute unit.  Their operands come from the caches, where
// partial lines cost less than idle units (whole calls, N = 15 in FP64, us, 8 or 16 columns per workgroup whatever their
// number | this rule | at least 2: 256 x 256 x 2048 45.6 | 28.6 | 28.8, 64 x 64 x 4096 62.6 | 46.6 | 49.8,
// 512 x 256 x 2048 45.2 | 31.5 | 31.6; the kernels of oz2_prepost.hip and oz2_columns.hip took 40.4, 55.9 and 44.3).
// vectors: padded number of vectors in the launch.
inline FusedPlan fused_plan(int64_t Kp, bool strips, int64_t vectors, size_t element) {
    static const int shapes[][2] = {{256, 1}, {512, 1}, {512, 2}, {512, 3}, {512, 4}, {1024, 3}, {1024, 4}};
    int64_t per = strips ? (Kp <= 1024 ? (element == 8 && vectors <= 6144 ? 4 : 8) : 16) : (Kp <= 1024 ? 4 : 2);
    if (strips && Kp > 2048) {
        const int64_t resident = 4 * Kp <= 512 * 3 * 8 ? 3 : 2;
        const double by8 = (double)((vectors / 8 + 255) / 256) * 8;
        const double by4 = (double)((vectors / 4 + 256 * resident - 1) / (256 * resident) * resident) * 4 * (element == 8 ? 1.1 : 1.3);
        per = by4 < by8 ? 4 : 8;
    }
    while (per > 1 && vectors < per * 256) per /= 2;
    const int64_t want = Kp * per;
    FusedPlan p{1024, 4, 0};
    for (const auto &s : shapes)
        if ((int64_t)s[0] * s[1] * 8 >= want) { p.threads = s[0]; p.pieces = s[1]; break; }
    const int64_t room = (int64_t)p.threads * p.pieces * 8;
    while (p.log_v < 5 && (Kp << (p.log_v + 1)) <= room && (16 << p.log_v) <= p.threads) ++p.log_v;
    return p;
}

// Groups of moduli get workgroups of their own where every one of those has a compute unit.  Only the smallest shape can have
// that few workgroups: the others have 256 at least.
constexpr int kFusedSplitThreads = 256, kFusedSplitPieces = 1;
inline bool fused_split_applies(const FusedPlan &p, int64_t workgroups, int64_t groups) {
    return groups > 1 && workgroups * groups <= 256 && p.threads == kFusedSplitThreads && p.pieces == kFusedSplitPieces;
}

// A factor of rows and one of columns share a launch up to here; beyond, the two forms want different
// workgroups and a launch more costs less.
constexpr int64_t kFusedShareLaunch = 2048;

inline bool supported(int64_t k, int N) {
    return N >= OZ2_MIN_MODULI && N <= OZ2_MAX_MODULI && k <= OZ2_MAX_K_BLOCKED;
}

// What a product call has to do once its arguments have passed the checks.
enum class Action { kNothing, kScaleC, kProduct };

// The argument checks of the product entry points, in the order their documentation states:
// sizes and ops, then the supported range, then empty products, then pointers and leading
// dimensions.  op(A) is m x k and op(B) is k x n (row-major storage).
inline oz2_status check_gemm_args(int opA, int opB, int64_t m, int64_t n, int64_t k, const void *A, int64_t lda,
                                  const void *B, int64_t ldb, const void *C, int64_t ldc, int N, Action *action) {
    *action = Action::kNothing;
    if (m < 0 || n < 0 || k < 0 || (opA != OZ2_OP_N && opA != OZ2_OP_T) || (opB != OZ2_OP_N && opB != OZ2_OP_T))
        return OZ2_INVALID_ARG;
    if (!supported(k, N)) return OZ2_UNSUPPORTED;
    if (m == 0 || n == 0) return OZ2_OK;
    if (!C || ldc < n) return OZ2_INVALID_ARG;
    if (k == 0) { *action = Action::kScaleC; return OZ2_OK; }
    const bool a_kc = opA == OZ2_OP_N, b_kc = opB == OZ2_OP_T;   // is k the contiguous index?
    if (!A || !B || lda < (a_kc ? k : m) || ldb < (b_kc ? k : n)) return OZ2_INVALID_ARG;
    *action = Action::kProduct;
    return OZ2_OK;
}

// Workspace: [scratch | tA | tB | residues of A | residues of B | products].  A product of
// prepared operands uses the product part only (its shifts and residues live in the operands).
struct Layout {
    int64_t m, n, k, Mp, Np, Kp;
    int N;
    bool prod_u8;
    bool with_operands;                    // the call converts its factors itself
    size_t off_bt, off_ta, off_tb, off_ra, off_rb, off_prod;
    size_t prod_whole, prod_min;           // product part: all of C at once / one 256 x 256 panel
    int ranges;                            // K ranges of a whole product (gemm_plan) ...
    size_t prod_ranges;                    // ... and what they take beyond prod_whole, if it is to be had
};

// Bytes of product workspace per entry of C: N planes of uint8, or of int32 (diagnostic form).
inline size_t bytes_per_entry(int N, bool prod_u8) { return (size_t)N * (prod_u8 ? 1 : 4); }

inline int whole_product_ranges(int64_t m, int64_t n, int64_t Mp, int64_t Np, int64_t Kp, int N);

inline Layout make_layout(int64_t m, int64_t n, int64_t k, int N, bool prod_u8, bool with_operands = true) {
    Layout L{};
    L.m = m; L.n = n; L.k = k; L.N = N; L.prod_u8 = prod_u8; L.with_operands = with_operands;
    L.Mp = round_up(m, kPadMN); L.Np = round_up(n, kPadMN); L.Kp = round_up(k, kPadK);
    size_t o = 0;
    if (with_operands) {
        L.off_bt = o;   o += align256(accurate_scratch_bytes(m, n));
        L.off_ta = o;   o += align256((size_t)m * 4);
        L.off_tb = o;   o += align256((size_t)n * 4);
        L.off_ra = o;   o += align256((size_t)N * L.Mp * L.Kp);
        L.off_rb = o;   o += align256((size_t)N * L.Np * L.Kp);
    }
    L.off_prod = o;
    L.prod_whole = align256((size_t)L.Mp * L.Np * bytes_per_entry(N, prod_u8));
    L.prod_min = align256((size_t)kPadMN * kPadMN * bytes_per_entry(N, prod_u8));
    L.ranges = prod_u8 ? whole_product_ranges(m, n, L.Mp, L.Np, L.Kp, N) : 1;
    L.prod_ranges = (size_t)(L.ranges - 1) * L.prod_whole;
    return L;
}

// How C is cut: panels of (pr x pc) entries (multiples of 256; the last ones may be smaller).
struct Panels {
    int64_t pr, pc, count;
};

// Panels whose N product planes fit into `avail` bytes: all of C if possible, otherwise as
// square as the shape allows (the INT8 GEMM re-reads a row panel of the A slices once per
// column panel and vice versa).  Panel sides below the full side are 256 times a power of two
// up to 4096 and multiples of 4096 beyond: then the workgroups of a launch (tiles x moduli) fill
// the 256 compute units evenly and the GEMM's tile map stays XCD-aware (measured at 16384^3,
// N = 16: panels of 2816^2 72 ms against 67.8 ms for 2048^2 and 62.9 ms for 4096^2).
inline int64_t panel_side(int64_t w) {
    if (w >= 4096) return w / 4096 * 4096;
    int64_t s = kPadMN;
    while (2 * s <= w) s *= 2;
    return s;
}

inline bool plan_panels(const Layout &L, size_t avail, Panels *out) {
    const size_t per = bytes_per_entry(L.N, L.prod_u8);
    if (avail >= L.prod_whole) { *out = Panels{L.Mp, L.Np, 1}; return true; }
    const int64_t entries = (int64_t)(avail / per);
    if (entries < kPadMN * kPadMN) return false;
    int64_t s = kPadMN;
    while ((s + kPadMN) * (s + kPadMN) <= entries) s += kPadMN;
    s = panel_side(s);
    int64_t pr = std::min(L.Mp, s), pc = std::min(L.Np, s);
    auto widen = [&](int64_t other, int64_t now, int64_t limit) {   // what fits beside `other`
        const int64_t w = entries / other / kPadMN * kPadMN;
        return std::max(now, w >= limit ? limit : panel_side(w));
    };
    pc = widen(pr, pc, L.Np);
    pr = widen(pc, pr, L.Mp);
    *out = Panels{pr, pc, ((L.Mp + pr - 1) / pr) * ((L.Np + pc - 1) / pc)};
    return true;
}

// How the INT8 GEMM launches of a product (of each workspace panel, if C is worked through in
// panels) are cut: into launches of at most kLaunchPanelRows x kLaunchPanelCols entries of C per
// modulus, each writing its part of the product buffer in place.  A launch over all of a large C
// runs hundreds of rounds of 256 workgroups; over such a launch the workgroups of a round drift
// apart, the operand tiles that an XCD's L2 holds are shared by fewer of its workgroups and the
// launch fetches a quarter more through the fabric.  A launch boundary every 32 rounds or so
// keeps them together.  Measured back to back on three devices, whole launch against these
// panels: 16384^3 1.2 to 4.6 % of the call (the slower the device, the more), 10000 x 9000 x
// 20000 4.5 %, 8192 x 8192 x 65536 1 to 3 %; no difference at 8192^3 or for k <= 4096, hence the
// limit on k.  (4096 x 4096 is as good at k = 16384 and 1 % worse at 8192^3; 2048-wide panels lose
// the XCD-aware tile order and are worse except for the longest contractions.)
#ifndef OZ2_LAUNCH_PANEL_ROWS
#define OZ2_LAUNCH_PANEL_ROWS 4096
#endif
#ifndef OZ2_LAUNCH_PANEL_COLS
#define OZ2_LAUNCH_PANEL_COLS 8192
#endif
#ifndef OZ2_LAUNCH_PANEL_MIN_K
#define OZ2_LAUNCH_PANEL_MIN_K 8192
#endif
constexpr int64_t kLaunchPanelRows = OZ2_LAUNCH_PANEL_ROWS, kLaunchPanelCols = OZ2_LAUNCH_PANEL_COLS;
constexpr int64_t kLaunchPanelMinK = OZ2_LAUNCH_PANEL_MIN_K;

// rows x cols: the padded extent of what the launches cover (all of C, or one workspace panel).
inline Panels launch_panels(int64_t rows, int64_t cols, int64_t Kp) {
    Panels Q{rows, cols, 1};
    if (kLaunchPanelRows <= 0 || Kp < kLaunchPanelMinK) return Q;
    Q.pr = std::min(rows, kLaunchPanelRows); Q.pc = std::min(cols, kLaunchPanelCols);
    Q.count = ((rows + Q.pr - 1) / Q.pr) * ((cols + Q.pc - 1) / Q.pc);
    return Q;
}

// ... and along k: a launch of such a panel is kept to about kLaunchMs of matrix-core work (counting
// 13.4 ns per element of k for a round of 256 tiles, what it took with 32x32x32 MFMAs; with 16x16x64 it is 11.5
// and the target about 6 ms), in equal K ranges that are multiples
// of 8192; the results of the ranges are folded modulo p_s in the GEMM's store phase like the
// ranges of 2^17 that exactness requires (Section 4.3).  Returns the length of a K range: Kp
// itself when one launch is short enough, never more than OZ2_MAX_K.  Measured: 8192 x 8192 x
// 65536, N = 18: 74.3 -> 72.3 ms; 4096 x 4096 x 131072, N = 16: 38.4 -> 36.6 ms.
#ifndef OZ2_LAUNCH_MS
#define OZ2_LAUNCH_MS 7.0
#endif
constexpr double kLaunchMs = OZ2_LAUNCH_MS, kRoundNsPerK = 13.4;
constexpr int64_t kLaunchKStep = 8192;

inline int64_t launch_k_len(int64_t Kp, int N, const Panels &Q) {
    const int64_t whole = std::min<int64_t>(Kp, OZ2_MAX_K);
    if (kLaunchPanelRows <= 0 || Kp < 2 * kLaunchPanelMinK) return whole;
    const int64_t tiles = (Q.pr / kPadMN) * (Q.pc / kPadMN) * N;
    const int64_t rounds = (tiles + 255) / 256;
    const double want = kLaunchMs * 1e6 / (kRoundNsPerK * (double)rounds);      // elements of k per launch
    int64_t len = std::max<int64_t>(kLaunchKStep, (int64_t)(want / kLaunchKStep + 0.5) * kLaunchKStep);
    if (2 * Kp < 3 * len) return whole;                    // less than one and a half launches: leave it whole
    const int64_t n = (Kp + len - 1) / len;
    len = round_up((Kp + n - 1) / n, kLaunchKStep);
    return std::min<int64_t>(len, OZ2_MAX_K);
}

// K ranges with planes of their own, at most: 16 keep a workgroup on at least 12 K tiles where they help.
constexpr int kMaxRanges = 16;

// The smallest products run their GEMMs and the accumulation as one launch (oz2_tiny.hip): tiles of 16 x 16 where these and
// the padding have a compute unit each, else of 32 x 32.
struct TinyGrid {
    int64_t tiles_m, tiles_n, padding;     // padding: workgroups that clear it
    int64_t tiles() const { return tiles_m * tiles_n; }
};
inline TinyGrid tiny_grid(int64_t m, int64_t n, int tile) {
    const int64_t tiles_m = (m + tile - 1) / tile, tiles_n = (n + tile - 1) / tile;
    const int64_t Mp = round_up(m, kPadMN), Np = round_up(n, kPadMN);
    return TinyGrid{tiles_m, tiles_n, (Mp / tile - tiles_m) * (Np / kPadMN) + (Np > tiles_n * tile ? tiles_m : 0)};
}
inline bool tiny_small_tiles(int64_t m, int64_t n) {
    const TinyGrid g = tiny_grid(m, n, 16);
    return g.tiles() + g.padding <= 256;
}

// Which products: at most one 32 x 32 tile of C per compute unit, at most 512 elements of k in a row for a wavefront (each of
// the 16 takes every 16th modulus), and few enough operands for a compute unit to load: 64 Kp N bytes with tiles of 32 x 32, 32 Kp N with
// 16 x 16.  Prepared operands gain nearly throughout (us, other operands in each call, graph, two launches | one: 400 x 400 x 256 N = 15 10.5 | 9.9,
// 512 x 512 x 512 FP32 N = 7 9.9 | 9.0, 512 x 512 x 256 N = 15 11.0 | 10.3, 500 x 500 x 128 N = 20 12.0 | 9.3, 150 x 150 x 512 N = 13 9.5 | 8.1; 300 x 300 x 512 FP32 N = 8
// 8.7 | 9.2).  Beyond the limits: 231 x 384 x 512 N = 14 (32 x 32) 10.0 | 12.6, 277 x 277 x 300 N = 16 0.86, 105 x 172 x 512 N = 16 (16 x 16) 0.97.
//
// A call that converts its factors itself gains less (whole calls, in a graph, us, two launches -> one: 209 x 209 x 512 N = 14 16.1 -> 15.8, 68 x 87 x 300
// N = 14 13.8 -> 12.3, 188 x 140 x 256 N = 15 13.1 -> 11.3, 142 x 142 x 64 N = 14 12.0 -> 9.5, 512 x 512 x 512 FP32 N = 7 15.3 -> 14.8, 1000 x 250 x 256 N = 15
// 18.1 -> 16.3), and may lose where C is about as wide as high and the moduli are many: 512 x 512 x 256 N = 16 17.4 -> 18.2,
// 319 x 319 x 256 N = 17 15.7 -> 17.0, 300 x 300 x 512 FP32 N = 8 14.1 -> 15.7, 400 x 400 x 256 N = 15 16.3 -> 17.2.  The lines below were drawn
// for a kernel that also requested chunks of k that do not exist and have not been drawn again.  On the side of two launches, calls one after
// another, two -> one: 200 x 200 x 256 N = 16 17.2 -> 15.3, 150 x 130 x 200 N = 17 16.7 -> 14.5, 300 x 300 x 128 N = 15 17.2 -> 15.7, 448 x 448 x 256 N = 16 18.4 -> 18.3,
// 312 x 528 x 128 N = 18 15.7 -> 16.2, 500 x 300 x 390 FP32 N = 8 14.5 -> 14.9.
inline bool tiny_product_applies(int64_t m, int64_t n, int64_t Kp, int N, bool prepared) {
    if ((m + 31) / 32 * ((n + 31) / 32) > 256 || (N + 15) / 16 * Kp > 512) return false;
    if (Kp * N > (tiny_small_tiles(m, n) ? 7168 : 4096)) return false;
    const int64_t longer = std::max(m, n), shorter = std::min(m, n);
    if (prepared || longer >= 4 * shorter) return true;
    if (tiny_small_tiles(m, n)) return N <= 15 || shorter <= 64;
    if (N <= 6 || (N <= 10 && Kp <= 256)) return true;
    if (N > 16) return longer > 384;       // the INT8 GEMM of the other form has a second round
    return longer > 448 && (Kp > 128 || N <= 13);
}

// The accumulation gives each thread kEpilogueColumns consecutive columns of a row, in workgroups of kEpilogueThreads, and works
// out a thread's place from its number in 31 bits: a launch covers at most this many rows (0: a row of U that takes
// 4 GiB per modulus, which is refused).
constexpr int kEpilogueColumns = 4, kEpilogueThreads = 256;
constexpr int64_t kEpilogueMaxThreads = (int64_t)0x7fffff00;     // whole workgroups below 2^31
inline int64_t epilogue_groups(int64_t n) { return (n + kEpilogueColumns - 1) / kEpilogueColumns; }
inline int64_t epilogue_rows(int64_t groups, int64_t max_threads = kEpilogueMaxThreads) {
    return groups > 0x3fffffff ? 0 : max_threads / groups;
}

// Which tiles the INT8 GEMM takes: 256 x 256, or 128 x 128 with 8 wavefronts and 6 stages of LDS (one workgroup per compute unit) or with 4
// and 4 (two share a unit).
//
// The small ones where at most 512 of them hold entries of C: large ones would leave half of the compute units without one, and up to
// there every unit has work with two of the small ones.  Prepared operands, other ones in
// each call, us, 128 x 128 | 256 x 256: 96 large tiles (1024^3 FP32 N = 6) 19.4 | 21.9; 112 19.8 | 22.7; 120 (2048 x 256 x 1024 N = 15) 20.5 | 22.8; 128
// (1024^3 FP32 N = 8) 21.4 | 23.9, (512 x 1024 x 8192 N = 16) 87.4 | 92.2, (2048^3 N = 2) 33.2 | 37.2; 135 (768 x 768 x 1024 N = 15) 26.8 | 24.0; 140
// 29.3 | 25.3; 168 (1024 x 768 x 1024 N = 14) 27.2 | 23.5; 224 (1024^3 N = 14) 33.5 | 28.1; 448 (2048^3 FP32 N = 7) 78.6 | 66.3.  Accurate mode's one slice, whole
// calls: 128 (2048 x 4096 x 2048 FP32 N = 6) 174 | 179, 144 (2304 x 4096 x 2048) 207 | 203.
//
// Of those, at most one per compute unit run with 8 wavefronts and 6 stages.  us as
// above, 4 and 4 | 8 and 6: 256 x 256 x 1024 N = 15 10.7 | 10.2, x 4096 30.7 | 26.0, 500 x 300 x 777 FP32 N = 8 9.9 | 9.6, 512 x 512 x 2048 N = 15 20.8 | 19.6, 512^3
// N = 14 10.8 | 10.7, N = 16 (256 tiles) 11.6 | 11.5, N = 17 (272) 12.6 | 14.9, 768 x 768 x 512 N = 8 (288) 13.1 | 15.4; accurate mode, whole calls, 512^3
// N = 15 35.9 | 34.7, 1024^3 63.1 | 61.4.
enum class GemmTile { kLarge, kOnePerUnit, kTwoPerUnit };
inline int64_t blocks_of_128(int64_t rows, int64_t cols) { return (rows + 127) / 128 * ((cols + 127) / 128); }

// Large tiles in the uint8 forms go to the kernel of oz2_wide_gemm.hip if there are more of them than compute units (many more where the
// contraction is short), or the contraction is long; its way to the first operands and its
// reduction, which has no other wavefront on its SIMD, weigh more where each unit has a single short tile.  Prepared products, us, oz2_int8_gemm.hip | oz2_wide_gemm.hip: 16384 x 8192 x 16384 N = 8 12205 | 11625, 8192^3 FP32 N = 8
// 3166 | 3020, 1536 x 1000 x 40000 N = 18 858 | 817, 4096^3 N = 14 755 | 732, 2048^3 N = 15 128.3 | 124.6, 8192 x 8192 x 1024 1181 | 1165, x 512 872 | 859;
// 4096 x 4096 x 384 222 | 219, 1500 x 1500 x 512 N = 16 45.0 | 44.4; at most one tile per unit: 1024 x 1024 x 16384 188 | 181, x 4096 59.7 | 59.4, 768 x 768 x 4096
// 50.9 | 51.7, 900 x 900 x 384 N = 16 23.3 | 23.9; short contractions with few tiles per unit: 1131 x 1290 x 469 N = 16 (480 tiles) 30.2 | 31.3, 2079 x 2123 x 747 FP32
// N = 8 (648) 46.0 | 47.6, 2391 x 1846 x 623 N = 14 (1120) 72.3 | 72.5, 2375 x 4052 x 442 FP32 N = 9 (1440) 80.8 | 80.6, 1779 x 3983 x 513 N = 15 (1680) 103.2 | 102.5 (36 shapes of 257 to
// 2048 tiles with k = 385 to 767: 0.6 % slower on average).  Beyond kWideMaxK its sums would not fit (see there).
constexpr int kWideMinKTiles = 6;
constexpr int64_t kWideMaxK = 65536, kWideLongK = 8192, kWideShortK = 768, kWideShortTiles = 2048;
// tiles: of all slices and K ranges; k_len elements of k in `ranges` ranges
inline bool wide_gemm_applies(int64_t tiles, int64_t k_len, int ranges) {
    if (k_len > kWideMaxK || k_len / (2 * kBlockK) / ranges * 2 < kWideMinKTiles) return false;
    const int64_t k = k_len / ranges;
    return k >= kWideLongK || tiles > (k >= kWideShortK ? 256 : kWideShortTiles);
}

// The contraction of a few tiles runs in K ranges at once, whose results meet in the accumulation: a range more is a workgroup more
// per tile, and costs a plane more per modulus to write and read.  The estimates, in us, are fits of
// prepared products (N = 16, k = 2048 to 40000, up to 16 ranges; 32 shapes, of which the choice made is within 3 % of the best on average):
// a workgroup of 256 x 256 takes 0.57 per K tile of 64 while at most half of the units have one and 0.75, at the board's power limit,
// when all have; one of 128 x 128 0.27 to 0.33, two that share a unit 0.55.  One range | chosen, us: 256 x 256 x 40000 175 | 67 (4 ranges, 128 x 128), x 4096 17.3 | 13.6;
// 512 x 512 x 40000 199 | 144 (4), 512 x 768 x 8192 77 | 60 (2), 768 x 768 x 40000 367 | 309 (5), 1280 x 1024 x 40000 786 | 643 (4; 320 tiles); nothing to be gained
// for 256 tiles, nor for 432 (1536 x 1000 x 40000 N = 18: 853 | 846, power).
struct GemmPlan {
    GemmTile tile;
    int ranges;
};
inline double large_tiles_us(double tiles, double kt) {      // rounds of 256, of which the last may be partial
    const double rounds = (double)(int64_t)(tiles / 256), last = tiles / 256 - rounds;
    return rounds * (0.75 * kt + 4) + (last > 0 ? (0.57 + 0.36 * std::max(0.0, last - 0.5)) * kt + 4 : 0);
}
inline double small_tiles_us(double tiles, double kt) {      // at most 256, then two per unit in rounds of 512
    if (tiles <= 256) return (0.27 + 0.08 * std::max(0.0, tiles / 256 - 0.25)) * kt;
    return (double)(int64_t)((tiles + 511) / 512) * (0.55 * kt + 2);
}
// rows x cols entries of C; `slices` of them, whose contraction has kt K tiles; may_range: the results of K ranges can be kept.
inline GemmPlan gemm_plan(int64_t rows, int64_t cols, int64_t slices, int64_t kt, bool may_range) {
    const int64_t blocks = blocks_of_128(rows, cols) * slices;
    const double large = (double)((rows + 255) / 256 * ((cols + 255) / 256) * slices);
    GemmPlan best{blocks <= 256 ? GemmTile::kOnePerUnit : blocks <= 512 ? GemmTile::kTwoPerUnit : GemmTile::kLarge, 1};
    if (!may_range || large > 448) return best;
    // A range less has to be clearly worse, the more so for ranges of large tiles where the estimate makes one range of small ones up to 40 % too
    // slow.  Those have a unit each and a contraction below 8192 (us, one range | as estimated, the estimate of the ratio: 191 x 390 x 7676 N = 12 26.2 | 22.8
    // (0.66), 481 x 212 x 6626 N = 14 24.0 | 23.8 (0.75), 181 x 404 x 6807 N = 18 25.1 | 26.5 (0.76), 586 x 191 x 7076 N = 14 26.3 | 27.2 (0.82), 244 x 386 x 4623 N = 18 21.2 | 23.9
    // (0.93)), or two share one and it is below 4480 (133 x 1163 x 4378 N = 18 32.2 | 30.2 (0.82), 1133 x 246 x 2834 N = 15 23.9 | 24.1 (0.87), 1637 x 618 x 4286 N = 5 35.4 | 36.4
    // (0.89), 418 x 1753 x 2274 N = 5 20.8 | 22.0 (0.93); 1303 x 477 x 4573 N = 8 33.7 | 32.5 (0.86), 967 x 1484 x 7032 N = 5 54.0 | 52.4 (0.93)).
    double best_us = 0.95 * (5 + (best.tile == GemmTile::kLarge ? large_tiles_us(large, (double)kt) : small_tiles_us((double)blocks, (double)kt)));
    const double large_us = best_us * (best.tile == GemmTile::kOnePerUnit && kt < 128 ? 0.8 : best.tile == GemmTile::kTwoPerUnit && kt < 70 ? 0.9 : 1.0);
    for (int s = 2; s <= kMaxRanges && kt / s >= 12; ++s) {
        const double k = (double)kt / s, extra = 9 + s * (double)(rows * cols * slices) / 3e6;
        const double some = large * s;
        // (all units at once finish and store: a little more)
        const double l = extra + large_tiles_us(some, k) + (some / 256 - (double)(int64_t)(some / 256 - 1e-9) > 0.9 ? 5 : 0);
        if (large >= 24 && l < std::min(best_us, large_us)) { best_us = l; best = GemmPlan{GemmTile::kLarge, s}; }
        const double o = extra + small_tiles_us((double)(blocks * s), k);
        if (blocks * s <= 256 && o < best_us) { best_us = o; best = GemmPlan{GemmTile::kOnePerUnit, s}; }
    }
    return best;
}

// A contraction of several launches (k beyond 2^17), which has no K ranges at once: blocks of padding are computed like the others
// where all of them have a compute unit each and at most half hold entries of C.  Their workgroups read the same rows of A or columns of B as
// those beside them, and with so few in the launch that help is worth more than the idle units (prepared, us, padding
// cleared | computed: 64 x 100 x 10^6 N = 6 4227 | 4020, 128 x 128 x 400000 N = 16 1721 | 1693, 16 x 16 x 10^6 N = 15 4292 | 4201, 200 x 100 x 150000 N = 14
// 649 | 637; with three quarters of the blocks in use 300 x 200 x 200000 N = 15 864 | 883).
inline bool padding_computed(int64_t rows, int64_t cols, int64_t valid_rows, int64_t valid_cols, int64_t slices) {
    return blocks_of_128(rows, cols) * slices <= 256 && 2 * blocks_of_128(valid_rows, valid_cols) <= blocks_of_128(rows, cols);
}

inline int whole_product_ranges(int64_t m, int64_t n, int64_t Mp, int64_t Np, int64_t Kp, int N) {
    const Panels Q = launch_panels(Mp, Np, Kp);
    if (Kp > OZ2_MAX_K || Q.count != 1 || launch_k_len(Kp, N, Q) != Kp) return 1;
    return gemm_plan(m, n, N, Kp / kBlockK, true).ranges;
}

// What the library's own workspace of `bytes` bytes has beside them for the planes of K ranges: as much as the planes of any product whose
// workspace fits `bytes` can take (15 times its first planes, with C of few tiles; 247.5 MiB, at 1 x 5377 x 108416 N = 12).
constexpr size_t kMaxPlanes = (size_t)256 << 20;
inline size_t planes_reserve(size_t bytes) { return std::min((size_t)(kMaxRanges - 1) * bytes, kMaxPlanes); }

// Side of a panel of the overlapped form: the INT8 GEMM loses nothing down to 4096 x 4096.
constexpr int64_t kOverlapPanel = 4096;

// The overlapped form (conversion of later panels beside the GEMMs of earlier ones) needs a long
// contraction and enough panels to hide something behind: panels of at most 4096 x 4096, at
// least four of them, k >= 8192 and k x panels >= 9 x 8192 (measured: with less, the conversion
// that precedes the first GEMM, or what the shorter GEMM launches lose, outweighs what is hidden).
inline bool overlap_applies(int64_t Kp, int64_t panels) {
    return panels >= 4 && panels <= 4096 && Kp >= 8192 && Kp * panels >= (int64_t)9 * 8192;
}

// Panels of the overlapped form for a layout: P capped at kOverlapPanel per side.
inline Panels overlap_panels(const Layout &L, Panels P) {
    P.pr = std::min(P.pr, kOverlapPanel); P.pc = std::min(P.pc, kOverlapPanel);
    P.count = ((L.Mp + P.pr - 1) / P.pr) * ((L.Np + P.pc - 1) / P.pc);
    return P;
}

}  // namespace oz2
