// Batched INT8 GEMM with exact (wrapping) INT32 accumulation on the gfx950 matrix cores:
// Algorithm 1 line 6, C'_s = A'_s B'_s for all moduli s in one launch.
//
// Operands are the padded residue slices in the K-blocked layout the residue kernel
// writes: A [batch][Kp/64][Mp][64] and B [batch][Kp/64][Np][64] (B transposed), i.e. 64
// consecutive k of one row are contiguous and consecutive rows of one 64-wide K block
// follow each other.  A (rows x 64) tile of either operand is then one contiguous run of
// memory, fetched as whole 128-byte lines, both tiles are staged through LDS the same way
// and every MFMA operand is a 16-byte K-run read with one ds_read_b128.
//
// Tiling: workgroup = WM x WN wavefronts, block tile (32 TM WM) x (32 TN WN) x 64, each
// wavefront owns (32 TM) x (32 TN), in 2 TM x 2 TN accumulators of v_mfma_i32_16x16x64_i8.  The
// large configuration is 2 x 4 wavefronts of 128 x 64 (a 256 x 256 block, 128 accumulator
// registers per lane, two wavefronts per SIMD).  Where there are many such blocks or the contraction is long, the uint8 forms go
// to 4 wavefronts of 128 x 128 instead (oz2_wide_gemm.hip; wide_gemm_applies has the line).
//
// Bound: board power for large products of random residues (the clock falls to 1.6 GHz), so the instruction that
// spends less energy per operation is the faster one: from registers 16x16x64 sustains 4.1 POP/s on
// random operands and 32x32x32, which reads and writes twice the accumulators per operation, 3.5 (4.95 both on
// constant ones).  Products of prepared operands, 32x32x32 -> 16x16x64, us: 8192^3 N = 14 6410 -> 5540, 4096^3 N = 14
// 858 -> 765, 2048^3 FP32 N = 7 69.8 -> 61.9, 8192 x 8192 x 512 N = 15 978 -> 922; 16384^3 N = 16 whole 56.7 -> 52.0 ms.
//
// Data movement: global_load_lds_dwordx4 copies HBM/L2 straight into a ring of STAGES LDS
// stages, STAGES-1 tiles ahead of the math, so no VGPRs or ds_write instructions are spent
// on staging.  A wavefront's 64 lanes fill 64 consecutive 16-byte LDS chunks per
// instruction; the XOR swizzle that keeps the fragment reads free of bank conflicts is
// applied on the global side (which 16 bytes of a row a lane fetches).  MFMA operands are fetched into registers
// shortly before they are used, across stage boundaries: A's in two sets of two rows in turn, B's in place.  (More of
// them, four rows at a time or a second set for B with the loop unrolled over two K tiles, measured 0.5 to 1 % slower.)
//
// Synchronisation per K tile: one s_waitcnt vmcnt(n) that leaves the youngest tiles in
// flight, then one s_barrier.  The compiler does not track LDS writes made by
// global_load_lds, so these two are what orders them against the ds_reads.
#include <algorithm>
#include <type_traits>

#include "oz2_epilogue.hpp"
#include "oz2_kernels.hpp"
#include "oz2_tilemap.hpp"
#include "oz2_wide_gemm.hpp"

namespace oz2 {
namespace {

constexpr int64_t kMaxExactK = (int64_t)1 << 17;   // Section 4.3: no INT32 overflow up to here
#ifndef OZ2_PERSISTENT_MAX_K
#define OZ2_PERSISTENT_MAX_K 4096
#endif
constexpr int64_t kPersistentMaxK = OZ2_PERSISTENT_MAX_K;   // contractions up to here run as a persistent grid

typedef int v4i __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

// s_waitcnt immediate that waits for vmcnt <= n only (gfx9 encoding: vmcnt in bits 3:0 and
// 15:14, expcnt 6:4 and lgkmcnt 11:8 left at their maxima).
constexpr int vmcnt_imm(int n) { return (n & 0xf) | ((n >> 4) << 14) | (0x7 << 4) | (0xf << 8); }

// LDS on this chip is 64 banks x 4 B: a 256-byte line is 16 slots of 16 B, and a ds_read_b128 is served 16
// lanes per clock: lanes {0-3, 12-15, 20-27} together, then {4-11, 16-19, 28-31}, likewise in the upper half.  A
// tile row is 4 slots, so the rows r and r + 4 start in the same slot and a fragment read (16 rows; lane l reads
// row l % 16, chunk l / 16) has four rows, in two chunks, that want the same slots in each such group.  XOR-ing the chunk index with
// 0, 2, 3, 1 for the row quads 0 to 3 gives each of the 16 lanes a slot of its own (0 conflict cycles per read in the
// counters; 0, 1, 2, 3, which suits fragments of 32 rows, 4 of 8).
__device__ inline int swizzle_mask(int row) {
    const int quad = row >> 2;
    return ((quad ^ (quad >> 1)) & 1) << 1 | (quad >> 1 & 1);
}

// What the store phase writes (Algorithm 1 lines 6-7):
//   kOutI32      C'_s as int32 (diagnostics: the raw products)
//   kOutI32Fold  int32: mod(old, p_s) + mod(C'_s, p_s)   (a further K range of a k > 2^17 product)
//   kOutU8       U_s = mod(C'_s, p_s) as uint8 -- the form the accumulation kernel wants
//   kOutU8Fold   uint8: (old + mod(C'_s, p_s)) mod p_s
//   kOutMax      nothing of the product itself: only its row and column maxima, folded into
//                two int arrays with atomic maxima (accurate mode of Section 4.2, where the
//                product Cbar = Abar * Bbar of the 7-bit matrices is needed for nothing else).
//                The kernel arguments then mean: C = the row maxima of the panel's rows,
//                C + c_plane (in ints) = the column maxima of its columns, c_ld = the number of
//                valid rows of the panel in its low and of valid columns in its high 32 bits.
//                (k_int8_gemm only.)
enum { kOutI32 = 0, kOutI32Fold = 1, kOutU8 = 2, kOutU8Fold = 3, kOutMax = 4 };

struct GemmMods {                       // moduli of the slices and what their reductions need
    int32_t p[kMaxModuli];
    int32_t pinv_prime[kMaxModuli];     // mulhi reduction (int32 forms)
    ByteMod byte_mod[kMaxModuli];       // reduction to bytes (uint8 forms)
};

// The uint8 forms start their sums at -2^31 (see oz2_bytemod.hpp), the others at 0.
constexpr int first_acc(int out) { return out == kOutU8 || out == kOutU8Fold ? (int)0x80000000 : 0; }

// No memory access moves across this in the compiler (no instruction; the hardware issues in order).
__device__ __forceinline__ void pin_memory_order() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The LDS of a workgroup: STAGES stages of (A rows | B rows) x 64 bytes.  Declared here, not
// passed around, so that every access is an offset from a base the compiler knows.
extern __shared__ v4i lds[];                              // [STAGES][ROWS][CPR]

// Everything one workgroup does for one output tile, shared by the two kernels below: where its
// lanes fetch from, the K loop, and the store phase.  A tile is identified by the global address
// its loads start at (tile_source) and by (slice, first row, first column) for the store.
template <int WM, int WN, int TM, int TN, int BK, int STAGES>
struct GemmCore {
    static constexpr int THREADS = 64 * WM * WN;              // WM x WN wavefronts
    static constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
    static constexpr int CPR = BK / 16;                       // 16-byte chunks per tile row
    static constexpr int ROWS = BM + BN;                      // A rows then B rows in one LDS stage
    static constexpr int CHUNKS = ROWS * CPR;
    static constexpr int LPT = CHUNKS / THREADS;              // LDS-direct loads per lane and tile
    static constexpr int FM = 2 * TM, FN = 2 * TN;            // 16 x 16 fragments of a wavefront
    static constexpr int STAGE_BYTES = CHUNKS * 16;
    static constexpr int ROWS_PER_LOAD = 64 / CPR;            // rows one wavefront-wide load covers
    static_assert(CHUNKS % THREADS == 0 && (BM * CPR) % (64 * LPT) == 0,
                  "each wavefront must load from one operand only");
    static_assert(BK == kBlockK, "the K tile is the K block of the operand layout");
    static_assert(CPR == 4, "the load-side swizzle below assumes one mask per lane");
    static_assert(STAGES >= 3 && (STAGES - 3) * LPT < 64, "vmcnt is a 6-bit counter");
    static constexpr int RB = 2, NB = FM / RB;                // blocks of rows that the K loop takes one after another
    static_assert(FM % (2 * RB) == 0 && LPT >= 2 && LPT <= 4, "fragments of two blocks in turn");
    static_assert(FN == 2 || FN == 4, "the store phase transposes groups of four blocks");

    int wm, wn, lrow, lquad;
    // Load i of this wavefront fills LDS chunks [64 q, 64 q + 64) of a stage, q = wave*LPT + i,
    // i.e. rows q*ROWS_PER_LOAD ...; lane -> (row, physical chunk) -> logical chunk to fetch.
    // In the blocked layout those 64 chunks are 1 KiB of contiguous memory, so the LPT loads of a
    // wavefront and tile differ by i KiB in the global AND in the LDS address: one address and
    // one LDS base (M0) per tile, the rest is the instruction's immediate offset, which the
    // hardware applies to both.
    static_assert(ROWS_PER_LOAD * BK == 1024 && (LPT - 1) * 1024 < 4096, "immediate offset of the loads");
    int row0, ch;
    bool from_a;                                              // uniform over the wavefront
    int64_t tile_step;                                        // next K block of the same rows
    int my_dst;                                               // uniform: byte offset within a stage
    // Fragment addressing: lane l reads row (l % 16) of a 16-row fragment, 16-byte chunk l / 16 of the
    // K tile (one MFMA takes all 64 of its k).  The swizzle mask depends on l % 16 only.
    int a_addr, b_addr;                                       // byte offsets within a stage

    __device__ __forceinline__ GemmCore(int64_t Mp, int64_t Np) {
        const int tid = threadIdx.x, lane = tid & 63;
        // the wavefront index as a scalar: everything derived from it stays in scalar registers
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        wm = wave / WN; wn = wave % WN;
        const int row0u = wave * LPT * ROWS_PER_LOAD;
        row0 = row0u + lane / CPR;
        ch = (lane % CPR) ^ swizzle_mask(row0);
        from_a = row0u < BM;
        tile_step = (from_a ? Mp : Np) * BK;
        my_dst = wave * LPT * 1024;
        lrow = lane & 15; lquad = lane >> 4;
        const int c = lquad ^ swizzle_mask(lrow);
        a_addr = ((wm * 32 * TM + lrow) * CPR + c) * 16;
        b_addr = ((BM + wn * 32 * TN + lrow) * CPR + c) * 16;
    }

    // Where this lane's loads of tile (s, tr, tc) start.  KB = K blocks per slice; the launch
    // contracts over blocks [kb0, kb0 + KT).
    __device__ __forceinline__ const int8_t *tile_source(const int8_t *A, const int8_t *B, int s, int tr, int tc,
                                                         int64_t Mp, int64_t Np, int64_t KB, int kb0) const {
        const int8_t *Ab = A + (((int64_t)s * KB + kb0) * Mp + (int64_t)tr * BM) * BK;
        const int8_t *Bb = B + (((int64_t)s * KB + kb0) * Np + (int64_t)tc * BN) * BK;
        return (from_a ? Ab + (int64_t)row0 * BK : Bb + (int64_t)(row0 - BM) * BK) + ch * 16;
    }

    // The loads of the K tile that start at src_t, into the stage at byte offset stage_off (uniform).  In assembly
    // (nothing is returned to registers), because the compiler takes the builtin for one that may complete out of
    // order with LDS reads, and then waits for all of those where the next of them is used.  M0, which is
    // nobody else's in these kernels, takes one wait state before it is read.
    __device__ __forceinline__ void issue_loads(const int8_t *src_t, int stage_off) const {
        static_assert(LPT == 2 || LPT == 4, "");
        const uint32_t dst = (uint32_t)(uintptr_t)(lds_ptr_t)lds + stage_off + my_dst;
        if constexpr (LPT == 2)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\t"
                         "global_load_lds_dwordx4 %1, off offset:1024" ::"s"(dst), "v"(src_t) : "memory");
        else
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\t"
                         "global_load_lds_dwordx4 %1, off offset:1024\n\tglobal_load_lds_dwordx4 %1, off offset:2048\n\t"
                         "global_load_lds_dwordx4 %1, off offset:3072" ::"s"(dst), "v"(src_t) : "memory");
    }

    // The first STAGES - 1 K tiles of a tile.  KT >= 2: every K range is a multiple of 128.
    __device__ __forceinline__ void issue_head(const int8_t *src_tile, int KT) const {
#pragma unroll
        for (int t = 0; t < STAGES - 1; ++t)
            if (t < KT) issue_loads(src_tile + (int64_t)t * tile_step, t * STAGE_BYTES);
    }

    // The K loop over a tile whose head has been requested: acc = first + A tile * B tile^T.
    // It is written so that the instruction stream between the MFMAs stays as short as it can be:
    // the loop is split into iterations that prefetch (all but the last STAGES - 1) and ones that
    // do not, so there is no branch per load; the LDS stage offsets are carried along, not
    // recomputed (measured against the same pipeline with a branch and a readfirstlane per load:
    // 3.5 % faster at 16 x 4096 x 4096 x 16384).
    // STORES: the vector stores that were issued after the head and before this call, if `stores` says so:
    // no fewer than that, or the relaxed wait below would pass K tiles that have not landed.
    template <int STORES = 0>
    __device__ __forceinline__ void contract(const int8_t *src_tile, int KT, int first, v4i (&acc)[FM][FN],
                                             bool stores = false) const {
        const v4i start = {first, first, first, first};
        v4i fa[2 * RB], fb[FN];
        const char *const lds_bytes = reinterpret_cast<const char *>(lds);
        auto load_a = [&](int stage_off, int i) {
            fa[i % (2 * RB)] = *reinterpret_cast<const v4i *>(lds_bytes + stage_off + a_addr + i * 16 * CPR * 16);
        };
        auto load_b = [&](int stage_off, int j) {
            fb[j] = *reinterpret_cast<const v4i *>(lds_bytes + stage_off + b_addr + j * 16 * CPR * 16);
        };

        // K tiles 0 and 1 must have landed before the first fragment reads.  In the persistent
        // kernel the stores of this workgroup's previous tile were issued after these loads.  Loads and
        // stores leave the counter in the order in which they were issued, so the youngest K tile and all
        // of the stores may stay outstanding: waiting for the stores here and after the first K tile
        // cost a write's way to memory per tile (8192 x 8192 x 512, N = 15: 1107 -> 1095 us for the call).
        constexpr int kYoungest = (STAGES - 3) * LPT;
        static_assert(kYoungest + STORES < 64, "vmcnt is a 6-bit counter");
        const bool lenient = STORES > 0 && stores && KT >= STAGES;
        if (lenient) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kYoungest + STORES));
        else if (KT >= STAGES - 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kYoungest));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int j = 0; j < FN; ++j) load_b(0, j);
#pragma unroll
        for (int i = 0; i < 2 * RB; ++i) load_a(0, i);

        // One K tile, in blocks of RB rows of MFMAs.  Behind a block the fragments of A of the block after the next one
        // are requested into its registers, and behind each column of the last block the next K tile's fragment of
        // B, so that LDS latency is covered by a block of MFMAs.  The K tile STAGES - 1 ahead is requested into the
        // stage read during the previous iteration, all of it behind a quarter of the MFMAs (prepared operands, us, at 1/8 | 1/4 |
        // 1/2 | 3/4, and half at 1/4 and half at 3/4: 16384 x 8192 x 16384 N = 8 12420 | 12220 | 12460 | 12550, 12335; 8192^3 N = 8
        // 3246 | 3200 | 3255 | 3280, 3222; the A tile at 1/4 and the B tile at 5/8 12725 and 3294).
        int cur_off = 0;
        const int8_t *src_ld = src_tile + (int64_t)(STAGES - 1) * tile_step;
        auto iteration = [&](auto opens_c, auto issued_c, auto last_c, bool after_stores = false) {
            constexpr bool opens = decltype(opens_c)::value, issued = decltype(issued_c)::value, last = decltype(last_c)::value;
            const int nxt_off = cur_off + STAGE_BYTES == STAGES * STAGE_BYTES ? 0 : cur_off + STAGE_BYTES;
            const int ld_off = cur_off == 0 ? (STAGES - 1) * STAGE_BYTES : cur_off - STAGE_BYTES;
#pragma unroll
            for (int p = 0; p < NB; ++p) {
#pragma unroll
                for (int j = 0; j < FN; ++j) {
#pragma unroll
                    for (int rr = 0; rr < RB; ++rr) {
                        const int i = p * RB + (j & 1 ? RB - 1 - rr : rr);   // a column starts with the row the last one ended with
                        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[j], fa[i % (2 * RB)], opens ? start : acc[i][j], 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (p == NB - 1 && !last) load_b(nxt_off, j);
                    if (issued && p * FN + j == NB * FN * 3 / 16) issue_loads(src_ld, ld_off);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    if (p + 2 < NB) load_a(cur_off, (p + 2) * RB + r);
                    else if (!last) load_a(nxt_off, (p + 2 - NB) * RB + r);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // Tile kt + 2 must be complete (and visible to every wavefront) before iteration
            // kt + 1 prefetches fragments from it; the barrier also frees the stage just read.
            if (STORES > 0 && issued && after_stores) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kYoungest + STORES));
            else if (issued) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kYoungest));
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            __builtin_amdgcn_s_barrier();
            cur_off = nxt_off;
            src_ld += tile_step;
        };
        constexpr std::true_type yes{};
        constexpr std::false_type no{};
        // The first K tile starts from `start` in every entry: no register of the accumulators is written beforehand.
        if (KT >= STAGES) iteration(yes, yes, no, lenient);
        else iteration(yes, no, no);
        int kt = 1;
        for (; kt + STAGES - 1 < KT; ++kt) iteration(no, yes, no);
        for (; kt + 1 < KT; ++kt) iteration(no, no, no);
        iteration(no, no, yes);
    }

    // Row and column maxima of the tile (kOutMax).  Entries are sums of products of non-negative
    // 7-bit numbers (k <= 2^17: below 2^29), the maxima start at 0 and zero entries (all the
    // padding) are skipped, so integer atomic maxima give the exact result whatever the order.  A
    // lane holds, per 16 x 16 block, 4 columns of one row: the row maximum is completed by the
    // lanes 16, 32 and 48 further on, a column maximum by the 16 lanes of the same quarter.
    __device__ __forceinline__ void store_maxima(const v4i (&acc)[FM][FN], int *rmax, int *cmax, int64_t bm,
                                                 int64_t bn, int valid_rows, int valid_cols) const {
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            int v = 0;
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) v = acc[i][j][r] > v ? acc[i][j][r] : v;
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) {
                const int o = __shfl_xor(v, off, 64);
                v = o > v ? o : v;
            }
            const int row = (int)bm + wm * 32 * TM + i * 16 + lrow;
            if (lquad == 0 && v > 0 && row < valid_rows) atomicMax(&rmax[row], v);
        }
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int v = 0;
#pragma unroll
                for (int i = 0; i < FM; ++i) v = acc[i][j][r] > v ? acc[i][j][r] : v;
#pragma unroll
                for (int off = 1; off < 16; off <<= 1) {
                    const int o = __shfl_xor(v, off, 64);
                    v = o > v ? o : v;
                }
                const int col = (int)bn + wn * 32 * TN + j * 16 + 4 * lquad + r;
                if (lrow == 0 && v > 0 && col < valid_cols) atomicMax(&cmax[col], v);
            }
    }

    // The store phase (Algorithm 1 lines 6-7 in the forms listed at kOut...).  The B fragment is
    // the MFMA's first operand, so the 16x16 accumulator is the transposed block: lane l holds
    // row (l % 16) of the C block and the four consecutive columns 4 * (l / 16) + {0,1,2,3}.  The
    // reduction to bytes is that of oz2_bytemod.hpp; the int32 forms use the mulhi reduction of Section 4.3.
    template <int OUT>
    __device__ __forceinline__ void store(const v4i (&acc)[FM][FN], void *C, int s, int plane, int64_t bm, int64_t bn,
                                          int64_t c_ld, int64_t c_plane, const GemmMods &mods) const {
        const int p = mods.p[s], pv = mods.pinv_prime[s];
        const int64_t c_off = (int64_t)plane * c_plane + bm * c_ld + bn;   // C: [plane][row][column]
        if (OUT == kOutU8 || OUT == kOutU8Fold) {
            const ByteMod b = mods.byte_mod[s];
            // The four residues a lane holds of a block pack into one dword; the lanes l, l + 16, l + 32 and
            // l + 48 hold the four dwords of a row.  Four blocks (side by side, or two by two) are exchanged
            // as a 4 x 4 transposition among these lanes, after which each of them holds a row of one block and
            // stores 16 contiguous bytes: whole 32- or 64-byte sectors of a row per instruction, and the L2
            // does not have to fetch lines to merge 4-byte stores.
            // (Staging the whole uint8 tile through LDS to store 64-byte row segments was measured
            // 3.5 ms slower per launch at 16 x 16384^3.)
            constexpr int ROWS_PER = 4 / FN;                  // block rows per group of four blocks
            const int row = wm * 32 * TM + (FN == 2 ? (lquad >> 1) * 16 : 0) + lrow;
            const int col = wn * 32 * TN + (FN == 2 ? lquad & 1 : lquad) * 16;
            uint8_t *const dst0 = static_cast<uint8_t *>(C) + c_off + (int64_t)row * c_ld + col;
#pragma unroll
            for (int i = 0; i < FM; i += ROWS_PER) {
                uint32_t d[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4i &x = acc[i + g / FN][g % FN];
                    d[g] = byte_mod_pack(x[0], x[1], x[2], x[3], b);
                }
                v4i q = exchange_quarters(d);
                v4i *dst = reinterpret_cast<v4i *>(dst0 + (int64_t)(i * 16) * c_ld);
                if (OUT == kOutU8Fold) {                   // a further K range: (old + new) mod p_s, byte by byte
                    const v4i old = *dst;
#pragma unroll
                    for (int w = 0; w < 4; ++w) q[w] = (int)add_mod_bytes((uint32_t)q[w], (uint32_t)old[w], p);
                }
                *dst = q;
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int row = wm * 32 * TM + i * 16 + lrow;
                const int col = wn * 32 * TN + j * 16 + 4 * lquad;
                v4i v = acc[i][j];
                v4i *dst = reinterpret_cast<v4i *>(static_cast<int32_t *>(C) + c_off + (int64_t)row * c_ld + col);
                if (OUT == kOutI32Fold) {
                    const v4i old = *dst;
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] = mod_small(old[c], p, pv) + mod_small(v[c], p, pv);
                }
                *dst = v;
            }
    }
};

// One workgroup per output tile.  For kOutMax the arguments mean: C = the row maxima of the
// panel's rows, C + c_plane (in ints) = the column maxima of its columns, c_ld = the number of
// valid rows of the panel in its low and of valid columns in its high 32 bits.
template <int WM, int WN, int TM, int TN, int BK, int STAGES, int OUT>
__global__ __launch_bounds__(64 * WM * WN) void k_int8_gemm(const int8_t *__restrict__ A,
                                                   const int8_t *__restrict__ B,
                                                   void *__restrict__ C, int64_t Mp,
                                                   int64_t Np, int64_t KB, int kb0,
                                                   int64_t c_ld, int64_t c_plane,
                                                   GemmGrid grid, GemmMods mods) {
    typedef GemmCore<WM, WN, TM, TN, BK, STAGES> Core;
    if (OUT == kOutU8 && Core::BM < kPadMN && (int)blockIdx.x >= grid.map.total) {
        const GemmItem it = padding_item(grid, (int)blockIdx.x - grid.map.total);
        uint8_t *const u = static_cast<uint8_t *>(C) + it.plane * c_plane + (int64_t)it.tr * Core::BM * c_ld + it.tc * Core::BN;
        for (int q = threadIdx.x; q < Core::BM * Core::BN / 16; q += Core::THREADS)
            *reinterpret_cast<v4i *>(u + q / (Core::BN / 16) * c_ld + q % (Core::BN / 16) * 16) = v4i{0, 0, 0, 0};
        return;
    }
    const Core core(Mp, Np);
    const GemmItem it = map_item(grid, (int)blockIdx.x);
    const int8_t *src = core.tile_source(A, B, it.s, it.tr, it.tc, Mp, Np, KB, kb0 + it.kb);
    core.issue_head(src, it.kt);
    v4i acc[Core::FM][Core::FN];
    core.contract(src, it.kt, first_acc(OUT), acc);
    const int64_t bm = (int64_t)it.tr * Core::BM, bn = (int64_t)it.tc * Core::BN;
    if (OUT == kOutMax) {
        int *rmax = static_cast<int *>(C);
        core.store_maxima(acc, rmax, rmax + c_plane, bm, bn, (int)(c_ld & 0xffffffff), (int)(c_ld >> 32));
    } else {
        core.template store<OUT>(acc, C, it.s, it.plane, bm, bn, c_ld, c_plane, mods);
    }
}

// The same as a persistent grid, for short contractions: as many workgroups as compute units,
// each walking over the tiles id = blockIdx.x, blockIdx.x + gridDim.x, ...  The head of the next
// tile (its first STAGES - 1 K tiles) is requested before the results of the last one are
// reduced and stored, and no workgroup is dispatched per tile.  With a short k a tile is a few
// microseconds of matrix-core work, so that the dispatch between tiles and the wait for the
// first operands weigh as much as the contraction.  For long contractions the two forms take the same time (the
// store phase, which nothing overlaps in either form, is what a tile costs beyond its K loop),
// so the plain one-workgroup-per-tile kernel is kept there.  Prepared operands, us, one workgroup per tile | this form: 8192 x 8192 x 128
// N = 15 649 | 584, x 512 930 | 886, x 1024 1287 | 1228, x 2048 1898 | 1848, x 4096 3180 | 3138, x 6144 4492 | 4477 (on another card 4507 | 4538);
// 2048 x 2048 x 512 N = 15 67.6 | 64.0; 2048^3 N = 14 129 | 125, 4096^3 N = 14 773 | 755; 8192^3 N = 8 3197 | 3190 (3215 | 3234), 4096 x 4096 x 8192 FP32 N = 8
// 798 | 814, 1536 x 1000 x 40000 N = 18 865 | 878.
template <int WM, int WN, int TM, int TN, int BK, int STAGES, int OUT>
__global__ __launch_bounds__(64 * WM * WN) void k_int8_gemm_persistent(const int8_t *__restrict__ A,
                                                   const int8_t *__restrict__ B,
                                                   void *__restrict__ C, int64_t Mp,
                                                   int64_t Np, int64_t KB, int kb0, int KT,
                                                   int64_t c_ld, int64_t c_plane,
                                                   TileMap tmap, GemmMods mods) {
    typedef GemmCore<WM, WN, TM, TN, BK, STAGES> Core;
    static_assert(OUT != kOutMax, "the maxima form runs one workgroup per tile");
    const Core core(Mp, Np);
    int tile = (int)blockIdx.x;
    int s, tile_r, tile_c;
    map_tile(tmap, tile, s, tile_r, tile_c);
    const int8_t *src = core.tile_source(A, B, s, tile_r, tile_c, Mp, Np, KB, kb0);
    core.issue_head(src, KT);
    bool stores = false;                                   // the previous tile's stores may be on their way
    for (;;) {
        // Where the next tile starts is worked out while the head of this one travels.
        const int next = tile + (int)gridDim.x;
        int s_next = 0, tile_r_next = 0, tile_c_next = 0;
        const int8_t *src_next = nullptr;
        if (next < tmap.total) {
            map_tile(tmap, next, s_next, tile_r_next, tile_c_next);
            src_next = core.tile_source(A, B, s_next, tile_r_next, tile_c_next, Mp, Np, KB, kb0);
        }
        v4i acc[Core::FM][Core::FN];
        // kStores: the number of store instructions of store<kOutU8>, one of 16 bytes per 32 x 32 block of a
        // wavefront.  (The fold forms also load what they add to, and wait for it themselves.)
        constexpr int kStores = OUT == kOutU8 ? TM * TN : 0;
        core.template contract<kStores>(src, KT, first_acc(OUT), acc, stores);
        // Every wavefront has passed the last barrier, so nothing reads the LDS stages any more:
        // the head of this workgroup's next tile is requested now and travels while the results
        // of this one are reduced and stored.
        if (next < tmap.total) core.issue_head(src_next, KT);
        // contract<kStores> takes the stores for younger than all of the head's loads: none may move across.
        pin_memory_order();
        core.template store<OUT>(acc, C, s, s, (int64_t)tile_r * Core::BM, (int64_t)tile_c * Core::BN, c_ld, c_plane,
                                 mods);
        pin_memory_order();
        if (next >= tmap.total) break;                    // uniform over the workgroup
        stores = true;
        tile = next; s = s_next; tile_r = tile_r_next; tile_c = tile_c_next; src = src_next;
    }
}

// Compute units of the current device (cached per device id).
int compute_units() {
    static thread_local int cached_dev = -1, cached = 0;     // contexts may launch from several threads
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (dev != cached_dev) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        cached = n; cached_dev = dev;
    }
    return cached;
}

// What the launches of one product (or one slice of it) have in common.
struct GemmLaunch {
    const int8_t *A, *B;
    void *C;
    int batch;
    int64_t Mp, Np, Kp, k_begin, k_len;
    GemmPanel pn;
    int ranges;                                               // K ranges with planes of their own
    GemmMods mods;
    hipStream_t stream;
};

template <typename Kernel>
hipError_t allow_lds(Kernel kernel, size_t bytes, int &attr_device) {
    int dev = -1;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    if (attr_device != dev) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
        attr_device = dev;
    }
    return hipSuccess;
}

// The tiles of a launch; false: more than an int can number (with a grid's stride to spare).
inline bool tiles_of(const GemmLaunch &g, int tile, GemmGrid *grid) {
    const int64_t total = (g.pn.rows / tile) * (g.pn.cols / tile) * g.batch * g.ranges;
    if (total > 0x7fff0000) return false;
    *grid = make_gemm_grid(g.pn.rows, g.pn.cols, g.pn.valid_rows, g.pn.valid_cols, tile, g.batch, g.ranges, (int)(g.k_len / kBlockK));
    return true;
}

template <int WM, int WN, int TM, int TN, int BK, int STAGES, int OUT>
hipError_t launch_persistent(const GemmLaunch &g) {
    constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
    constexpr size_t lds_bytes = (size_t)STAGES * (BM + BN) * BK;
    static_assert(lds_bytes > 80 * 1024, "one workgroup per compute unit is assumed");
    static thread_local int attr_device = -1;                // the attribute is per device (set again per thread: harmless)
    if (hipError_t e = allow_lds(&k_int8_gemm_persistent<WM, WN, TM, TN, BK, STAGES, OUT>, lds_bytes, attr_device)) return e;
    GemmGrid grid;
    if (!tiles_of(g, BM, &grid)) return hipErrorInvalidValue;
    const TileMap &tm = grid.map;
    // The grid is a multiple of 8, so that tile id -> XCD stays id mod 8 as in the tile map.
    const int units = compute_units() / 8 * 8;
    if (units < 8) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_int8_gemm_persistent<WM, WN, TM, TN, BK, STAGES, OUT>), dim3((unsigned)std::min(tm.total, units)),
                       dim3(64 * WM * WN), lds_bytes, g.stream, g.A + g.pn.row0 * BK, g.B + g.pn.col0 * BK, g.C, g.Mp, g.Np, g.Kp / BK,
                       (int)(g.k_begin / BK), (int)(g.k_len / BK), g.pn.c_ld, g.pn.c_plane, tm, g.mods);
    return hipGetLastError();
}

template <int WM, int WN, int TM, int TN, int BK, int STAGES, int OUT>
hipError_t launch(const GemmLaunch &g) {
    constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
    constexpr size_t lds_bytes = (size_t)STAGES * (BM + BN) * BK;
    static thread_local int attr_device = -1;                // the attribute is per device (set again per thread: harmless)
    if (hipError_t e = allow_lds(&k_int8_gemm<WM, WN, TM, TN, BK, STAGES, OUT>, lds_bytes, attr_device)) return e;
    GemmGrid grid;
    if (!tiles_of(g, BM, &grid)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_int8_gemm<WM, WN, TM, TN, BK, STAGES, OUT>), dim3((unsigned)(grid.map.total + (OUT == kOutU8 ? grid.padding : 0))),
                       dim3(64 * WM * WN), lds_bytes, g.stream, g.A + g.pn.row0 * BK, g.B + g.pn.col0 * BK, g.C, g.Mp, g.Np, g.Kp / BK,
                       (int)(g.k_begin / BK), g.pn.c_ld, g.pn.c_plane, grid, g.mods);
    return hipGetLastError();
}

template <int OUT>
hipError_t launch_out(const GemmLaunch &g) {
    // (The maxima by the padded extents: with 8 wavefronts there are more atomic maxima per tile, and 628 x 6208 x 205 took 11.7 us in 245 workgroups
    // of them, one per compute unit, and 7.7 with 4 wavefronts.)
    const GemmTile tile = gemm_plan(OUT == kOutMax ? g.pn.rows : g.pn.valid_rows, OUT == kOutMax ? g.pn.cols : g.pn.valid_cols, g.batch,
                                    g.k_len / kBlockK, g.ranges > 1).tile;
    if (tile == GemmTile::kOnePerUnit) return launch<2, 4, 2, 1, 64, 6, OUT>(g);
    if (tile == GemmTile::kTwoPerUnit) return launch<2, 2, 2, 2, 64, 4, OUT>(g);
    if constexpr (OUT == kOutU8 || OUT == kOutU8Fold) {
        GemmGrid grid;
        if (!tiles_of(g, 256, &grid)) return hipErrorInvalidValue;
        if (wide_gemm_applies(grid.map.total, g.k_len, g.ranges)) {
            const int units = compute_units() / 8 * 8;
            if (units < 8) return hipErrorInvalidValue;
            WideMods mods{};
            for (int i = 0; i < g.batch; ++i) { mods.p[i] = g.mods.p[i]; mods.byte_mod[i] = make_byte_mod(g.mods.p[i], kWideFirst); }
            return launch_wide_gemm(g.A + g.pn.row0 * kBlockK, g.B + g.pn.col0 * kBlockK, static_cast<uint8_t *>(g.C), g.Mp, g.Np, g.Kp / kBlockK,
                                    (int)(g.k_begin / kBlockK), g.pn.c_ld, g.pn.c_plane, grid, mods, OUT == kOutU8Fold, units, g.stream);
        }
    }
    // 8 wavefronts (2 per SIMD), each 128 x 64
    if constexpr (OUT != kOutMax)
        if (g.k_len <= kPersistentMaxK && g.ranges == 1)   // short contraction: see k_int8_gemm_persistent
            return launch_persistent<2, 4, 4, 2, 64, 4, OUT>(g);
    return launch<2, 4, 4, 2, 64, 4, OUT>(g);
}

// Whole tiles that exist, and at least a row and a column in the last of them.
bool panel_fits(const GemmPanel &pn, int64_t Mp, int64_t Np) {
    return pn.row0 >= 0 && pn.col0 >= 0 && pn.rows >= kPadMN && pn.cols >= kPadMN && pn.row0 % kPadMN == 0 && pn.col0 % kPadMN == 0 &&
           pn.rows % kPadMN == 0 && pn.cols % kPadMN == 0 && pn.row0 + pn.rows <= Mp && pn.col0 + pn.cols <= Np &&
           pn.valid_rows > pn.rows - kPadMN && pn.valid_rows <= pn.rows && pn.valid_cols > pn.cols - kPadMN && pn.valid_cols <= pn.cols;
}

}  // namespace

hipError_t launch_int8_gemm_maxima(const int8_t *A, const int8_t *B, int64_t Mp, int64_t Np, int64_t Kp,
                                   int64_t k_begin, int64_t k_len, const GemmPanel &pn, int *row_max, int *col_max,
                                   hipStream_t stream) {
    if (!panel_fits(pn, Mp, Np) || k_begin < 0 || k_len < kPadK || k_len > kMaxExactK || k_begin % kPadK ||
        k_len % kPadK || k_begin + k_len > Kp || !row_max || !col_max)
        return hipErrorInvalidValue;
    // the kernel's view of these arguments: see kOutMax
    GemmLaunch g{A, B, row_max, 1, Mp, Np, Kp, k_begin, k_len, pn, 1, GemmMods{}, stream};
    g.pn.c_ld = pn.valid_rows | (pn.valid_cols << 32);
    g.pn.c_plane = col_max - row_max;
    return launch_out<kOutMax>(g);
}

hipError_t launch_int8_gemm(const int8_t *A, const int8_t *B, void *C, int batch, int64_t Mp,
                            int64_t Np, int64_t Kp, int64_t k_begin, int64_t k_len, bool as_u8,
                            bool fold, const ModArgs *ma, hipStream_t stream, const GemmPanel *panel, int ranges) {
    const GemmPanel pn = panel ? *panel : GemmPanel{0, Mp, 0, Np, Np, Mp * Np, Mp, Np};
    if (!panel_fits(pn, Mp, Np) || pn.c_ld < pn.cols || pn.c_ld % 16 || pn.c_plane % 16)
        return hipErrorInvalidValue;                       // whole tiles, 16-byte stores
    if (ranges < 1 || (ranges > 1 && (!as_u8 || fold || k_len / kBlockK < 2 * ranges))) return hipErrorInvalidValue;
    GemmLaunch g{A, B, C, batch, Mp, Np, Kp, k_begin, k_len, pn, ranges, GemmMods{}, stream};
    if (ma)
        for (int i = 0; i < ma->n; ++i) {
            g.mods.p[i] = ma->p[i]; g.mods.pinv_prime[i] = (int32_t)ma->pinv_prime[i];
            g.mods.byte_mod[i] = make_byte_mod(ma->p[i]);
        }
    else if (as_u8 || fold)
        return hipErrorInvalidValue;                       // the reduced forms need the moduli
    if (as_u8) return fold ? launch_out<kOutU8Fold>(g) : launch_out<kOutU8>(g);
    // (the int32 forms compute the products of the padding, too)
    g.pn.valid_rows = pn.rows; g.pn.valid_cols = pn.cols;
    return fold ? launch_out<kOutI32Fold>(g) : launch_out<kOutI32>(g);
}

}  // namespace oz2
