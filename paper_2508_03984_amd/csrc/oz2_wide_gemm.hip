// The INT8 GEMM on tiles of 256 x 256 by 4 wavefronts of 128 x 128, one per SIMD (Algorithm 1 lines 6-7, uint8 forms).
//
// Against the 8 wavefronts of 128 x 64 of oz2_int8_gemm.hip: a third less fragment reads from LDS, and a wavefront has a SIMD's 512
// registers: 256 accumulators, the fragments of two K tiles, and what the reduction of a tile needs beside them.  So
//   - the fragments of a K tile are read during the whole K tile before it and no MFMA waits for LDS; a stage of LDS is free
//     for the next load one K tile earlier, which puts three K tiles in flight into the same four stages;
//   - K tiles form one stream across the output tiles of a workgroup: the first ones of the next tile are requested during the last
//     ones of the present one, at the same pace (the head of a tile at once, 128 loads per compute unit, took 3600 cycles);
//   - a tile is reduced to bytes and stored beside the MFMAs of its last and of the next tile's first K tile.
// One wavefront per SIMD issues an instruction every 4 to 5 cycles and an MFMA takes 16, so everything else stands between the MFMAs at
// an even pace, in the order written (all 8 loads of a K tile at once cost 15 %, 64-bit addresses in vector registers 2 %).
//
// Accumulators: a0 to a255, named in the assembly of the MFMAs.  As values of the compiler's they were copied and spilled wherever
// two forms of a K tile meet.  Nothing else in these kernels uses an AGPR or M0, which the tests read from the assembly.
//
// The sums start at -2^30 (0xc0000000, which as binary32 is the inline constant -2.0: a register quad for it would be four AGPRs too
// many), so that u = x + 3 2^30 is what byte_mod works on.  |x| <= 2^30 for k <= 65536 = kWideMaxK: 127^2 k < 2^30 for the odd moduli; the
// sum of 2^30 that p = 256 allows wraps to 0, the same class.
//
// Bound: board power for long contractions.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "oz2_epilogue.hpp"
#include "oz2_wide_gemm.hpp"

namespace oz2 {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

// f(integral_constant 0), ..., f(integral_constant N - 1)
template <typename F, int... I>
__device__ __forceinline__ void static_for_(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) { static_for_(f, std::make_integer_sequence<int, N>{}); }

// Waits for vmcnt <= vm and lgkmcnt = 0 (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).
constexpr int wait_imm(int vm) { return (vm & 0xf) | ((vm >> 4) << 14) | (0x7 << 4); }

__device__ __forceinline__ void pin_memory_order() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// (the swizzle of the 16-byte chunks of a row: see oz2_int8_gemm.hip)
__device__ inline int swizzle_mask(int row) {
    const int quad = row >> 2;
    return ((quad ^ (quad >> 1)) & 1) << 1 | (quad >> 1 & 1);
}

extern __shared__ v4i lds[];                                  // [STAGES][A rows | B rows][64 bytes]

struct WideCore {
    static constexpr int BM = 256, BN = 256, BK = kBlockK, STAGES = 4, THREADS = 256;
    static constexpr int LOADS = 8;                           // of a wavefront and K tile, 1 KiB each
    static constexpr int F = 8;                               // fragments of 16 rows (columns) of a wavefront
    static constexpr int STORES = 16;                         // of a wavefront and tile, 16 bytes per lane each
    static constexpr int STAGE_BYTES = (BM + BN) * BK;
    static_assert(BK == 64 && STAGE_BYTES == THREADS / 64 * LOADS * 1024, "");

    int wm, wn, lrow, lquad;
    int row0, lane_off, my_dst;                               // first row of the wavefront's loads; a lane's place in them; in a stage
    int a_addr, b_addr;                                       // fragments: byte offsets within a stage
    bool from_a;                                              // uniform over the wavefront: rows 0 to 255 of a stage are A's
    int64_t tile_step;                                        // next K block of the same rows

    __device__ __forceinline__ WideCore(int64_t Mp, int64_t Np) {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        wm = wave >> 1; wn = wave & 1;
        row0 = wave * 128;
        from_a = row0 < BM;
        tile_step = (from_a ? Mp : Np) * BK;
        my_dst = wave * LOADS * 1024;
        lane_off = (lane >> 2) * BK + ((lane & 3) ^ swizzle_mask(lane >> 2)) * 16;
        lrow = lane & 15; lquad = lane >> 4;
        const int c = lquad ^ swizzle_mask(lrow);
        a_addr = ((wm * 128 + lrow) * 4 + c) * 16;
        b_addr = ((BM + wn * 128 + lrow) * 4 + c) * 16;
    }

    // Where this wavefront's loads of an item start (uniform).
    __device__ __forceinline__ const int8_t *source(const int8_t *A, const int8_t *B, const GemmItem &it, int64_t Mp, int64_t Np,
                                                    int64_t KB, int kb0) const {
        const int64_t kb = (int64_t)it.s * KB + kb0 + it.kb;
        return from_a ? A + (kb * Mp + (int64_t)it.tr * BM + row0) * BK : B + (kb * Np + (int64_t)it.tc * BN + row0 - BM) * BK;
    }

    // Load H of a K tile.  The immediate offset applies to both addresses and M0 stays for four of them.
    template <int H>
    __device__ __forceinline__ void load(const int8_t *src, int stage_off) const {
        const uint32_t dst = (uint32_t)(uintptr_t)(lds_ptr_t)lds + stage_off + my_dst + H / 4 * 4096;
        const int8_t *const base = src + H / 4 * 4096;
        if constexpr (H % 4 == 0)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(lane_off), "s"(base) : "memory");
        else
            asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(lane_off), "s"(base), "n"(H % 4 * 1024) : "memory");
    }

    struct Fragments {
        v4i a[2][F], b[2][F];                                 // of the K tile at hand and of the next one
    };
    // Fragment U of a K tile, in the order in which the MFMAs use them.
    template <int SET, int U>
    __device__ __forceinline__ void read(Fragments &f, int stage_off) const {
        const char *const l = reinterpret_cast<const char *>(lds) + stage_off;
        if constexpr (U < 2) f.a[SET][U] = *reinterpret_cast<const v4i *>(l + a_addr + U * 1024);
        else if constexpr (U < 10) f.b[SET][U - 2] = *reinterpret_cast<const v4i *>(l + b_addr + (U - 2) * 1024);
        else f.a[SET][U - 8] = *reinterpret_cast<const v4i *>(l + a_addr + (U - 8) * 1024);
    }

    // Accumulator (i, j), the transposed 16 x 16 block of fragments i of A and j of B, is a[32 i + 4 j] to a[32 i + 4 j + 3].
    template <int I, int J, bool OPENS>
    static __device__ __forceinline__ void mfma(const v4i &b, const v4i &a) {
        constexpr int lo = 32 * I + 4 * J, hi = lo + 3;
        if constexpr (OPENS) asm volatile("v_mfma_i32_16x16x64_i8 a[%2:%3], %0, %1, -2.0" ::"v"(b), "v"(a), "n"(lo), "n"(hi));
        else asm volatile("v_mfma_i32_16x16x64_i8 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(b), "v"(a), "n"(lo), "n"(hi));
    }
    // Step T of the 32 of a K tile: two MFMAs, rows of blocks 2 (T / 8) and the one after, column T % 8 (a column starts with
    // the row that the last one ended with).
    template <bool OPENS, int SET, int T>
    __device__ __forceinline__ void mfmas(const Fragments &f) const {
        constexpr int j = T % 8, i0 = T / 8 * 2 + (j & 1), i1 = T / 8 * 2 + 1 - (j & 1);
        mfma<i0, j, OPENS>(f.b[SET][j], f.a[SET][i0]);
        mfma<i1, j, OPENS>(f.b[SET][j], f.a[SET][i1]);
        __builtin_amdgcn_sched_barrier(0);
    }

    // A K tile, whose fragments are in set SET: those of the next K tile are read (READS), the K tile 4 ahead (src) goes into the stage
    // of this one, which nobody reads any more (LOADS_AHEAD), and `beside` adds what else there is to do at step T.  At its end, all but the youngest
    // WAIT memory instructions of this wavefront (STORES more if `stores`) are complete; that has to include the loads of the K tile after
    // the next one.
    template <bool OPENS, int SET, int WAIT, bool READS = true, bool LOADS_AHEAD = true, typename Beside>
    __device__ __forceinline__ void k_tile(Fragments &f, int &stage_off, const int8_t *src, Beside &&beside, bool stores = false) const {
        const int next_off = stage_off == (STAGES - 1) * STAGE_BYTES ? 0 : stage_off + STAGE_BYTES;
        static_for<32>([&](auto step) {
            constexpr int T = decltype(step)::value;
            mfmas<OPENS, SET, T>(f);
            if constexpr (READS && T % 3 != 2 && T / 3 * 2 + T % 3 < 2 * F) read<SET ^ 1, T / 3 * 2 + T % 3>(f, next_off);
            if constexpr (LOADS_AHEAD && T % 4 == 1) load<T / 4>(src, stage_off);
            beside(step);
            __builtin_amdgcn_sched_barrier(0);
        });
        if (stores) __builtin_amdgcn_s_waitcnt(wait_imm(WAIT + STORES));
        else __builtin_amdgcn_s_waitcnt(wait_imm(WAIT));
        __builtin_amdgcn_s_barrier();
        stage_off = next_off;
    }

    // The reduction of a tile to bytes (oz2_bytemod.hpp) and its stores, in kPieces pieces of about four instructions: 20 for each of
    // 16 groups of 16 entries (row of blocks G / 2, four blocks of it).  As in byte_mod_pack, with each kind of instruction for the
    // whole group, so that nothing waits for the one before it.
    static constexpr int kGroupPieces = 20, kPieces = 16 * kGroupPieces;
    struct Reduction {
        uint32_t x[16], f[16], w[16];
        float q[16];
    };
    template <int N>
    static __device__ __forceinline__ uint32_t accumulator() {
        uint32_t x;
        asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(x) : "n"(N));
        return x;
    }
    template <bool FOLD, int N>
    static __device__ __forceinline__ void piece(Reduction &r, const ByteMod &b, int fold_p, uint8_t *dst0, int64_t c_ld) {
        constexpr int G = N / kGroupPieces, m = N % kGroupPieces;
        if constexpr (m < 4) {
            static_assert(4 * F == 32, "");
            r.x[4 * m] = accumulator<16 * G + 4 * m>();
            r.x[4 * m + 1] = accumulator<16 * G + 4 * m + 1>();
            r.x[4 * m + 2] = accumulator<16 * G + 4 * m + 2>();
            r.x[4 * m + 3] = accumulator<16 * G + 4 * m + 3>();
        } else if constexpr (m < 8) {
#pragma unroll
            for (int e = 4 * (m - 4); e < 4 * (m - 3); ++e) r.f[e] = __builtin_amdgcn_udot4(r.x[e], b.coef, b.base, false);
        } else if constexpr (m < 12) {
#pragma unroll
            for (int e = 4 * (m - 8); e < 4 * (m - 7); ++e) r.q[e] = __builtin_fmaf(__builtin_bit_cast(float, r.f[e]), b.pinv, b.magic);
        } else if constexpr (m < 16) {
#pragma unroll
            for (int e = 4 * (m - 12); e < 4 * (m - 11); ++e) r.w[e] = (uint32_t)__mul24(__builtin_bit_cast(int, r.q[e]), b.neg_p) + r.f[e];
        } else if constexpr (m < 18) {                        // the low bytes of four words in one, first in pairs
#pragma unroll
            for (int h = 4 * (m - 16); h < 4 * (m - 15); ++h) r.x[h] = __builtin_amdgcn_perm(r.w[2 * h + 1], r.w[2 * h], 0x0c0c0400u);
        } else if constexpr (m == 18) {
#pragma unroll
            for (int h = 0; h < 4; ++h) r.f[h] = __builtin_amdgcn_perm(r.x[2 * h + 1], r.x[2 * h], 0x05040100u);
        } else {
            const uint32_t d[4] = {r.f[0], r.f[1], r.f[2], r.f[3]};
            v4i q = exchange_quarters(d);
            v4i *const dst = reinterpret_cast<v4i *>(dst0 + (int64_t)(G / 2 * 16) * c_ld + G % 2 * 64);
            if (FOLD) {                                       // a further K range: (old + new) mod p_s, byte by byte
                const v4i old = *dst;
#pragma unroll
                for (int w = 0; w < 4; ++w) q[w] = (int)add_mod_bytes((uint32_t)q[w], (uint32_t)old[w], fold_p);
            }
            *dst = q;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    template <bool FOLD, int FROM, int TO>
    static __device__ __forceinline__ void pieces(Reduction &r, const ByteMod &b, int fold_p, uint8_t *dst0, int64_t c_ld) {
        static_for<TO - FROM>([&](auto n) { piece<FOLD, FROM + decltype(n)::value>(r, b, fold_p, dst0, c_ld); });
    }
};

#define OZ2_TEN(n) "a" #n "0", "a" #n "1", "a" #n "2", "a" #n "3", "a" #n "4", "a" #n "5", "a" #n "6", "a" #n "7", "a" #n "8", "a" #n "9"
__device__ __forceinline__ void claim_accumulators() {
    asm volatile("" ::: "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", OZ2_TEN(1), OZ2_TEN(2), OZ2_TEN(3), OZ2_TEN(4), OZ2_TEN(5),
                 OZ2_TEN(6), OZ2_TEN(7), OZ2_TEN(8), OZ2_TEN(9), OZ2_TEN(10), OZ2_TEN(11), OZ2_TEN(12), OZ2_TEN(13), OZ2_TEN(14), OZ2_TEN(15),
                 OZ2_TEN(16), OZ2_TEN(17), OZ2_TEN(18), OZ2_TEN(19), OZ2_TEN(20), OZ2_TEN(21), OZ2_TEN(22), OZ2_TEN(23), OZ2_TEN(24), "a250",
                 "a251", "a252", "a253", "a254", "a255");
}
#undef OZ2_TEN

// A workgroup per compute unit at most, each walking over the items blockIdx.x, blockIdx.x + gridDim.x, ...  Every item has an
// even number of K tiles, at least kWideMinKTiles.
template <bool FOLD>
__global__ __launch_bounds__(WideCore::THREADS, 1) void k_wide_gemm(const int8_t *__restrict__ A, const int8_t *__restrict__ B,
                                                                    uint8_t *__restrict__ C, int64_t Mp, int64_t Np, int64_t KB, int kb0,
                                                                    int64_t c_ld, int64_t c_plane, GemmGrid grid, WideMods mods) {
    typedef WideCore W;
    // What stays outstanding at the end of a K tile: the two youngest K tiles; after the first two of a tile also the stores of the tile
    // before, if there is one, which are younger than the loads those two wait for.
    constexpr int kYoungest = 2 * W::LOADS;
    static_assert(kYoungest + W::STORES < 64, "vmcnt is a 6-bit counter");
    claim_accumulators();
    const W core(Mp, Np);
    int id = (int)blockIdx.x;
    GemmItem it = map_item(grid, id);
    const int8_t *src = core.source(A, B, it, Mp, Np, KB, kb0);
    static_for<W::STAGES * W::LOADS>([&](auto n) {
        constexpr int t = decltype(n)::value / W::LOADS, h = decltype(n)::value % W::LOADS;
        core.template load<h>(src + t * core.tile_step, t * W::STAGE_BYTES);
    });
    W::Fragments f;
    __builtin_amdgcn_s_waitcnt(wait_imm(3 * W::LOADS));       // K tile 0
    __builtin_amdgcn_s_barrier();
    static_for<2 * W::F>([&](auto u) { core.template read<0, decltype(u)::value>(f, 0); });
    __builtin_amdgcn_s_waitcnt(wait_imm(kYoungest));          // K tile 1
    __builtin_amdgcn_s_barrier();
    int stage_off = 0;
    const auto nothing = [](auto) {};
    src += W::STAGES * core.tile_step;                        // the K tile that is requested next
    core.template k_tile<true, 0, kYoungest>(f, stage_off, src, nothing);
    src += core.tile_step;
    for (bool stores = false;; stores = true) {
        const int next = id + (int)gridDim.x;
        const bool more = next < grid.map.total;              // uniform over the workgroup
        core.template k_tile<false, 1, kYoungest>(f, stage_off, src, nothing, stores);
        src += core.tile_step;
        for (int kt = 2; kt + W::STAGES < it.kt; kt += 2) {
            core.template k_tile<false, 0, kYoungest>(f, stage_off, src, nothing);
            src += core.tile_step;
            core.template k_tile<false, 1, kYoungest>(f, stage_off, src, nothing);
            src += core.tile_step;
        }
        const ByteMod b = mods.byte_mod[it.s];
        const int fold_p = FOLD ? mods.p[it.s] : 0;
        uint8_t *const dst0 = C + (int64_t)it.plane * c_plane + ((int64_t)it.tr * W::BM + core.wm * 128 + core.lrow) * c_ld +
                              (int64_t)it.tc * W::BN + core.wn * 128 + core.lquad * 16;
        // In the last K tile the reduction begins with what its first steps complete, up to the first store.
        constexpr int kBeside = W::kGroupPieces - 1, kFirstStep = 10;
        static_assert(kFirstStep + kBeside <= 32, "");
        W::Reduction r;
        const auto begin = [&](auto step) {
            constexpr int n = decltype(step)::value - kFirstStep;
            if constexpr (n >= 0 && n < kBeside) W::piece<FOLD, n>(r, b, fold_p, dst0, c_ld);
        };
        if (!more) {
            core.template k_tile<false, 0, W::LOADS, true, false>(f, stage_off, src, nothing);
            core.template k_tile<false, 1, 0, true, false>(f, stage_off, src, nothing);
            core.template k_tile<false, 0, 0, true, false>(f, stage_off, src, nothing);
            core.template k_tile<false, 1, 0, false, false>(f, stage_off, src, begin);
            W::pieces<FOLD, kBeside, W::kPieces>(r, b, fold_p, dst0, c_ld);
            break;
        }
        // The last four K tiles request the first four of the next item.
        it = map_item(grid, next);
        src = core.source(A, B, it, Mp, Np, KB, kb0);
        core.template k_tile<false, 0, kYoungest>(f, stage_off, src, nothing);
        src += core.tile_step;
        core.template k_tile<false, 1, kYoungest>(f, stage_off, src, nothing);
        src += core.tile_step;
        core.template k_tile<false, 0, kYoungest>(f, stage_off, src, nothing);
        src += core.tile_step;
        core.template k_tile<false, 1, kYoungest>(f, stage_off, src, begin);
        pin_memory_order();
        src += core.tile_step;
        // Rows of blocks 0 and 1, then the next tile's first K tile, whose MFMAs of two rows of blocks follow the reduction of these.
        constexpr int kRows = 4 * W::kGroupPieces, kPace = kRows / 8;
        W::pieces<FOLD, kBeside, kRows>(r, b, fold_p, dst0, c_ld);
        core.template k_tile<true, 0, kYoungest>(f, stage_off, src, [&](auto step) {
            constexpr int from = kRows + decltype(step)::value * kPace;
            if constexpr (from < W::kPieces) W::pieces<FOLD, from, from + kPace>(r, b, fold_p, dst0, c_ld);
        }, true);
        pin_memory_order();
        src += core.tile_step;
        id = next;
    }
}

}  // namespace

hipError_t launch_wide_gemm(const int8_t *A, const int8_t *B, uint8_t *C, int64_t Mp, int64_t Np, int64_t KB, int kb0, int64_t c_ld,
                            int64_t c_plane, const GemmGrid &grid, const WideMods &mods, bool fold, int units, hipStream_t stream) {
    constexpr size_t lds_bytes = (size_t)WideCore::STAGES * WideCore::STAGE_BYTES;
    static thread_local int attr_device = -1;                // the attribute is per device (set again per thread: harmless)
    int dev = -1;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    if (attr_device != dev) {
        for (const void *kernel : {reinterpret_cast<const void *>(&k_wide_gemm<false>), reinterpret_cast<const void *>(&k_wide_gemm<true>)})
            if (hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes)) return e;
        attr_device = dev;
    }
    const dim3 blocks((unsigned)std::min(grid.map.total, units));
    if (fold)
        hipLaunchKernelGGL((k_wide_gemm<true>), blocks, dim3(WideCore::THREADS), lds_bytes, stream, A, B, C, Mp, Np, KB, kb0, c_ld, c_plane, grid, mods);
    else
        hipLaunchKernelGGL((k_wide_gemm<false>), blocks, dim3(WideCore::THREADS), lds_bytes, stream, A, B, C, Mp, Np, KB, kb0, c_ld, c_plane, grid, mods);
    return hipGetLastError();
}

}  // namespace oz2
