// Device code shared by the kernels that end a product (Algorithm 1 lines 6-12): residues of the INT32
// sums as bytes, and the last steps of an entry of C.
#pragma once
#include "oz2_bytemod.hpp"
#include "oz2_kernels.hpp"

namespace oz2 {

// The low bytes of four words in one.
__device__ __forceinline__ uint32_t pack_low_bytes(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) {
    const uint32_t lo = __builtin_amdgcn_perm(w1, w0, 0x0c0c0400u), hi = __builtin_amdgcn_perm(w3, w2, 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// (a + b) mod p on each of the four bytes of a and b, all of them below p <= 256: the even and
// the odd bytes as two pairs of 16-bit sums (at most 510), each reduced by one packed unsigned
// minimum (s - p wraps to a large number when s < p).
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t add_mod_bytes(uint32_t a, uint32_t b, int p) {
    const us2 pp = {(unsigned short)p, (unsigned short)p};
    auto reduce = [&](uint32_t x) {
        const us2 v = __builtin_bit_cast(us2, x);
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(v, (us2)(v - pp)));
    };
    const uint32_t even = reduce((a & 0x00ff00ffu) + (b & 0x00ff00ffu));
    const uint32_t odd = reduce(((a >> 8) & 0x00ff00ffu) + ((b >> 8) & 0x00ff00ffu));
    return even | (odd << 8);
}

// byte_mod_word on the device, for four sums, whose residues come packed: 3.75 vector instructions per entry, none of them a
// 32-bit multiplication (the mulhi form of mod_small has two).  All four v_dot4 first, because what reads the result of one has
// to stay three instructions behind it.  Measured for whole calls, us, mulhi form -> this one with the dot product converted by a
// subtraction: 8192 x 8192 x 512, N = 15, 1299 -> 1245; 4096 x 3072 x 2048 prepared 454 -> 435; then, prepared, without the
// subtraction and without writing the accumulators before the first K tile: 8192 x 8192 x 128 623 -> 590, x 512 924 -> 904, 2048^3
// N = 15 132.5 -> 129.7, 4096^3 N = 14 765 -> 757; no difference at 16384^3, where the store phase is 2 % of a tile.
__device__ __forceinline__ uint32_t byte_mod_pack(int a0, int a1, int a2, int a3, const ByteMod &b) {
    const int acc[4] = {a0, a1, a2, a3};
    uint32_t f[4], w[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) f[c] = __builtin_amdgcn_udot4((uint32_t)acc[c], b.coef, b.base, false);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float q = __builtin_fmaf(__builtin_bit_cast(float, f[c]), b.pinv, b.magic);
        w[c] = (uint32_t)__mul24(__builtin_bit_cast(int, q), b.neg_p) + f[c];
    }
    return pack_low_bytes(w[0], w[1], w[2], w[3]);
}

// The 4 x 4 transposition of words among the lanes l, l + 16, l + 32 and l + 48 (quarters 0 to 3): quarter q gets the four
// quarters' d[q], in ascending order.  v_permlane32_swap(a, b): the upper half of a and the lower half of b change places;
// v_permlane16_swap(a, b): the odd quarters of a and the even quarters of b.
typedef int exchanged_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ exchanged_t exchange_quarters(const uint32_t (&d)[4]) {
    const auto s02 = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false);
    const auto s13 = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
    return exchanged_t{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
}

template <typename OutT>
__device__ inline OutT finish(double c, double alpha, double beta, const OutT *Cin) {
    double r;
    if (beta == 0.0) r = (alpha == 1.0) ? c : alpha * c;
    else r = fma(alpha, c, beta * (double)*Cin);
    return (OutT)r;
}

// Q = rint(P_inv C1), C'' = fma(-P2, Q, fma(-P1, Q, C1) + C2), c = C'' 2^-(tA_i + tB_j), then alpha and beta.
template <typename OutT>
__device__ __forceinline__ OutT crt_entry(double C1, double C2, int shift, const ModArgs &ma, double alpha, double beta,
                                          const OutT *Cin) {
    const double Q = rint(ma.Pinv * C1);
    const double T_ = fma(-ma.P1, Q, C1);
    const double Cpp = fma(-ma.P2, Q, T_ + C2);
    return finish<OutT>(ldexp(Cpp, -shift), alpha, beta, Cin);
}

}  // namespace oz2
