// mod(x, p) of an int32 sum as the low byte of a register: the reduction of Algorithm 1 line 7 in
// the store phase of the INT8 GEMM.  The constants per modulus and the arithmetic, in one place for
// the device and for a host build (no HIP needed), so that the CPU can check every value.
//
// The sums start at -2^31 (oz2_int8_gemm.hip, oz2_tiny.hip) or at -2^30 (oz2_wide_gemm.hip) instead of 0, so that what they hold is, as an
// unsigned number, u = x + first with first = 2^31 or 3 2^30.  Then, with h = (p - 1) / 2:
//   f = t + sum_j byte_j(u) (256^j mod p), one v_dot4_u32_u8.  t in [0, p) is chosen so that
//       f = x - h (mod p); f <= 255 (1 + 3 * 255) + 255 < 2^18;
//   q = round(f / p) by one FMA.  The bits of f are those of the subnormal binary32 number 2^-149 f, so no
//       conversion is needed (subnormals cost nothing and are on in these kernels): times 2^127 / p it is 2^-22 f / p, and the
//       added 3 + 2^-22 j rounds it to a multiple of 2^-22.  f / p is at least 1/(2p) >= 2^-9 away from a
//       half-integer, and the rounded reciprocal misplaces it by less than 2^18 / 173 * 2^-24 < 2^-13;
//   f - p q = mod(x, p) - h.  j is chosen so that -p j = h (mod 256), and what else the two bit
//       patterns hold is a multiple of 256: the low byte of bits(f) - p * bits(q) is mod(x, p).
// p = 256: the coefficients are (1, 0, 0, 0) and t = 0; the low byte of f is the result whatever q is.
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>

namespace oz2 {

struct ByteMod {
    uint32_t coef;                      // 256^j mod p in byte j (p = 256: byte 0 only)
    uint32_t base;                      // t
    float pinv, magic;                  // 2^127 / p; 3 + 2^-22 j
    int32_t neg_p;
};

// first: what the sums start at (u = x + first modulo 2^32, which has to be x + first itself, for p = 256 modulo 256).
inline ByteMod make_byte_mod(int p, uint32_t first = 0x80000000u) {
    ByteMod b{};
    uint32_t power = 1 % p;
    for (int j = 0; j < 4; ++j) { b.coef |= power << (8 * j); power = power * 256u % (uint32_t)p; }
    const int h = (p - 1) / 2;
    // x = u - first, so t = -first - h (mod p)
    const int t = p == 256 ? 0 : (int)((((int64_t)p << 32) - (int64_t)first - h) % p);
    b.base = (uint32_t)t;
    // -p j = h (mod 256): the inverse of an odd p modulo 256 by Newton's iteration (3, 6, 12 bits)
    uint32_t inverse = (uint32_t)p;
    inverse *= 2u - (uint32_t)p * inverse;
    inverse *= 2u - (uint32_t)p * inverse;
    const uint32_t j = p % 2 ? (0u - inverse * (uint32_t)h) & 0xffu : 0u;
    b.pinv = std::ldexp(1.0f, 127) / (float)p;
    b.magic = 3.0f + std::ldexp((float)j, -22);
    b.neg_p = -p;
    return b;
}

// What the device computes from the biased sum u: a word whose low byte is mod(u - first, p).
inline uint32_t byte_mod_word(uint32_t u, const ByteMod &b) {
    uint32_t f = b.base;
    for (int j = 0; j < 4; ++j) f += ((u >> (8 * j)) & 0xffu) * ((b.coef >> (8 * j)) & 0xffu);
    float y, q;
    std::memcpy(&y, &f, 4);
    q = std::fmaf(y, b.pinv, b.magic);
    uint32_t qb;
    std::memcpy(&qb, &q, 4);
    const int32_t q24 = (int32_t)(qb << 8) >> 8;            // the 24-bit operand of v_mad_i32_i24
    return (uint32_t)q24 * (uint32_t)b.neg_p + f;
}

}  // namespace oz2
