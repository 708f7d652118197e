// 4-bit integer codes as operands of the 6-bit floating-point matrix instruction of gfx950
// (v_mfma_f32_32x32x64_f8f6f4 with E2M3 operands).
//
// E2M3 holds every integer of magnitude 0..15 exactly, in units of 1/8 and with the magnitude itself as the
// five low bits (0..7 are the subnormals m/8, 8..15 are 1 + m/8), so a product of two codes is an exact multiple
// of 1/64 and fp32 sums of up to 2^24 / 64 such units are exact integers.  The instruction multiplies 64
// codes in the time in which the int8 one multiplies 32 (measured: 8 .. 9 PFLOP/s against 3.8 POP/s).
//
// A 32-code operand of a lane is 24 bytes, 32 six-bit fields.  Four packed dwords (32 nibbles) become six dwords:
// every pair of packed dwords (wa, wb) fills three dwords (16 fields).  Which nibble goes to which field is
// chosen so that the fields of wa are where its nibbles already are and those of wb where a rotation by two
// puts them (bit 6 f of the 96 = nibble position, or nibble position - 2 modulo 32):
//     dword 0:  wa nibbles 0, 3, 6 at bits 0, 12, 24;   wb nibbles 2, 5 at 6, 18, low half of nibble 0 at 30
//     dword 1:  wa nibbles 1, 4, 7 at bits 4, 16, 28;   wb high half of nibble 0 at 0, nibbles 3, 6 at 10, 22
//     dword 2:  wa nibbles 2, 5    at bits 8, 20;       wb nibbles 1, 4, 7 at 2, 14, 26
// Both operands use the same order, so it leaves the sums unchanged.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr uint32_t fp6_bits(uint32_t field, int a, int b, int c = -1) {
    return (field << a) | (field << b) | (c >= 0 ? field << c : 0u);
}

// a (32 codes) x b (32 codes) per lane, lane half h holding half of the 64 codes of the step
__device__ __forceinline__ v16f mfma_fp6(const v8i &a, const v8i &b, const v16f &c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 2, 2, 0, 0, 0, 0);
}
// the same with the products of a lane's row of a times 2^(a_exponent - 127), of its column of b times 2^(b_exponent - 127)
__device__ __forceinline__ v16f mfma_fp6_scaled(const v8i &a, const v8i &b, const v16f &c, int a_exponent, int b_exponent) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 2, 2, 0, a_exponent, 0, b_exponent);
}

// Two packed dwords -> three dwords of fields holding code + 8 (0..15, sign bit 0): the offset turns two's
// complement into a magnitude by flipping one bit, which the merging does on the way (7 instructions for 16 codes).
// A sum of products with such an operand exceeds the wanted one by 8 x (sum of the other operand).
// An instruction reads one constant from scalar registers: the masks of the first dword are held in vector registers (the empty
// statements keep the compiler from taking them for constants, which would cost three instructions more).
struct Fp6Masks {
    uint32_t a0 = fp6_bits(15, 0, 12, 24), a1 = fp6_bits(15, 4, 16, 28), a2 = fp6_bits(15, 8, 20);
    __device__ __forceinline__ Fp6Masks() { asm("" : "+v"(a0), "+v"(a1), "+v"(a2)); }
};
// (p & mask) ^ q
__device__ __forceinline__ uint32_t and_xor(uint32_t p, uint32_t mask, uint32_t q) {
    return __builtin_amdgcn_bitop3_b32(p, mask, q, 0x6A);
}
__device__ __forceinline__ void fp6_offset16(const Fp6Masks &m, uint32_t wa, uint32_t wb, int &d0, int &d1, int &d2) {
    const uint32_t r = __builtin_amdgcn_alignbit(wb, wb, 2);   // rotate right by two
    constexpr uint32_t b0 = fp6_bits(15, 6, 18) | (3u << 30), b1 = fp6_bits(15, 10, 22) | 3u, b2 = fp6_bits(15, 2, 14, 26);
    constexpr uint32_t x0 = fp6_bits(8, 0, 12, 24) | fp6_bits(8, 6, 18);
    constexpr uint32_t x1 = fp6_bits(8, 4, 16, 28) | fp6_bits(8, 10, 22) | 2u;
    constexpr uint32_t x2 = fp6_bits(8, 8, 20) | fp6_bits(8, 2, 14, 26);
    d0 = static_cast<int>(and_xor(r, b0, and_xor(wa, m.a0, x0)));
    d1 = static_cast<int>(and_xor(r, b1, and_xor(wa, m.a1, x1)));
    d2 = static_cast<int>(and_xor(r, b2, and_xor(wa, m.a2, x2)));
}

// Two packed dwords -> three dwords of signed fields (sign and magnitude), same order.
__device__ __forceinline__ void fp6_signed16(uint32_t wa, uint32_t wb, int &d0, int &d1, int &d2) {
    const uint32_t sa = (wa >> 3) & 0x11111111u, sb = (wb >> 3) & 0x11111111u;
    const uint32_t ma = (wa ^ ((sa << 4) - sa)) + sa;   // magnitudes 0..8 (no carry leaves a nibble)
    const uint32_t mb = (wb ^ ((sb << 4) - sb)) + sb;
    const uint32_t r = __builtin_amdgcn_alignbit(mb, mb, 2);
    const uint32_t t = __builtin_amdgcn_alignbit(wa, wa, 30);   // sign bits of wa's nibbles, two places up
    constexpr uint32_t a0 = fp6_bits(15, 0, 12, 24), b0 = fp6_bits(15, 6, 18) | (3u << 30);
    constexpr uint32_t a1 = fp6_bits(15, 4, 16, 28), b1 = fp6_bits(15, 10, 22) | 3u;
    constexpr uint32_t a2 = fp6_bits(15, 8, 20), b2 = fp6_bits(15, 2, 14, 26);
    constexpr uint32_t sa0 = fp6_bits(1, 5, 17, 29), sb0 = fp6_bits(1, 11, 23);
    constexpr uint32_t sa1 = fp6_bits(1, 9, 21), sb1 = fp6_bits(1, 3, 15, 27);
    constexpr uint32_t sa2 = fp6_bits(1, 1, 13, 25), sb2 = fp6_bits(1, 7, 19, 31);
    d0 = static_cast<int>((ma & a0) | (r & b0) | (t & sa0) | (wb & sb0));
    d1 = static_cast<int>((ma & a1) | (r & b1) | (t & sa1) | (wb & sb1));
    d2 = static_cast<int>((ma & a2) | (r & b2) | (t & sa2) | (wb & sb2));
}

// Digits 1 and 2 of eight numbers in signed base 16 (w1, w2 one digit a nibble), taken together as d1 + 16 d2 for sums
// in -16 .. 16: the low four bits of the magnitudes and, in bits 3 and 2 of each nibble, sign and sixteens bit.
struct Fp6Parts { uint32_t low, top; };
__device__ __forceinline__ Fp6Parts fp6_upper8(uint32_t w1, uint32_t w2) {
    constexpr uint32_t ones = 0x11111111u;
    const uint32_t n2 = w2 & ones;                                         // d2 is 1 or -1
    const uint32_t sign = ((w1 >> 3) & ones & ~n2) | ((w2 >> 3) & ones);   // of d2, or of d1 where d2 is 0
    uint32_t any = w1 | (w1 >> 1);
    any = (any | (any >> 2)) & ones;                                       // d1 is not 0
    const uint32_t neg = sign & any;
    return {(w1 ^ ((neg << 4) - neg)) + neg, (sign << 3) | ((n2 & ~any) << 2)};
}

// Two such eights -> three dwords of signed fields of magnitude 0..16 (16 is E2M3's 10000b, again the number itself).
__device__ __forceinline__ void fp6_upper16(uint32_t wa1, uint32_t wa2, uint32_t wb1, uint32_t wb2, int &d0, int &d1, int &d2) {
    const Fp6Parts a = fp6_upper8(wa1, wa2), b = fp6_upper8(wb1, wb2);
    const uint32_t r = __builtin_amdgcn_alignbit(b.low, b.low, 2);
    const uint32_t t = __builtin_amdgcn_alignbit(a.top, a.top, 30);   // top bits of a's nibbles, two places up
    constexpr uint32_t a0 = fp6_bits(15, 0, 12, 24), b0 = fp6_bits(15, 6, 18) | (3u << 30);
    constexpr uint32_t a1 = fp6_bits(15, 4, 16, 28), b1 = fp6_bits(15, 10, 22) | 3u;
    constexpr uint32_t a2 = fp6_bits(15, 8, 20), b2 = fp6_bits(15, 2, 14, 26);
    constexpr uint32_t ta0 = fp6_bits(3, 4, 16, 28), tb0 = fp6_bits(3, 10, 22);
    constexpr uint32_t ta1 = fp6_bits(3, 8, 20), tb1 = fp6_bits(3, 2, 14, 26);
    constexpr uint32_t ta2 = fp6_bits(3, 0, 12, 24), tb2 = fp6_bits(3, 6, 18, 30);
    d0 = static_cast<int>((a.low & a0) | (r & b0) | (t & ta0) | (b.top & tb0));
    d1 = static_cast<int>((a.low & a1) | (r & b1) | (t & ta1) | (b.top & tb1));
    d2 = static_cast<int>((a.low & a2) | (r & b2) | (t & ta2) | (b.top & tb2));
}

// Sum of the 8 codes of a packed dword, added to acc.
__device__ __forceinline__ int sum_codes8(uint32_t w, int acc) {
    return __builtin_amdgcn_sdot8(static_cast<int>(w), 0x11111111, acc, false);
}

}  // namespace
