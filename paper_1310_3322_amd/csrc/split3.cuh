// FP32 products on the bf16 matrix cores (gfx950) by exact three-way splits.
//
// An FP32 value is the sum of three bf16 values: hi = bf16(x), mid = bf16(x - hi),
// lo = x - hi - mid (8 + 8 + 8 significand bits; every difference is exact).  A product
// of two split values needs six of the nine partial products; the three left out
// (mid lo, lo mid, lo lo) are below 2^-26 of it.  The partial products are exact in
// the matrix core, which adds them in FP32.  The bf16 instructions reach 2.4 PFLOP/s
// where the FP32 ones reach 157 TFLOP/s, so the six take 0.4 of their time (0.55 once
// the power they draw lowers the clock), and they leave the vector ALUs free for other
// waves, which the FP32 instructions do not.
//
// Error of a step of the forward against 64 bits (rms of the logarithm of its sum, 8 banks of
// each kind), with the FP32 instructions in brackets, at 64 and 256 states: Dirichlet rows of
// concentration 1 5.1e-9 (6.9e-9) and 5.9e-9 (8.7e-9), of 0.5 6.0e-9 (7.2e-9) and 6.3e-9 (9.5e-9),
// of 0.2 1.8e-8 (1.2e-8) and 1.7e-8 (4.8e-8; equal near 96 states).  Beside one large product the
// matrix core drops low bits of the small ones, here more of them than in FP32: rows with an entry of
// 0.9 3.9e-8 (1.0e-8) and 5.6e-8 (2.1e-8), all below one FP32 rounding per step.  A sum of its own for
// each 32 products does not help (3.8e-8 and 5.4e-8) and costs 2 to 27 % of the time.  The small
// terms are added first: products of 32 states are then off by 3.9e-8, with hi hi first by 1.3e-7.
//
// Range: bf16 has FP32's exponents, but the matrix core and the dot products below flush
// denormals, so the pieces of a value below 2^-110 lose bits that FP32 keeps.  Both factors are
// therefore split SPLIT_SHIFT binades above their place (callers scale by the power of two and
// take it out of the result, both exact): the last bit of any FP32 number, denormals
// included, is 2^-149 or more, and 2^-117 or more there, so every piece is a normal number.
// Split at their place, log-likelihoods were off by 3e-5 (64 states) and 1.2e-4 (256) with every
// third emission near 1e-37, where this and FP32 give 5e-8, and -inf near 1e-38; the shift costs no
// instruction per step (256 states, 16384 sequences: 20.1 ms either way, runs differ by 1 %).
// Values from 2^(127 - SPLIT_SHIFT) up overflow; probabilities end at 1.
#pragma once

#include "common.cuh"

namespace hmm {

constexpr int SPLIT_SHIFT = 32;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

// The pairs (-1, 0) and (0, -1), kept in scalar registers: subtracting one half of a
// packed pair is then a single two-term dot product.  (Given as literals, the
// compiler encodes them as inline constants that the instruction reads differently.)
struct SplitConst {
    bf16x2 lo, hi;
    __device__ __forceinline__ SplitConst() {
        uint32_t a = 0x0000bf80u, b = 0xbf800000u;
        asm("" : "+s"(a), "+s"(b));
        lo = __builtin_bit_cast(bf16x2, a);
        hi = __builtin_bit_cast(bf16x2, b);
    }
};

// Pieces of a and b as packed pairs (3.5 vector instructions per value).
__device__ __forceinline__ void split_pair(const SplitConst &c, float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
    const bf16x2 hp = __builtin_convertvector(floatx2{a, b}, bf16x2);
    const float ra = __builtin_amdgcn_fdot2_f32_bf16(hp, c.lo, a, false);
    const float rb = __builtin_amdgcn_fdot2_f32_bf16(hp, c.hi, b, false);
    const bf16x2 mp = __builtin_convertvector(floatx2{ra, rb}, bf16x2);
    const float sa = __builtin_amdgcn_fdot2_f32_bf16(mp, c.lo, ra, false);
    const float sb = __builtin_amdgcn_fdot2_f32_bf16(mp, c.hi, rb, false);
    const bf16x2 lp = __builtin_convertvector(floatx2{sa, sb}, bf16x2);
    h = __builtin_bit_cast(uint32_t, hp);
    m = __builtin_bit_cast(uint32_t, mp);
    l = __builtin_bit_cast(uint32_t, lp);
}

// Eight values as matrix-core operands, one per piece.
struct Split8 {
    bf16x8 p[3];
};

__device__ __forceinline__ Split8 split8(const SplitConst &c, const float (&x)[8]) {
    uintx4 q[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t h, m, l;
        split_pair(c, x[2 * i], x[2 * i + 1], h, m, l);
        q[0][i] = h;
        q[1][i] = m;
        q[2][i] = l;
    }
    Split8 r;
#pragma unroll
    for (int k = 0; k < 3; ++k) r.p[k] = __builtin_bit_cast(bf16x8, q[k]);
    return r;
}

// The six partial products (piece of A, piece of x), smallest first.
constexpr int SPLIT_TERMS = 6;
constexpr int SPLIT_A[SPLIT_TERMS] = {2, 0, 1, 1, 0, 0};
constexpr int SPLIT_X[SPLIT_TERMS] = {0, 2, 1, 0, 1, 0};

}  // namespace hmm
