// Pieces for 16-row tiles: the 16x16x32 product, and the solve of a 16-row
// triangular block in the registers of 16 lanes.
#pragma once

#include "device.h"

namespace treewy {

// D(16x16) += A(16x32) B(32x16) on the matrix cores, bf16 in, fp32 accumulate.
// Lane l supplies row l%16 of A and column l%16 of B, each with the eight
// contraction indices of group l/16; lane l receives column l%16 of D at rows
// 4*(l/16) + r in accumulator element r.
__device__ __forceinline__ f32x4 mma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Four floats -> bf16 hi + lo (see split8).
__device__ __forceinline__ void split4(f32x4 x, uint2 &hi, uint2 &lo) {
    hi.x = pack_bf2(x[0], x[1]);
    hi.y = pack_bf2(x[2], x[3]);
    lo.x = pack_bf2(x[0] - __builtin_bit_cast(float, hi.x << 16), x[1] - __builtin_bit_cast(float, hi.x & 0xffff0000u));
    lo.y = pack_bf2(x[2] - __builtin_bit_cast(float, hi.y << 16), x[3] - __builtin_bit_cast(float, hi.y & 0xffff0000u));
}

// Four floats -> bf16 hi + mid + lo, exactly (24 bits; past the type's range of exponents lo may round).
__device__ __forceinline__ void split4(f32x4 x, uint2 &hi, uint2 &mid, uint2 &lo) {
    auto rest = [](f32x4 &y, uint2 h) {
        y[0] -= __builtin_bit_cast(float, h.x << 16);
        y[1] -= __builtin_bit_cast(float, h.x & 0xffff0000u);
        y[2] -= __builtin_bit_cast(float, h.y << 16);
        y[3] -= __builtin_bit_cast(float, h.y & 0xffff0000u);
    };
    hi = make_uint2(pack_bf2(x[0], x[1]), pack_bf2(x[2], x[3]));
    rest(x, hi);
    mid = make_uint2(pack_bf2(x[0], x[1]), pack_bf2(x[2], x[3]));
    rest(x, mid);
    lo = make_uint2(pack_bf2(x[0], x[1]), pack_bf2(x[2], x[3]));
}

// Two values of four contraction entries each, in the two halves of a lane group's eight slots.
__device__ __forceinline__ bf16x8 both8(uint2 x, uint2 y) { return __builtin_bit_cast(bf16x8, make_uint4(x.x, x.y, y.x, y.y)); }

// Four contraction entries of a lane group as the low half of its eight slots, the others empty.
__device__ __forceinline__ bf16x8 low8(uint2 x) { return __builtin_bit_cast(bf16x8, make_uint4(x.x, x.y, 0u, 0u)); }

// Operand of a transposed LDS read: within each 16 lanes, lane 4 j + y points at
// four 16-bit entries of row j and lane i receives column i of the 4 x 16 block.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef s16x4 __attribute__((address_space(3))) lds_s16x4;

// A bijection of t % 16 onto the 16 granules of a row, which sends four
// consecutive rows to four different groups of four granules.  The LDS serves
// a 16-byte read in sets of sixteen lanes, 0-3, 12-15, 20-27 and 4-11, 16-19,
// 28-31 and the same past 32 (found by which pairs of lanes collide), so rows
// 0-3 and 12-15 of lane group g come with rows 4-11 of group g ^ 1: the
// granules of the former are closed under ^ 1, so those of the latter, one
// group on, are the other eight.  (With t / 4 as it is in the low bits each
// such read took 8.2 cycles instead of 5.8.)
__device__ __forceinline__ int swz(int t) {
    return ((t & 3) << 2) | (((t >> 2) ^ (t >> 3)) & 1) << 1 | ((t >> 2) & 1);
}

// LDS written and read again by the same wave: the hardware keeps a wave's
// LDS accesses in order; this keeps the compiler from reordering accesses of
// different types.
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// r[j] += x * (b[j] of lane I of each row of 16 lanes), j = 0 .. NJ - 1: the row
// broadcast rides on the multiply-add (the compiler leaves it a move of its
// own).  (A DPP source must have been written two wait states before: s_nop.)
template <int I, int NJ> __device__ __forceinline__ void fmac_bcast(float *r, const float *b, float x) {
    static_assert(NJ == 4 || NJ == 8, "groups of four or eight");
#define TW_F(n, m) "v_fmac_f32_dpp %" #n ", %" #m ", %[x] row_newbcast:%[i] row_mask:0xf bank_mask:0xf\n\t"
    if constexpr (NJ == 4)
        asm("s_nop 1\n\t" TW_F(0, 4) TW_F(1, 5) TW_F(2, 6) TW_F(3, 7)
            : "+&v"(r[0]), "+&v"(r[1]), "+&v"(r[2]), "+&v"(r[3])
            : "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), [x] "v"(x), [i] "n"(I));
    else
        asm("s_nop 1\n\t" TW_F(0, 8) TW_F(1, 9) TW_F(2, 10) TW_F(3, 11) TW_F(4, 12) TW_F(5, 13) TW_F(6, 14) TW_F(7, 15)
            : "+&v"(r[0]), "+&v"(r[1]), "+&v"(r[2]), "+&v"(r[3]), "+&v"(r[4]), "+&v"(r[5]), "+&v"(r[6]), "+&v"(r[7])
            : "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(b[4]), "v"(b[5]), "v"(b[6]), "v"(b[7]), [x] "v"(x),
              [i] "n"(I));
#undef TW_F
}

// Column I of the sweep that builds row t of a 16-row diagonal block of
// T = (I + B)^{-1}, then the next column down: with the columns past I done,
// T[t, I] = -(B[t, I] + sum over i > I of T[t, i] B[i, I]), held in r[I].  Row I of B comes from lane I's registers,
// so the sweep reads no LDS.  The multiply-adds go in groups of four or
// eight columns: those at or past I add x times a zero of B.
template <int I> __device__ __forceinline__ void sweep16(float (&r)[16], const float (&b)[16], int t) {
    const float x = I < t ? -r[I] : 0.f;                 // T[t, I] (zero on and above the diagonal)
    r[I] = x;
    if constexpr (I > 0) {
        fmac_bcast<I, (I > 4 ? 8 : 4)>(r, b, x);
        if constexpr (I > 8) fmac_bcast<I, (I > 12 ? 8 : 4)>(r + 8, b + 8, x);
        sweep16<I - 1>(r, b, t);
    }
}

}  // namespace treewy
