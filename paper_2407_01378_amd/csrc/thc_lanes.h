// Butterfly stages between the lanes of a wave, without LDS.
//
// A lane of a wave that holds coordinates i0..i4 in its registers owns block B = i5..i10 of the
// wave's 2048 coordinates.  For i5..i8 the partner's value arrives through a data-parallel
// primitive inside the multiply-add itself: v <- v + s * partner with s = +1 in the lower
// lane and -1 in the upper one, one vector operation per value and stage, the same as a stage
// between registers.  One rounding, of the exact sum: the lower lane gets lo + hi, the upper
// one hi - lo, the exact negative of the stage's lo - hi.  Every later stage combines values
// of lanes with the same i5..i8, so the negation (by the parity of the lane's upper bits among
// the stages done) is carried to the end and undone there, where the consumer multiplies by a
// constant anyway.
//
// The primitives exchange lanes l and l ^ 1, l ^ 2, l ^ 7 (mirror of 8) and l ^ 15 (mirror of
// 16), so lane l owns the block whose bits are
//     i5 = l0 ^ l2,  i6 = l1 ^ l2,  i7 = l2 ^ l3,  i8 = l3,  i9 = l4,  i10 = l5:
// each of the four exchanges then flips exactly one of i5..i8.
// i9 and i10 come into the registers by the swap instructions of gfx950 (row 2k+1 of one
// register against row 2k of another, and the halves of a wave alike): half an operation per
// value for a stage.
#pragma once

#include "thc_device.h"
#include "thc_layout14.h"

#pragma clang fp contract(off)

namespace thc {
namespace lanes {

constexpr int kRegs = 32;

using lay14::block_of_lane;

// The inline assembly hides its register accesses from the compiler's hazard recognizer: a
// lane exchange may read a register two wait states after it was written at the earliest, so
// each block of eight waits in front (what it reads) and behind (what it wrote).
#define THC_LANE_FMAC8(CTRL, R)                                                                     \
    asm("s_nop 1\n\t"                                                                               \
        "v_fmac_f32_dpp %0, %0, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                         \
        "v_fmac_f32_dpp %1, %1, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                         \
        "v_fmac_f32_dpp %2, %2, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                         \
        "v_fmac_f32_dpp %3, %3, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                         \
        "v_fmac_f32_dpp %4, %4, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                         \
        "v_fmac_f32_dpp %5, %5, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                         \
        "v_fmac_f32_dpp %6, %6, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                         \
        "v_fmac_f32_dpp %7, %7, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                         \
        "s_nop 1"                                                                                   \
        : "+v"(v[R]), "+v"(v[R + 1]), "+v"(v[R + 2]), "+v"(v[R + 3]), "+v"(v[R + 4]), "+v"(v[R + 5]), \
          "+v"(v[R + 6]), "+v"(v[R + 7])                                                            \
        : "v"(s))

// Stage 5 + K (K = 0..3) on the 32 registers; s = -1 in the lanes whose bit i(5 + K) is set, else
// +1.  All 64 lanes must be active.
template <int K>
__device__ __forceinline__ void lane_stage(float (&v)[kRegs], float s) {
    if constexpr (K == 0) {
        THC_LANE_FMAC8("quad_perm:[1,0,3,2]", 0);
        THC_LANE_FMAC8("quad_perm:[1,0,3,2]", 8);
        THC_LANE_FMAC8("quad_perm:[1,0,3,2]", 16);
        THC_LANE_FMAC8("quad_perm:[1,0,3,2]", 24);
    } else if constexpr (K == 1) {
        THC_LANE_FMAC8("quad_perm:[2,3,0,1]", 0);
        THC_LANE_FMAC8("quad_perm:[2,3,0,1]", 8);
        THC_LANE_FMAC8("quad_perm:[2,3,0,1]", 16);
        THC_LANE_FMAC8("quad_perm:[2,3,0,1]", 24);
    } else if constexpr (K == 2) {
        THC_LANE_FMAC8("row_half_mirror", 0);
        THC_LANE_FMAC8("row_half_mirror", 8);
        THC_LANE_FMAC8("row_half_mirror", 16);
        THC_LANE_FMAC8("row_half_mirror", 24);
    } else {
        THC_LANE_FMAC8("row_mirror", 0);
        THC_LANE_FMAC8("row_mirror", 8);
        THC_LANE_FMAC8("row_mirror", 16);
        THC_LANE_FMAC8("row_mirror", 24);
    }
}
#undef THC_LANE_FMAC8

// Register bit 4 <-> lane bit 3 (SWAP 8), 4 (SWAP 16) or 5 (SWAP 32).
template <int SWAP>
__device__ __forceinline__ void swap_top_register_bit(float (&v)[kRegs]) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const uint32_t a = __float_as_uint(v[r]), b = __float_as_uint(v[r + 16]);
        if constexpr (SWAP == 8) {   // rotation by 8 within a row of 16 = lane ^ 8, written in half of the lanes
            v[r] = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp((int)a, (int)b, 0x128, 0xF, 0xC, false));
            v[r + 16] = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp((int)b, (int)a, 0x128, 0xF, 0x3, false));
        } else if constexpr (SWAP == 16) {
            const auto q = __builtin_amdgcn_permlane16_swap(a, b, false, false);
            v[r] = __uint_as_float(q[0]);
            v[r + 16] = __uint_as_float(q[1]);
        } else {
            const auto q = __builtin_amdgcn_permlane32_swap(a, b, false, false);
            v[r] = __uint_as_float(q[0]);
            v[r + 16] = __uint_as_float(q[1]);
        }
    }
}

// Larger of x and the partner lane's x, as unsigned words; STEP = 1, 2, 7, 15 (lane exchanged
// with lane ^ STEP), 16 or 32.
template <int STEP>
__device__ __forceinline__ uint32_t umax_step(uint32_t x) {
    if constexpr (STEP >= 16) {
        uint32_t a, b;
        if constexpr (STEP == 16) {
            const auto q = __builtin_amdgcn_permlane16_swap(x, x, false, false);
            a = q[0];
            b = q[1];
        } else {
            const auto q = __builtin_amdgcn_permlane32_swap(x, x, false, false);
            a = q[0];
            b = q[1];
        }
        return a > b ? a : b;
    } else {
        constexpr int ctrl = STEP == 1 ? 0xB1 : STEP == 2 ? 0x4E : STEP == 7 ? 0x141 : 0x140;
        const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xF, 0xF, false);
        return y > x ? y : x;
    }
}

}  // namespace lanes
}  // namespace thc
