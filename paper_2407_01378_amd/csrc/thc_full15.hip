// First pass of the full rotation over chunks of 2^15 coordinates: stages 0..14, one workgroup of 1024 threads
// (16 waves) per chunk, 32 coordinates per thread in registers, results in fp32.
//
// What it is for: the passes behind it move a row of the array per 2^s0 coordinates, and with 11 stages left
// behind chunks of 2^14 those rows are 64-byte pieces, which memory serves at 0.7 of the rate of whole
// lines.  One stage more in front makes 10 stages (whole lines) of the 11: see full_first_log2.
//
// Bound by memory.  A wave's 2^11 coordinates are loaded in whole 1 KB runs, a lane holding 2^RB consecutive
// coordinates of several runs (16 bytes each), so nothing is staged: stages 0..RB-1 between registers, RB..RB+3
// between lanes (thc_lanes.h), the rest up to 10 after swaps of register bit 4 with lane bits 4 and 5.
// One exchange through LDS then brings i11..i14 into the registers, half of them at a time so that it takes
// 64 KB: two workgroups and 32 waves per CU, whose loads and stores overlap the other's arithmetic.
// Measured, 25.6 M fp32 coordinates in 2^25: 45 us (39 us over chunks of 2^14: 780 chunks are 1.5 rounds), the range
// behind it 21.5 us instead of 32.5, the quantizing pass 36 instead of 42.5, the inverse 35 + 49 instead of 29 + 66.
#include "thc_core14.h"
#include "thc_internal.h"

#pragma clang fp contract(off)

namespace thc {
namespace {

using k14::butterflies;
using k14::kRegs;

constexpr uint32_t kLog2 = 15;
constexpr int kThreads = 1024;

// What a chunk is made of: a gradient with the sign diagonal, values as they stand, or stored sums.
enum class From : int { F32 = 0, BF16 = 1, Plain = 2, U8 = 3, U16 = 4 };
// Consecutive coordinates of a lane (log2): 16 bytes of input, 16 sums.
constexpr uint32_t run_log2(From src) { return src == From::BF16 ? 3u : src == From::U8 || src == From::U16 ? 4u : 2u; }

// LDS place of a 16-byte unit (i0, i1) by c = i2..i9, inside the 256 units of i10..i14 fixed: eight lanes that
// store together differ in three consecutive bits of i2..i6 and take all values of the low three bits; the
// lanes of a half wave that load words differ in i0..i4 and take all 32 banks.
__device__ __forceinline__ uint32_t unit15(uint32_t c) {
    return ((c >> 2) & 1u) | (((c ^ (c >> 3)) & 3u) << 1) | (c & 0xF8u);
}

template <From SRC>
__global__ __launch_bounds__(kThreads, 8) void first_pass15_kernel(const ChunkArgs a) {
    constexpr uint32_t RB = run_log2(SRC);
    constexpr bool kSigned = SRC == From::F32 || SRC == From::BF16;
    constexpr int kRuns = 1 << (5 - (int)RB);        // of a thread
    __shared__ float4 xb[4096];
    __shared__ alignas(16) uint32_t sign[kSigned ? 1u << (kLog2 - 5u) : 4u];
    const uint32_t t = threadIdx.x, lane = t & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));   // i11..i14
    const uint32_t b = lay14::block_of_lane(lane);   // the lane's run: i_RB .. i_(RB+5)
    const uint64_t g0 = (uint64_t)blockIdx.x << kLog2;
    float v[kRegs];

    if constexpr (kSigned) {
        constexpr uint32_t kElem = SRC == From::BF16 ? 2u : 4u;
        const uint64_t rest = a.n - g0;
        const uint32_t left = rest < (1ull << kLog2) ? (uint32_t)rest : 1u << kLog2;
        const uint8_t* in = static_cast<const uint8_t*>(a.in) + g0 * kElem;
        // (reads past the range return zero; the check is made for each dword, so the last coordinate of an
        // odd count of bf16 is fetched by itself.  The whole place of a unit is in the vector offset: the
        // scalar offset is not part of the documented range check)
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t*>(in), 0, (int)(SRC == From::BF16 ? (left & ~1u) * 2u : left * 4u), 0x00020000);
        u32x4_vec raw[kRuns];
#pragma unroll
        for (int j = 0; j < kRuns; ++j)
            raw[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, wave * (2048u * kElem) + b * 16u + (uint32_t)j * 1024u, 0, 0);
        if (SRC == From::BF16 && (left & 1u)) {
            const uint32_t last = left - 1u;   // coordinate 2 d of unit j of one thread
            const uint32_t word = reinterpret_cast<const uint16_t*>(in)[last];
#pragma unroll
            for (int j = 0; j < kRuns; ++j)
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    if (last == wave * 2048u + (uint32_t)j * 512u + 8u * b + 2u * d) raw[j][d] = word;
        }
        if (t < 256u) {
            u32x4 s = sign_block((g0 >> 7) + t, a.key0, a.key1);
            if (SRC == From::BF16) {
#pragma unroll
                for (int i = 0; i < 4; ++i) s.w[i] = k14::unshuffle_bits(s.w[i]);
            }
            *reinterpret_cast<u32x4*>(&sign[4 * t]) = s;
        }
        if (a.zero_word && blockIdx.x == 0 && t == 0) *a.zero_word = 0u;   // raised by a later pass
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kRuns; ++j) {
            const uint32_t word = sign[wave * 64u + (uint32_t)j * (SRC == From::BF16 ? 16u : 8u) + (b >> (5u - RB))];
            if constexpr (SRC == From::BF16) {   // (even bits in the low half, odd bits in the high half)
                const uint32_t s = word << (12u - 4u * (b & 3u));
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const uint32_t x = xor_masked(raw[j][d], s << (3 - d), 0x80008000u);
                    v[8 * j + 2 * d] = __uint_as_float(x << 16);
                    v[8 * j + 2 * d + 1] = __uint_as_float(x & 0xFFFF0000u);
                }
            } else {
                const uint32_t s = word >> (4u * (b & 7u));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * j + e] = __uint_as_float(xor_masked(raw[j][e], s << (31 - e), 0x80000000u));
            }
        }
    } else if constexpr (SRC == From::Plain) {
        const float4* in = reinterpret_cast<const float4*>(static_cast<const float*>(a.in) + g0) + wave * 512u + b;
#pragma unroll
        for (int j = 0; j < kRuns; ++j) {
            const float4 f = in[j * 64];
            v[4 * j] = f.x;
            v[4 * j + 1] = f.y;
            v[4 * j + 2] = f.z;
            v[4 * j + 3] = f.w;
        }
    } else {
        constexpr uint32_t kSize = SRC == From::U8 ? 1u : 2u;
        const uint4* in = reinterpret_cast<const uint4*>(static_cast<const uint8_t*>(a.in) + g0 * kSize) +
                          (wave * 128u + b) * kSize;
        const float s = a.scale_in[0];   // yhat = S q - s
        const float step = (s + s) / (float)a.levels;
        const float q = step / (float)a.W;
#pragma unroll
        for (int j = 0; j < kRuns; ++j)
#pragma unroll
            for (uint32_t k = 0; k < kSize; ++k) {
                const uint4 x = in[(uint32_t)j * 64u * kSize + k];
                const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                for (uint32_t e = 0; e < 16u / kSize; ++e) {
                    constexpr uint32_t per = 4u / kSize;
                    const uint32_t S = (w[e / per] >> (8u * kSize * (e % per))) & (kSize == 1u ? 0xFFu : 0xFFFFu);
                    v[16 * j + 16u / kSize * k + e] = (float)S * q - s;
                }
            }
    }

    // registers: i0 .. i_(RB-1), i_(RB+6) .. i10 (bit 4)
    butterflies<0, (int)RB>(v);
    lanes::lane_stage<0>(v, (b & 1u) ? -1.0f : 1.0f);   // i_RB .. i_(RB+3)
    lanes::lane_stage<1>(v, (b & 2u) ? -1.0f : 1.0f);
    lanes::lane_stage<2>(v, (b & 4u) ? -1.0f : 1.0f);
    lanes::lane_stage<3>(v, (b & 8u) ? -1.0f : 1.0f);
    lanes::swap_top_register_bit<16>(v);                // i10 <-> i_(RB+4)
    butterflies<4, 5>(v);
    lanes::swap_top_register_bit<32>(v);                // i_(RB+4) <-> i_(RB+5)
    butterflies<4, 5>(v);
    butterflies<(int)RB, 4>(v);                         // i_(RB+6) .. i9
    lanes::swap_top_register_bit<16>(v);                // i_(RB+5) <-> i10
    butterflies<4, 5>(v);
    // now lane bit 4 = i_(RB+5), lane bit 5 = i_(RB+4)

    const uint32_t lane_bits = ((b & 15u) << RB) | ((lane >> 5) << (RB + 4u)) | (((lane >> 4) & 1u) << (RB + 5u));
    const float* words = reinterpret_cast<const float*>(xb);
    const uint32_t from = 4u * unit15((t >> 2) & 0xFFu) | (t & 3u);   // i0..i9 = t
#pragma unroll
    for (int half = 0; half < 2; ++half) {   // i10
        if (half) __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            // register bits 2 and 3: i2, i3 or, from RB on, i_(RB+6) ..
            const uint32_t i = lane_bits | ((uint32_t)(q & 1) << (RB > 2u ? 2u : RB + 6u)) |
                               ((uint32_t)(q >> 1) << (RB > 3u ? 3u : RB == 3u ? RB + 6u : RB + 7u));
            xb[unit15(i >> 2) | (wave << 8)] =
                make_float4(v[16 * half + 4 * q], v[16 * half + 4 * q + 1], v[16 * half + 4 * q + 2], v[16 * half + 4 * q + 3]);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) v[16 * half + r] = words[from + 1024u * r];   // r = i11..i14
    }
    butterflies<0, 3>(v);
    // The values are negated where i_RB .. i_(RB+3) have odd parity, which are bits of t.  The last stage undoes
    // it in its multiply-adds by +-1 (one rounding, of the same sum: a difference of equal values is +0 as the stage gives
    // it; only the sign of a sum of two zeros can be another).
    const float sgn = k14::odd_parity4(t >> RB) ? -1.0f : 1.0f;
#pragma unroll
    for (int r = 0; r < kRegs; ++r)
        if ((r & 8) == 0) {
            const float lo = v[r], hi = v[r + 8] * sgn;
            v[r] = __builtin_fmaf(lo, sgn, hi);
            v[r + 8] = __builtin_fmaf(lo, sgn, -hi);
        }
    // (through a descriptor: the 32 places are the thread's plus a scalar)
    const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(static_cast<float*>(a.out) + g0, 0, 4 << kLog2, 0x00020000);
#pragma unroll
    for (int r = 0; r < kRegs; ++r)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[r]), out, t * 4u,
                                              (r >> 4) * 4096 + (r & 15) * 8192, 0);
}

}  // namespace

// a: as for the chunk-2^14 kernels, with chunk_log2 = 15 and one scale for all chunks.
hipError_t launch_full_first15(Mode mode, const ChunkArgs& a, hipStream_t stream) {
    const dim3 grid((uint32_t)(a.padded >> kLog2)), block(kThreads);
    if (grid.x == 0) return hipSuccess;
    if (mode == Mode::Forward && a.in_bf16)
        hipLaunchKernelGGL(first_pass15_kernel<From::BF16>, grid, block, 0, stream, a);
    else if (mode == Mode::Forward)
        hipLaunchKernelGGL(first_pass15_kernel<From::F32>, grid, block, 0, stream, a);
    else if (mode == Mode::Plain)
        hipLaunchKernelGGL(first_pass15_kernel<From::Plain>, grid, block, 0, stream, a);
    else if (mode == Mode::PlainDecode && a.sum_bytes == 1)
        hipLaunchKernelGGL(first_pass15_kernel<From::U8>, grid, block, 0, stream, a);
    else if (mode == Mode::PlainDecode)
        hipLaunchKernelGGL(first_pass15_kernel<From::U16>, grid, block, 0, stream, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace thc
