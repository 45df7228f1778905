// Tuned kernels for chunk_log2 = 14 (the chunk size of every large workload): one
// workgroup of 512 threads per chunk, the chunk lives in registers (32 coordinates per
// thread) and is re-shuffled through LDS between groups of butterfly stages, see
// thc_core14.h.  Used when every pointer is 16-byte aligned; the generic kernels cover
// everything else with identical results.
#include "thc_core14.h"
#include "thc_internal.h"
#include "thc_resident.h"

#pragma clang fp contract(off)

namespace thc {
namespace k14 {
namespace {

// One chunk per workgroup, gradient of ONE worker: rotation / range / encode.
//   BF16   input type;  MODE  Forward | Absmax | MinMax | Encode;  BITS payload width (Encode)
// A call of one worker often has fewer chunks than the chip holds at once (512): the time is then
// one chunk's chain of loads, exchanges and barriers, not a throughput.  Absmax and Encode therefore
// run stages 5..8 between lanes (rotate_lanes_to_l3): one exchange less, three barriers instead
// of six up to the range.  Forward keeps the LDS maps (long calls
// of it are bound by memory: 6 TB/s); MinMax keeps them too, the lanes have not been timed there.
// Measured at 7 M bf16 (433 chunks): range 8.0 -> 6.5 us, 8-bit encode 11.1 -> 9.4; per-call round of
// eight workers 177 -> 153 us.  Encode also draws its rounding bytes (a tenth of its operations) and reads the given range
// while the input is on its way: 8 bits, 433 chunks 8.8 -> 8.5 us, 512 9.3 -> 8.8, 2048 29.9 -> 26.8, fp32 2048 38.8 -> 35.5.
//   PRIO  the rotation ahead of the other workgroup's quantizer, for launches of up to two workgroups per CU: 433 chunks
//         8.4 -> 7.9, 512 8.7 -> 8.25.  In longer ones it would hold up the loads of the workgroups that follow: fp32 1024 chunks
//         20.1 us, with it 20.8; 2048 33.8 and 35.4.  (The range has nothing behind the rotation to put back.)
template <bool BF16, Mode MODE, int BITS, bool PRIO = false>
__global__ __launch_bounds__(kThreads) void per_worker_kernel(const ChunkArgs a) {
    __shared__ Shared sh;
    constexpr int kUnits = BF16 ? 4 : 8;
    constexpr int kElem = BF16 ? 2 : 4;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint64_t p = blockIdx.x;
    const uint64_t g0 = p << kChunkLog2;
    const uint64_t left = a.n - g0;
    const uint32_t valid = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;

    // Encode: the given range is read, and the rounding stream drawn, while the input is on its way
    float lo = 0.0f, hi = 0.0f;
    if constexpr (MODE == Mode::Encode) {
        if (a.range_in) {
            lo = a.range_in[2 * p];
            hi = a.range_in[2 * p + 1];
        } else if (a.scale_in) {
            hi = a.scale_in[p];
        }
    }
    Drawn drawn;
    constexpr bool kLanes = MODE == Mode::Absmax || MODE == Mode::Encode;
    const uint32_t block = lay14::block_of_lane(lane), tp = kLanes ? (t & ~63u) | block : t;
    constexpr bool kDirect = kLanes && BF16;   // every thread loads its own 64 bytes
    Raw<kUnits> raw;
    load_raw<kUnits, kElem, kDirect>(raw, static_cast<const uint8_t*>(a.in) + g0 * kElem, valid, kDirect ? tp : t);
    fill_sign_table<!BF16, BF16>(sh.sign[0], g0, a.key0, a.key1, t);
    if constexpr (MODE == Mode::Encode) drawn.draw(g0 + 32u * tp, a.worker, a.key0, a.key1);
    if (!kDirect) raw_to_lds<kUnits>(sh, raw, t);
    __syncthreads();
    float v[kRegs];
    if (kDirect) units_to_l1<kUnits, true>(sh.sign[0], raw.u, v, tp);
    else lds_to_l1<kUnits, true>(sh, sh.sign[0], v, tp);
    // (a wave reads the units of its own 8 KB of the buffer, and the first exchange stores there: no barrier)
    if constexpr (kLanes) rotate_lanes_to_l3<PRIO>(sh, v, lane, block, wave);
    else rotate_l1_to_l3<false>(sh, v, lane, wave);
    const float sgn = odd_parity4(block) ? -1.0f : 1.0f;   // Encode: the thread's values are negated

    if constexpr (MODE == Mode::Forward) {
        // (the first pass of a longer rotation also zeroes the word its last pass raises)
        if (a.zero_word && p == 0 && t == 0) *a.zero_word = 0u;
        l3_to_l4d<false>(sh, v, lane, wave);
        float* y = static_cast<float*>(a.out) + g0;
#pragma unroll
        for (int h = 0; h < 8; ++h)
            *reinterpret_cast<float4*>(y + h * 2048 + t * 4) =
                make_float4(v[4 * h] * a.inv_sqrt_c, v[4 * h + 1] * a.inv_sqrt_c, v[4 * h + 2] * a.inv_sqrt_c,
                            v[4 * h + 3] * a.inv_sqrt_c);   // 2^-7, or 1 as the first pass of a longer rotation
    } else if constexpr (MODE == Mode::Absmax) {
        const float m = chunk_absmax(sh, v, lane, wave) * kInvSqrtC;
        if (t == 0) static_cast<float*>(a.out)[p] = m;
    } else if constexpr (MODE == Mode::MinMax) {
        const MinMax r = chunk_minmax(sh, v, lane, wave);
        if (t == 0) {
            static_cast<float*>(a.out)[2 * p] = rotated_end(r.lo);
            static_cast<float*>(a.out)[2 * p + 1] = rotated_end(r.hi);
        }
    } else if (a.range_in) {   // Encode on the min/max grid
        l3_to_l4e_lanes<PRIO>(sh, v, lane, block, wave);
        quantize_store_range<BITS>(v, lo, hi, a.levels, g0, a.worker, a.key0, a.key1,
                                   static_cast<uint8_t*>(a.out), tp, kInvSqrtC * sgn, &drawn);
    } else {
        const float s = a.scale_in ? hi : chunk_absmax(sh, v, lane, wave) * kInvSqrtC;
        if (a.scale_out && t == 0) a.scale_out[p] = s;
        l3_to_l4e_lanes<PRIO>(sh, v, lane, block, wave);
        quantize_store<BITS, true, true>(v, s, a.levels, g0, a.worker, a.key0, a.key1, static_cast<uint8_t*>(a.out),
                                         tp, sgn, &drawn);
    }
}

// The "no rotation" arm of the min/max variant: y is the zero-padded gradient itself, so a
// chunk needs no exchange at all.  Thread t loads its 32 consecutive coordinates, and
// either the workgroup reduces them to (min, max) or the thread quantizes them onto the
// given range and stores its 4 * BITS payload bytes.
template <bool BF16, Mode MODE, int BITS>
__global__ __launch_bounds__(kThreads) void unrotated_kernel(const ChunkArgs a) {
    __shared__ Shared sh;
    constexpr int kUnits = BF16 ? 4 : 8;
    constexpr int kElem = BF16 ? 2 : 4;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint64_t p = blockIdx.x;
    const uint64_t g0 = p << kChunkLog2;
    const uint64_t left = a.n - g0;
    const uint32_t valid = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;
    Raw<kUnits> raw;
    load_raw<kUnits, kElem, true>(raw, static_cast<const uint8_t*>(a.in) + g0 * kElem, valid, t);
    float v[kRegs];
    units_to_l1<kUnits, false>(sh.sign[0], raw.u, v, t);
    if constexpr (MODE == Mode::MinMax) {
        const MinMax r = chunk_minmax(sh, v, lane, wave);
        if (t == 0) {
            static_cast<float*>(a.out)[2 * p] = r.lo;
            static_cast<float*>(a.out)[2 * p + 1] = r.hi;
        }
    } else {
        const float lo = a.range_in[2 * p], hi = a.range_in[2 * p + 1];
        quantize_store_range<BITS, false>(v, lo, hi, a.levels, g0, a.worker, a.key0, a.key1,
                                          static_cast<uint8_t*>(a.out), t);
    }
}

// Inverse direction, one chunk per workgroup.
//   SRC 0: rotated fp32 values (rht_inverse);  1: u8 sums;  2: u16 sums (thc_decode);
//       3: packed saturated aggregate, offset binary (thc_sat_decode)
//   SIGNED false: no sign diagonal on output (a pass of the full rotation)
template <int SRC, bool SIGNED = true>
__global__ __launch_bounds__(kThreads) void inverse_kernel(const ChunkArgs a) {
    __shared__ Shared sh;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t block = lay14::block_of_lane(lane), tp = (t & ~63u) | block;   // the thread's 32 coordinates
    const uint64_t p = blockIdx.x;
    const uint64_t g0 = p << kChunkLog2;
    const uint64_t left = a.n - g0;
    const uint32_t valid = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;
    float v[kRegs];
    if (SIGNED) fill_sign_table<true, false>(sh.sign[0], g0, a.key0, a.key1, t);
    if constexpr (SRC == 0) {
        Raw<8> raw;   // y is complete (padded), so every unit exists
        load_raw<8, 4>(raw, static_cast<const float*>(a.in) + g0, (uint32_t)kChunk, t);
        raw_to_lds<8>(sh, raw, t);
        __syncthreads();
        lds_to_l1<8, false>(sh, sh.sign[0], v, tp);
        // (a wave reads the units of its own 8 KB of the buffer, and the exchange stores there: no barrier)
    } else {
        // symmetric grid: yhat = S q - s;  min/max grid: yhat = S q + lo
        const bool ranged = a.range_in != nullptr;
        const float lo = ranged ? a.range_in[2 * p] : 0.0f;
        const float s = ranged ? -lo : a.scale_in[a.scale_shared ? 0 : p];
        const float step = (ranged ? a.range_in[2 * p + 1] - lo : s + s) / (float)a.levels;
        const float q = step / (float)a.W;
        if constexpr (SRC == 3) {
            // 32 coordinates = 4 * bits bytes per thread
            const uint32_t bits = a.bits;
            const uint32_t* src = reinterpret_cast<const uint32_t*>(
                static_cast<const uint8_t*>(a.in) + (g0 * bits) / 8u + (uint64_t)tp * (4u * bits));
            const int centre = (int)(a.levels >> 1);
            uint32_t word[8];
#pragma unroll
            for (int d = 0; d < 8; ++d) word[d] = (uint32_t)d < bits ? src[d] : 0u;
#pragma unroll
            for (int r = 0; r < kRegs; ++r) {
                uint32_t A;
                if (bits == 2) A = (word[r >> 4] >> (2 * (r & 15))) & 3u;
                else if (bits == 4) A = (word[r >> 3] >> (4 * (r & 7))) & 15u;
                else A = (word[r >> 2] >> (8 * (r & 3))) & 255u;
                v[r] = (float)((int)A - centre) * q;
            }
        } else if constexpr (SRC == 1) {
            const uint4* src = reinterpret_cast<const uint4*>(static_cast<const uint8_t*>(a.in) + g0) + 2 * tp;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint4 w = src[k];
                const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int d = 0; d < 4; ++d)
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        v[16 * k + 4 * d + b] = (float)((ww[d] >> (8 * b)) & 0xFFu) * q - s;
            }
        } else {
            const uint4* src = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.in) + g0) + 4 * tp;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint4 w = src[k];
                const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int d = 0; d < 4; ++d)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        v[8 * k + 2 * d + b] = (float)((ww[d] >> (16 * b)) & 0xFFFFu) * q - s;
            }
        }
    }
    NoHook none;
    rotate_lanes_to_l4d(sh, v, lane, block, wave, none);   // (its barrier also orders the sign table)
    store_signed_l4d<SIGNED>(sh.sign[0], v, static_cast<float*>(a.out) + g0, valid, t,
                             l4d_negated(lane, wave) ? -a.inv_sqrt_c : a.inv_sqrt_c);
}

template <bool BF16, Mode MODE>
hipError_t launch_bits(const ChunkArgs& a, dim3 grid, hipStream_t stream) {
    if constexpr (MODE == Mode::Encode) {
        const bool prio = grid.x <= 2u * (uint32_t)device_cus();
#define THC_ENCODE(BITS)                                                                                                  \
    if (prio) hipLaunchKernelGGL((per_worker_kernel<BF16, MODE, BITS, true>), grid, dim3(kThreads), 0, stream, a);        \
    else hipLaunchKernelGGL((per_worker_kernel<BF16, MODE, BITS, false>), grid, dim3(kThreads), 0, stream, a)
        if (a.bits == 2) {
            THC_ENCODE(2);
        } else if (a.bits == 4) {
            THC_ENCODE(4);
        } else {
            THC_ENCODE(8);
        }
#undef THC_ENCODE
    } else {
        hipLaunchKernelGGL((per_worker_kernel<BF16, MODE, 4>), grid, dim3(kThreads), 0, stream, a);
    }
    return hipGetLastError();
}

template <bool BF16>
hipError_t launch_unrotated(Mode mode, const ChunkArgs& a, dim3 grid, hipStream_t stream) {
    if (mode == Mode::MinMax)
        hipLaunchKernelGGL((unrotated_kernel<BF16, Mode::MinMax, 4>), grid, dim3(kThreads), 0, stream, a);
    else if (a.bits == 2)
        hipLaunchKernelGGL((unrotated_kernel<BF16, Mode::Encode, 2>), grid, dim3(kThreads), 0, stream, a);
    else if (a.bits == 4)
        hipLaunchKernelGGL((unrotated_kernel<BF16, Mode::Encode, 4>), grid, dim3(kThreads), 0, stream, a);
    else
        hipLaunchKernelGGL((unrotated_kernel<BF16, Mode::Encode, 8>), grid, dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace
}  // namespace k14

bool fast14_applicable(Mode mode, const ChunkArgs& a) {
    if (a.chunk_log2 != 14) return false;
    if ((a.padded >> 14) > 0x7FFFFFFFull) return false;
    if (a.out_bf16 || mode == Mode::Plain || mode == Mode::PlainDecode) return false;
    // without the rotation: the range and the encoder on a given range have a tuned form
    if (a.no_rotate && !(mode == Mode::MinMax || (mode == Mode::Encode && a.range_in))) return false;
    // a range is one or two scalar stores per chunk: its place needs no more than the ABI's alignment
    // (a worker's row of a W x chunks array starts anywhere)
    const bool scalar_out = mode == Mode::Absmax || mode == Mode::MinMax;
    return k14::aligned16(a.in) && (scalar_out || k14::aligned16(a.out));
}

hipError_t launch_fast14(Mode mode, const ChunkArgs& a, hipStream_t stream) {
    using namespace k14;
    const dim3 grid((uint32_t)(a.padded >> 14));
    if (grid.x == 0) return hipSuccess;
    if (a.no_rotate)
        return a.in_bf16 ? launch_unrotated<true>(mode, a, grid, stream) : launch_unrotated<false>(mode, a, grid, stream);
    switch (mode) {
        case Mode::Forward:
            return a.in_bf16 ? launch_bits<true, Mode::Forward>(a, grid, stream)
                             : launch_bits<false, Mode::Forward>(a, grid, stream);
        case Mode::Absmax:
            return a.in_bf16 ? launch_bits<true, Mode::Absmax>(a, grid, stream)
                             : launch_bits<false, Mode::Absmax>(a, grid, stream);
        case Mode::MinMax:
            return a.in_bf16 ? launch_bits<true, Mode::MinMax>(a, grid, stream)
                             : launch_bits<false, Mode::MinMax>(a, grid, stream);
        case Mode::Encode:
            return a.in_bf16 ? launch_bits<true, Mode::Encode>(a, grid, stream)
                             : launch_bits<false, Mode::Encode>(a, grid, stream);
        case Mode::Inverse:
            hipLaunchKernelGGL(inverse_kernel<0>, grid, dim3(kThreads), 0, stream, a);
            return hipGetLastError();
        case Mode::Plain:
            hipLaunchKernelGGL((inverse_kernel<0, false>), grid, dim3(kThreads), 0, stream, a);
            return hipGetLastError();
        case Mode::PlainDecode:
            if (a.sum_bytes == 1)
                hipLaunchKernelGGL((inverse_kernel<1, false>), grid, dim3(kThreads), 0, stream, a);
            else
                hipLaunchKernelGGL((inverse_kernel<2, false>), grid, dim3(kThreads), 0, stream, a);
            return hipGetLastError();
        case Mode::Decode:
            if (a.sat)
                hipLaunchKernelGGL(inverse_kernel<3>, grid, dim3(kThreads), 0, stream, a);
            else if (a.sum_bytes == 1)
                hipLaunchKernelGGL(inverse_kernel<1>, grid, dim3(kThreads), 0, stream, a);
            else
                hipLaunchKernelGGL(inverse_kernel<2>, grid, dim3(kThreads), 0, stream, a);
            return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

}  // namespace thc
