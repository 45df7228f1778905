// The workers' payload words of one thread (32 consecutive coordinates) and their exact sum:
// shared by the decoders.
#pragma once

#include "thc_device.h"
#include "thc_internal.h"

#pragma clang fp contract(off)

namespace thc {
namespace k14 {

// The records of a batched launch were written by earlier kernels and are never written by
// this one: reading them through the constant address space lets the compiler use scalar
// loads (one request per wave, served by the scalar cache) where a global pointer, which
// might alias the kernel's stores, would get a vector load and its full memory latency.
#define THC_CONSTANT __attribute__((address_space(4)))
typedef const BatchRecord THC_CONSTANT* ConstRecordPtr;
typedef const uint64_t THC_CONSTANT* ConstU64Ptr;
// A pointer that was read from a record as an integer, as a pointer into global memory: the
// compiler then uses global loads and stores for it, as it does for pointers that arrive as
// kernel arguments, instead of the slower generic (flat) ones, which also count as LDS
// operations in the wait counters.
template <typename T>
__device__ __forceinline__ T* global_ptr(uint64_t address) {
    typedef T __attribute__((address_space(1))) * Global;
    return (T*)(Global)address;
}

template <int BITS>
struct PayloadWords {
    uint32_t w[BITS];
};
template <int BITS>
__device__ __forceinline__ PayloadWords<BITS> load_payload_words(const uint8_t* p) {
    PayloadWords<BITS> r;
    if (BITS == 2) {
        const uint2 q = load_last_use(reinterpret_cast<const uint2*>(p));
        r.w[0] = q.x;
        r.w[1] = q.y;
    } else {
#pragma unroll
        for (int k = 0; k < BITS / 4; ++k) {
            const uint4 q = load_last_use(reinterpret_cast<const uint4*>(p) + k);
            r.w[4 * k] = q.x;
            r.w[4 * k + 1] = q.y;
            r.w[4 * k + 2] = q.z;
            r.w[4 * k + 3] = q.w;
        }
    }
    return r;
}

// Sum of the workers' payload words of one thread (its 32 coordinates) in sub-word lanes,
// built up group by group: a group is the payload of kGroup workers in flight at once.
// WIDE: 16-bit accumulators for 4-bit payloads too (W * L > 255: more than 17 workers); lane q
// then holds coordinates q (low half) and q + 16 / BITS (high half) of the dword's 32 / BITS.
// GROUP 0: at most 16 registers of payload in flight.
template <int BITS, bool BATCH = false, bool WIDE = false, int GROUP = 0>
struct PayloadSum {
    static_assert(!(WIDE && BITS == 8), "8-bit payloads always sum in 16-bit lanes");
    static constexpr int kWords = BITS;                        // payload dwords per worker per thread
    static constexpr int kLanes = BITS == 8 ? 2 : (WIDE ? 16 : 8) / BITS;   // sub-word accumulators per dword
    static constexpr uint32_t kMask = BITS == 8 ? 0x00FF00FFu
                                      : WIDE    ? (BITS == 4 ? 0x000F000Fu : 0x00030003u)
                                                : (BITS == 4 ? 0x0F0F0F0Fu : 0x03030303u);
    static constexpr int kGroup = GROUP != 0 ? GROUP : (BITS == 8 ? 2 : 4);
    const FusedPayloadPtrs& ptrs;   // single bucket: the payload pointers, in the kernel arguments
    ConstU64Ptr pp;                 // batched: those of the bucket being summed, in its record
    uint32_t W;
    uint32_t acc[kWords][kLanes];
    PayloadWords<BITS> x[kGroup];

    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int d = 0; d < kWords; ++d)
#pragma unroll
            for (int k = 0; k < kLanes; ++k) acc[d][k] = 0u;
    }
    __device__ __forceinline__ void issue(uint64_t byte0, uint32_t group) {
#pragma unroll
        for (int j = 0; j < kGroup; ++j)
            if (group * kGroup + j < W) {
                const uint8_t* src = BATCH ? global_ptr<const uint8_t>(pp[group * kGroup + j])
                                           : ptrs.p[group * kGroup + j];
                x[j] = load_payload_words<BITS>(src + byte0);
            }
    }
    __device__ __forceinline__ void add(uint32_t group) {
#pragma unroll
        for (int j = 0; j < kGroup; ++j)
            if (group * kGroup + j < W) {
#pragma unroll
                for (int d = 0; d < kWords; ++d)
#pragma unroll
                    for (int q = 0; q < kLanes; ++q) acc[d][q] += (x[j].w[d] >> (BITS * q)) & kMask;
            }
    }
    __device__ __forceinline__ uint32_t groups() const { return (W + kGroup - 1) / kGroup; }

    // Sub-word lanes -> one sum per coordinate.
    __device__ __forceinline__ void unpack(uint32_t (&S)[32]) const {
#pragma unroll
        for (int d = 0; d < kWords; ++d) {
            if (BITS == 8) {         // dword d: coordinates 4d..4d+3; lane 0 = even, lane 1 = odd
                S[4 * d + 0] = acc[d][0] & 0xFFFFu;
                S[4 * d + 1] = acc[d][1] & 0xFFFFu;
                S[4 * d + 2] = acc[d][0] >> 16;
                S[4 * d + 3] = acc[d][1] >> 16;
            } else if (WIDE) {       // dword d: 32/BITS coordinates; lane q = coordinates q and q + 16/BITS
                constexpr int per = 32 / BITS;
#pragma unroll
                for (int q = 0; q < kLanes; ++q) {
                    S[per * d + q] = acc[d][q] & 0xFFFFu;
                    S[per * d + kLanes + q] = acc[d][q] >> 16;
                }
            } else {                 // dword d: 32/BITS coordinates; lane q byte b = coordinate (8/BITS) b + q
                constexpr int per = 32 / BITS;
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int q = 0; q < kLanes; ++q)
                        S[per * d + kLanes * b + q] = (acc[d][q] >> (8 * b)) & 0xFFu;
            }
        }
    }
};

// The thread's 32 sums to the caller's integer aggregate: u16 or u8 elements from `dst` on.
__device__ __forceinline__ void store_sums16(const uint32_t (&S)[32], uint16_t* dst) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
        *reinterpret_cast<uint4*>(dst + 8 * k) =
            make_uint4(S[8 * k] | (S[8 * k + 1] << 16), S[8 * k + 2] | (S[8 * k + 3] << 16),
                       S[8 * k + 4] | (S[8 * k + 5] << 16), S[8 * k + 6] | (S[8 * k + 7] << 16));
}
__device__ __forceinline__ void store_sums8(const uint32_t (&S)[32], uint8_t* dst) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        uint32_t o[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int r = 16 * k + 4 * d;
            o[d] = S[r] | (S[r + 1] << 8) | (S[r + 2] << 16) | (S[r + 3] << 24);
        }
        *reinterpret_cast<uint4*>(dst + 16 * k) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

}  // namespace k14
}  // namespace thc
