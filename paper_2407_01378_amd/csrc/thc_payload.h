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
// Read for the last time (ONCE) - but 8-bit payloads take two loads per thread from the same lines, and a line that the
// first one marks as used up may be gone before the second: unless stream_payloads they are read by ordinary
// loads (4 bits, one load per thread: the same either way).
template <int BITS, bool ONCE = BITS != 8>
__device__ __forceinline__ PayloadWords<BITS> load_payload_words(const uint8_t* p) {
    PayloadWords<BITS> r;
    if (BITS == 2) {
        const uint2 q = load_last_use(reinterpret_cast<const uint2*>(p));
        r.w[0] = q.x;
        r.w[1] = q.y;
    } else {
#pragma unroll
        for (int k = 0; k < BITS / 4; ++k) {
            const uint4* src = reinterpret_cast<const uint4*>(p) + k;
            const uint4 q = ONCE ? load_last_use(src) : *src;
            r.w[4 * k] = q.x;
            r.w[4 * k + 1] = q.y;
            r.w[4 * k + 2] = q.z;
            r.w[4 * k + 3] = q.w;
        }
    }
    return r;
}

// 8-bit payloads, `coords` of each of W workers, that are read as for the last time: those that outgrow the last-level
// cache (256 MB) beside the output, and, by the decoders of chunks of 2^14, those of a pass that about fills it with its
// gradients, where lines that are done with make room.  Encoder and decoder, three sets of buffers in turn, ordinary
// loads | last use, us:
//   chunk 2^14, exact sums  bf16, 8 workers: 22 MiB of payloads 34.1 | 33.8, 32 45.7 | 41.7, 40 58.0 | 54.6, 48 65.9 | 64.2, 58 75.3 | 74.2,
//                           72 90.4 | 92.3; 32 workers 26 43.7 | 43.4, 32 53.0 | 48.3, 54 78.1 | 72.6; fp32, 8 workers 22 41.3 | 40.1, 32 54.5 | 53.0,
//                           48 75.5 | 76.5, 54 85.4 | 88.4, 62 94.4 | 97.4
//                           8 workers x 17 M 144 | 153, x 25 M 220 | 220, x 34 M 294 | 292; 4 x 67 M 310 | 306; 16 x 17 M 304 | 297;
//                           batched 112 MB 128 | 136, 480 MB 670 | 654, 1048 MB 1127 | 1111
//   saturating              8 workers, 32 MiB 45.4 | 42.0, 48 67.3 | 64.0; x 21 M 186 | 190, x 25 M 221 | 221, x 34 M 294 | 292, x 67 M 580 | 567
//   min/max                 8 workers, 32 MiB 48.4 | 45.2, 48 70.0 | 69.6
//   small chunks            8 workers x 6 M 62 | 67, x 17 M 147 | 154, x 21 M 193 | 193, x 25 M 230 | 227, x 34 M 304 | 301 (it also stores the sums)
// Up to 8 M coordinates (more than 28 workers) ordinary loads hold longer: 64 x 5 M 375 | 387 us, 64 x 8 M 609 | 612, 32 x
// 8 M 333 | 336, saturating 378 | 390, 595 | 599 and 332 | 337, small chunks 32 x 8 M 330 | 335; 32 x 9 M 391 | 388, 390 | 383.
inline bool stream_payloads(uint32_t W, uint64_t coords, bool small_chunks = false) {
    const uint64_t bytes = W * coords;
    if (!small_chunks && bytes > 20ull << 20 && bytes <= 52ull << 20) return true;
    return bytes > (small_chunks ? 176ull : 224ull) << 20 && coords > 8ull << 20;
}

// The workers' payload words of one thread (its 32 coordinates) on their way into registers, group by
// group: a group is the payload of GROUP workers.  Two groups can be in flight at once (buffers 0 and 1, 32
// registers): while one is combined the next one's loads are on their way.
template <int BITS, bool BATCH, int GROUP = BITS == 8 ? 2 : 4, bool ONCE = BITS != 8>
struct PayloadLoads {
    static constexpr uint32_t kGroup = GROUP;
    // For a persistent kernel's next chunk: one group in flight (buffer 0) instead of two.  8-bit payloads that come
    // near the size of the last-level cache or outgrow it are served from both places, and more loads in flight do
    // not help there: 8 workers behind their encoder, 25 M coordinates 217.4 -> 215.3 us, 29 M 253.5 -> 252, 34 M
    // 286.5 -> 284.8; saturating 32 M 279 -> 273, 17 M 154.5 -> 153.3; smaller ones the same either way (17 M
    // 141).  4 bits: 8 x 26 M 188.5 us with two, 190 with one.
    static constexpr bool kOneAhead = BITS == 8;
    const FusedPayloadPtrs& ptrs;   // single bucket: the payload pointers, in the kernel arguments
    ConstU64Ptr pp;                 // batched: those of the bucket being summed, in its record
    uint32_t W;
    PayloadWords<BITS> x[2][GROUP];

    __device__ __forceinline__ const uint8_t* pointer(uint32_t w) const {
        return BATCH ? global_ptr<const uint8_t>(pp[w]) : ptrs.p[w];
    }
    __device__ __forceinline__ uint32_t groups() const { return (W + kGroup - 1u) / kGroup; }
    // Loads of one group into buffer B (nothing past the last worker).  A whole group has no condition per
    // worker: its pointers come in one scalar load.
    template <int B>
    __device__ __forceinline__ void issue(uint64_t byte0, uint32_t group) {
        const uint32_t w0 = group * kGroup;
        if (w0 >= W) return;
        if (w0 + kGroup <= W) {
#pragma unroll
            for (uint32_t j = 0; j < kGroup; ++j) x[B][j] = load_payload_words<BITS, ONCE>(pointer(w0 + j) + byte0);
            // (the empty assembly statements differ, so that the two branches are not merged into one that
            // picks its registers by address, which would put x into memory)
            asm volatile("; whole group");
        } else {
#pragma unroll
            for (uint32_t j = 0; j + 1u < kGroup; ++j)
                if (w0 + j < W) {
                    x[B][j] = load_payload_words<BITS, ONCE>(pointer(w0 + j) + byte0);
                    asm volatile("; worker of a part of a group");
                }
            asm volatile("; part of a group");
        }
    }
    // The same of a group that is known to be whole.
    template <int B>
    __device__ __forceinline__ void issue_whole(uint64_t byte0, uint32_t group) {
#pragma unroll
        for (uint32_t j = 0; j < kGroup; ++j)
            x[B][j] = load_payload_words<BITS, ONCE>(pointer(group * kGroup + j) + byte0);
    }
    __device__ __forceinline__ void begin(uint64_t byte0) {
        issue<0>(byte0, 0u);
        issue<1>(byte0, 1u);
    }
    __device__ __forceinline__ void begin_ahead(uint64_t byte0) {
        if constexpr (kOneAhead) issue<0>(byte0, 0u);
        else begin(byte0);
    }
};

// Their exact sum in sub-word lanes.
//   One group at a time, added as soon as it was loaded, is a chain of memory latencies for a thread that
//   sums more than the few groups that ride along with the previous chunk's rotation: 64 workers x 2^21
//   coordinates (128 chunks, 4 bits) 45 -> 22 us with two groups in flight and the 8-bit lanes below.
// WIDE: 16-bit accumulators for 4-bit payloads too (W * L > 255: more than 17 workers); lane q
// then holds coordinates q (low half) and q + 4 (high half) of the dword's 8.  The workers
// meet in 8-bit lanes first, kFlush groups of them (16 * 15 <= 255), which takes half the operations.
template <int BITS, bool BATCH = false, bool WIDE = false, bool ONCE = BITS != 8>
struct PayloadSum : PayloadLoads<BITS, BATCH, BITS == 8 ? 2 : 4, ONCE> {
    static_assert(!(WIDE && BITS != 4), "8-bit payloads always sum in 16-bit lanes, 2-bit ones in 8-bit lanes");
    using Loads = PayloadLoads<BITS, BATCH, BITS == 8 ? 2 : 4, ONCE>;
    using Loads::groups;
    using Loads::kGroup;
    using Loads::kOneAhead;
    using Loads::W;
    using Loads::x;
    static constexpr int kWords = BITS;                        // payload dwords per worker per thread
    static constexpr int kLanes = BITS == 8 ? 2 : 8 / BITS;    // sub-word accumulators per dword while adding
    static constexpr uint32_t kMask = BITS == 8 ? 0x00FF00FFu : BITS == 4 ? 0x0F0F0F0Fu : 0x03030303u;
    static constexpr uint32_t kFlush = 16u / kGroup;           // WIDE: groups that fit the 8-bit lanes
    uint32_t acc[kWords][kLanes];
    uint32_t wide[WIDE ? kWords : 1][4];

    __device__ __forceinline__ PayloadSum(const FusedPayloadPtrs& ptrs, ConstU64Ptr pp, uint32_t W)
        : Loads{ptrs, pp, W, {}} {}
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int d = 0; d < kWords; ++d)
#pragma unroll
            for (int k = 0; k < kLanes; ++k) acc[d][k] = 0u;
    }
    __device__ __forceinline__ void add_whole(const PayloadWords<BITS> (&y)[kGroup]) {
#pragma unroll
        for (uint32_t j = 0; j < kGroup; j += 2u)
#pragma unroll
            for (int d = 0; d < kWords; ++d)
#pragma unroll
                for (int q = 0; q < kLanes; ++q)   // (one three-operand addition for two workers)
                    acc[d][q] += ((y[j].w[d] >> (BITS * q)) & kMask) + ((y[j + 1].w[d] >> (BITS * q)) & kMask);
    }
    __device__ __forceinline__ void add_one(const PayloadWords<BITS>& y) {
#pragma unroll
        for (int d = 0; d < kWords; ++d)
#pragma unroll
            for (int q = 0; q < kLanes; ++q) acc[d][q] += (y.w[d] >> (BITS * q)) & kMask;
    }
    template <int B>
    __device__ __forceinline__ void add(uint32_t group) {
        const uint32_t w0 = group * kGroup;
        if (w0 + kGroup <= W) {
            add_whole(x[B]);
        } else {
#pragma unroll
            for (uint32_t j = 0; j + 1u < kGroup; ++j)
                if (w0 + j < W) add_one(x[B][j]);
        }
    }
    // WIDE: the 8-bit lanes into the wide ones, before they could overflow.
    __device__ __forceinline__ void flush() {
        if constexpr (WIDE) {
#pragma unroll
            for (int d = 0; d < kWords; ++d)
#pragma unroll
                for (int q = 0; q < kLanes; ++q) {
                    wide[d][q] += acc[d][q] & 0x00FF00FFu;
                    wide[d][q + 2] += (acc[d][q] >> 8) & 0x00FF00FFu;
                    acc[d][q] = 0u;
                }
        }
    }
    // The same behind the addition of `group`, where it is due.
    __device__ __forceinline__ void flush(uint32_t group) {
        if (WIDE && ((group + 1u) % kFlush == 0u || group + 1u == groups())) flush();
    }
    __device__ __forceinline__ void clear_wide() {
        if constexpr (WIDE) {
#pragma unroll
            for (int d = 0; d < kWords; ++d)
#pragma unroll
                for (int k = 0; k < 4; ++k) wide[d][k] = 0u;
        }
    }
    // Adds the groups from `from` on (even, less than kFlush; the caller has added those before), the first
    // two of which are in flight.
    __device__ __forceinline__ void rest(uint64_t byte0, uint32_t from) {
        clear_wide();
        for (uint32_t g = from; g < groups(); g += 2u) {
            add<0>(g);
            flush(g);
            this->template issue<0>(byte0, g + 2u);
            if (g + 1u < groups()) {
                add<1>(g + 1u);
                flush(g + 1u);
            }
            this->template issue<1>(byte0, g + 3u);
        }
    }
    // The same with one group in flight, `from` in buffer 0.
    __device__ __forceinline__ void rest_one_ahead(uint64_t byte0, uint32_t from) {
        for (uint32_t g = from; g < groups(); ++g) {
            if (g != from) this->template issue<0>(byte0, g);
            add<0>(g);
        }
    }
    __device__ __forceinline__ void all(uint64_t byte0) {
        this->begin(byte0);
        rest(byte0, 0u);
    }
    // The same for a kernel in which nothing rides along with the sum, and where its wait is a good part of the time.
    // The workers beyond the whole groups are loaded first and added last, so that the loop has whole
    // groups only: no condition between a load and its use, each wait is for its own group alone (`all` waits for the
    // first worker of a part of a group before it loads the second), and less code to fetch for few workers.
    // Small-chunk decoder, `all` | this, 2^10 coordinates per chunk, us: 64 workers x 2^20 at 8 bits 22.7 | 18.0,
    // at 4 bits 15.6 | 13.5, at 2 bits 14.4 | 9.4; 8 workers 6.9 | 6.5, 5.7 | 5.5, 5.7 | 5.4; 1 worker at 2 bits 6.2 | 6.0.
    // (The decoder of chunks of 2^14 has no registers left for it where it prepares a next chunk.)
    __device__ __forceinline__ void all_alone(uint64_t byte0) {
        const uint32_t whole = W / kGroup, more = W % kGroup;
        PayloadWords<BITS> y[kGroup - 1u];
#pragma unroll
        for (uint32_t j = 0; j + 1u < kGroup; ++j)
            if (j < more) y[j] = load_payload_words<BITS, ONCE>(this->pointer(whole * kGroup + j) + byte0);
        clear_wide();
        if (whole > 1u) {
            this->template issue_whole<0>(byte0, 0u);
            this->template issue_whole<1>(byte0, 1u);
            uint32_t g = 0;
            for (; g + 3u < whole; g += 2u) {
                add_whole(x[0]);
                this->template issue_whole<0>(byte0, g + 2u);
                add_whole(x[1]);
                this->template issue_whole<1>(byte0, g + 3u);
                if ((g + 2u) % kFlush == 0u) flush();
            }
            const bool three = (whole & 1u) != 0u;   // groups left: two or three
            add_whole(x[0]);
            if (three) this->template issue_whole<0>(byte0, g + 2u);
            add_whole(x[1]);
            if ((g + 2u) % kFlush == 0u) flush();
            if (three) add_whole(x[0]);
        } else if (whole != 0u) {
            this->template issue_whole<0>(byte0, 0u);
            add_whole(x[0]);
        }
#pragma unroll
        for (uint32_t j = 0; j + 1u < kGroup; ++j)
            if (j < more) add_one(y[j]);
        flush();   // (at most three whole groups and three workers since the last time: 15 * 15 <= 255)
    }

    // Sub-word lanes -> one sum per coordinate.
    __device__ __forceinline__ void unpack(uint32_t (&S)[32]) const {
#pragma unroll
        for (int d = 0; d < kWords; ++d) {
            if (BITS == 8) {         // dword d: coordinates 4d..4d+3; lane 0 = even, lane 1 = odd
                S[4 * d + 0] = acc[d][0] & 0xFFFFu;
                S[4 * d + 1] = acc[d][1] & 0xFFFFu;
                S[4 * d + 2] = acc[d][0] >> 16;
                S[4 * d + 3] = acc[d][1] >> 16;
            } else if (WIDE) {       // dword d: 8 coordinates; lane q = coordinates q and q + 4
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    S[8 * d + q] = wide[d][q] & 0xFFFFu;
                    S[8 * d + 4 + q] = wide[d][q] >> 16;
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
