// Fused kernels for chunk_log2 = 14.
//
// encode_all: ONE pass over every worker's gradient.  A work item is (chunk p, worker
// w); the workgroup that owns it rotates the chunk, publishes the chunk's largest
// magnitude to per-chunk slots in global memory, waits until all W workers of chunk p
// have published, and only then quantizes - the rotated chunk never leaves registers,
// so each gradient is read from HBM once.  The grid is persistent and no larger than
// what is resident at once (occupancy x CUs), items are dealt round-robin
// (item = workgroup + k * grid), so the W owners of a chunk run side by side and every
// wait is for a workgroup that is already running.  Waits are bounded: on time-out an
// error word is set and the wave carries on, so every wave always exits.
//
// aggregate_decode: sums the W payloads of a chunk in packed sub-word lanes straight
// into the inverse rotation; the integer sums never touch HBM unless asked for.
#include "thc_core14.h"
#include "thc_internal.h"
#include "thc_payload.h"
#include "thc_resident.h"

#pragma clang fp contract(off)

namespace thc {
namespace k14 {
namespace {

constexpr uint32_t kWaves = kThreads / 64;
// Second argument of __launch_bounds__ (waves per SIMD the compiler must allow): two
// workgroups of 8 waves per CU = 4 waves on each of the 4 SIMDs = at most 128 VGPRs.
constexpr int kWavesPerSimd = 4;
// How the workgroups of a chunk tell one another its range (template argument of the encoder).
enum class Words : int {
    PerWave = 0,    // every wave publishes a word and reads all words: up to 16 workers
    PerGroup = 1,   // one word per workgroup (the waves' maxima meet in LDS), read by every wave: up to 32, and see one_reader
    OneReader = 2   // the same, read by one wave for all: beyond
};
constexpr uint32_t kPerWaveMaxWorkers = 16;
constexpr uint32_t kPerGroupMaxWorkers = 32;
// Pauses of the wait for the peers' range words, in units of 64 clocks (s_sleep): in front of the first read,
// and between reads.  A word takes about 2 us from one workgroup to another, the peers of a chunk
// publish up to about 2 us apart, and reads that come back incomplete load the path the words travel on.
//   PerWave    8 workers x 1600 chunks: 16 .. 48 alike, 8 and 64 2 to 3 % slower
//   PerGroup   32 workers x 512 chunks 270 us with 32, 256 with 40, 184 chunks the same; 24 x 244 chunks 94.7 -> 92
//   OneReader  an eighth of the reads; a longer pause from the 8th round on, because how long a workgroup is out of
//              the way of the other one on its CU decides whether the two stay half an item apart.  64 workers, bf16, 4 bits,
//              128 chunks 140 -> 130 us, 256 chunks 279 -> 248; 8 bits, 245 chunks 363 -> 284 (32 workers x 184
//              chunks would lose 5 %)
//   few rounds bf16 and up to 4 bits 16: 32 workers x 48 chunks 24.1 us (32: 24.4), 64 x 16 chunks 19.6 (20.2); fp32 or 8
//              bits, where an item is longer, 32: 32 x 64 chunks bf16 8 bits 32.1 (16: 35.5), fp32 4 bits 43.2 (46.1), 64 x 32 fp32 41.0 (44.6)
//   one item   (PerWave) 4 chunks x 8 workers 14.7 -> 14.4 us with the decoder, 2 chunks x 2 workers 13.0 -> 12.4; where more than
//              three quarters of the places are taken 24: with the decoder, fp32 4 bits, 8 | 24, 15 x 34 chunks 23.9 | 21.0, 14 x 36
//              23.5 | 21.3, 16 x 32 25.3 | 22.4, bf16 9 x 50 19.5 | 17.9; fewer, 12 x 30 17.4 | 18.5, 8 x 33 15.6 | 16.6
constexpr int kFirstPollSleep = 32;
constexpr int kFirstPollSleepPerGroup = 40;
constexpr int kFirstPollSleepLate = 48;
constexpr uint32_t kLateRound = 8;
constexpr int kFirstPollSleepFewRounds = 16;   // PerGroup, OneReader
constexpr uint32_t kFewRounds = 4;
constexpr int kFirstPollSleepOne = 8, kFirstPollSleepOneCrowded = 24;   // PerWave
constexpr int kPollSleep = 8;
constexpr int kPollSleepOneReader = 4;
// fp32 gradients of all workers that do not fit the last-level cache (256 MB, and a quarter more, because part of them is
// still there) are read as for the last time: 64 KB per item.  A pass over 8 workers with one | two | three sets of
// gradients in turn, us, ordinary loads -> these: 134 MB 43.2 -> 47.4 | 44.0 -> 46.6 | 49.1 -> 47.4, 268 MB 77.1 -> 81.0 |
// 83.7 -> 80.9 | 83.9 -> 81.8, 336 MB 99.6 -> 99.7 | 101.7 -> 99.0; 818 MB 238 -> 228; 64 workers, 537 MB 183 -> 162.  A
// thread of bf16 input loads its own 64 bytes, four times from the same lines, and needs the caches for it.
constexpr uint64_t kStreamedItems = (320ull << 20) >> 16;
// ------------------------------------------------------------------ encode_all
__device__ __forceinline__ ConstRecordPtr batch_record(const BatchArgs& batch, uint32_t k) {
    return (ConstRecordPtr)(batch.records + (uint64_t)k * batch.record_bytes);
}

// What an item needs to know about the bucket its chunk belongs to; the same for every
// lane, so it lives in scalar registers.  A single-bucket call has one view for good; a
// batched call looks the view up in the records as its chunks move from bucket to bucket.
struct BucketView {
    uint64_t n;          // coordinates of the bucket
    uint64_t chunk0;     // number of its first chunk in the launch's chunk numbering
    uint32_t key0, key1;
    const void* grad;    // of this workgroup's worker
    uint8_t* payload;
    float* scale;
};

// ODD: bf16 input with an odd number of coordinates.  Its last coordinate shares a dword
// with nothing, which the range check of a buffer load (done per dword) would cut off: its owner
// fetches it by itself and puts it in when the item starts.  (An element-wise loader for the last chunk, which
// merged its registers with the whole chunks' on every item, left it to the compiler whether an item waited for the loads
// that it had just issued: 8 workers x 8.2 M, 4 bits 66.3 us, 72.8 in a build with the registers allocated otherwise, 65.5 so; 8 x 4.2 M
// 41.6 -> 40.4, 64 x 1 M 77.5 -> 69.4.)
// BATCH: the launch covers several buckets (a.chunks is their total, chunks are numbered
// through all of them); everything per bucket comes from the records in device memory.
// MINMAX: the grid runs from the chunk's smallest to its largest value instead of
// symmetrically around zero: every wave publishes two words (the maximum, then the negated
// minimum, both through order_key() so that both are combined by a maximum), `scale` receives
// (lo, hi) pairs, and the quantizer subtracts lo.
// WORDS PerGroup, OneReader: one range word per WORKGROUP instead of one per wave (the waves' maxima are combined
// through LDS at the barrier that opens the last exchange, and wave 0 publishes and clears).
// For many workers: with W = 64 a chunk would otherwise have 512 words, every polling wave
// would read 2 KB per poll, and that traffic delays the words it waits for.  At W = 8 the
// later publication costs more than the lighter polls save, so the per-wave form stays.
// ONE: a launch of one item per workgroup.  There is no next item to load for, and the rounding bytes are drawn while
// the input is on its way.  With the decoder and the pauses above, us: 8 workers x 50257 14.2 -> 13.0, 8 x 50 chunks 18.1 -> 17.3, fp32
// 19.4 -> 17.2, 16 x 23 chunks at 8 bits 26.2 -> 20.9, 2 x 200 17.5 -> 16.5, 20 x 20 19.6 -> 18.9, 32 x 9 at 8 bits 23.6 -> 22.9, 48 x 8 at 8
// bits 27.6 -> 26.8, 64 x 8 26.5 -> 25.9.
template <bool BF16, bool ODD, bool BATCH, bool MINMAX = false, Words WORDS = Words::PerWave, bool ONE = false>
struct EncodeAllCtx {
    static constexpr bool WGWORD = WORDS == Words::PerGroup || WORDS == Words::OneReader;
    static_assert(!MINMAX || WORDS == Words::PerWave, "the other forms exist for the symmetric grid only");
    static constexpr uint32_t kWordsPerWorker = WGWORD ? 1u : kWaves;
    static constexpr int kUnits = BF16 ? 4 : 8;
    static constexpr int kElem = BF16 ? 2 : 4;
    // bf16: every thread loads its own 64 consecutive bytes one item ahead, so the input
    // never crosses LDS.  fp32 (128 bytes per thread, 32 registers in flight) loads in
    // coalesced order when the item starts and goes through the buffer.
    static constexpr bool kDirect = BF16;
    const EncodeAllArgs& a;
    const FusedWorkerPtrs& ptrs;
    const BatchArgs& batch;
    Shared& sh;
    Raw<kUnits> raw;        // input of the next item to enter the pipeline, in flight
    struct Nothing {};      // (members that a form does not have take no part in its register allocation)
    std::conditional_t<ODD, uint32_t, Nothing> odd_tail;   // the last coordinate of an odd count, in the thread that owns it, with that input
    uint32_t t, lane, wave, nwords;
    uint32_t block, tp;     // the lane's block of 32 coordinates in the wave (thc_lanes.h), in the chunk
    uint32_t w;             // worker of every item of this workgroup (the grid is a multiple of W)
    uint32_t dp;            // chunk stride between consecutive items of this workgroup
    uint32_t parity;        // which sign table the next front() reads
    uint32_t prev;          // chunk of the workgroup's previous item, kNone before the first
    uint32_t bidx;          // BATCH: bucket of the most recent look-up (chunks only move forward)
    uint64_t boundary;      // BATCH: first chunk of the bucket after that one
    BucketView cur, nxt;    // of the item being processed / of the item whose input is in flight
    std::conditional_t<ONE, Drawn, Nothing> drawn;         // the item's rounding bytes
    static constexpr uint32_t kNone = 0xFFFFFFFFu;

    // MINMAX: the chunk's words as 8-byte pairs (the slots start 16-byte aligned and a chunk
    // has an even number of 32-bit words)
    __device__ __forceinline__ uint64_t* pairs(uint64_t p) const {
        return reinterpret_cast<uint64_t*>(a.slots + p * nwords);
    }

    __device__ __forceinline__ BucketView view_of(uint64_t p) {
        if constexpr (BATCH) {
            while (bidx + 1u < batch.count && p >= batch_record(batch, bidx + 1u)->chunk0) ++bidx;
            ConstRecordPtr r = batch_record(batch, bidx);
            boundary = bidx + 1u < batch.count ? batch_record(batch, bidx + 1u)->chunk0 : ~0ull;
            ConstU64Ptr ptr = (ConstU64Ptr)(r + 1);   // W gradients, then W payloads
            BucketView bv{r->n, r->chunk0, r->key0, r->key1, reinterpret_cast<const void*>(ptr[w]),
                          reinterpret_cast<uint8_t*>(ptr[a.W + w]), r->scale};
            // The record has arrived before the look-up returns.  Scalar loads complete out of
            // order, so one that is still in flight when the item's LDS exchanges start would
            // make every wait on an LDS load a wait for ALL of them (no overlap of the
            // exchange with the arithmetic that follows it), on every item, although a
            // look-up happens once per bucket.
            asm volatile("" : "+s"(bv.n), "+s"(bv.chunk0), "+s"(bv.key0), "+s"(bv.key1), "+s"(bv.grad),
                         "+s"(bv.payload), "+s"(bv.scale), "+s"(boundary), "+s"(bidx));
            return bv;
        } else {
            return BucketView{a.n, 0u, a.key0, a.key1, ptrs.grad[w], ptrs.payload[w], a.scale};
        }
    }

    // The chunk's raw 16-byte units.  Through a buffer descriptor whose range is the part of
    // the chunk that exists, reads beyond it return zero: there is no ragged path, and the
    // load may be issued for a chunk past the end (range 0), which keeps the prefetch of the
    // next item unconditional.
    __device__ __forceinline__ void load(uint64_t p, const BucketView& bv) {
        const uint64_t g0 = (p - bv.chunk0) << kChunkLog2;
        uint64_t left = p < a.chunks ? bv.n - g0 : 0u;
        if (left > (uint64_t)kChunk) left = kChunk;
        uint64_t addr = reinterpret_cast<uint64_t>(bv.grad) + (p < a.chunks ? g0 * kElem : 0u);
        // the descriptor is the same for every lane: it belongs in scalar registers
        addr = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(addr >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)addr);
        const uint32_t bytes = (ODD ? (uint32_t)left & ~1u : (uint32_t)left) * kElem;   // a multiple of 4
        __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            reinterpret_cast<void*>(addr), 0, bytes, 0x00020000);
        auto units = [&](auto policy) {
            typedef uint32_t u4v __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int j = 0; j < kUnits; ++j) {
                // fp32: the wave's own 8 KB in coalesced order, dealt out through its part of the buffer
                const uint32_t unit = kDirect ? kUnits * tp + j : wave * 512u + j * 64u + lane;
                const u4v q = __builtin_amdgcn_raw_buffer_load_b128(rsrc, unit * 16u, 0, decltype(policy)::value);
                raw.u[j] = make_uint4(q.x, q.y, q.z, q.w);
            }
        };
        if (!kDirect && a.chunks * a.W > kStreamedItems) units(std::integral_constant<int, kStreaming>{});
        else units(std::integral_constant<int, 0>{});
        if constexpr (ODD) {
            if (left & 1u) {   // (the bucket's last chunk)
                odd_tail = 0u;
                if (tp == (uint32_t)left >> 5) odd_tail = reinterpret_cast<const uint16_t*>(addr)[left - 1u];
            }
        }
    }
    __device__ __forceinline__ auto drawn_bytes() const {
        if constexpr (ONE) return static_cast<const Drawn*>(&drawn);
        else return nullptr;
    }
    // ODD: odd_tail into the input of chunk p, whose bucket is cur.
    __device__ __forceinline__ void put_odd_tail(uint64_t p) {
        const uint64_t left = cur.n - ((p - cur.chunk0) << kChunkLog2);
        if (left >= (uint64_t)kChunk || !(left & 1u) || tp != (uint32_t)left >> 5) return;
        const uint32_t d = ((uint32_t)left & 31u) >> 1;   // dword of the thread's 16 that holds it
#pragma unroll
        for (int k = 0; k < kUnits; ++k) {
            raw.u[k].x = d == 4u * k ? odd_tail : raw.u[k].x;
            raw.u[k].y = d == 4u * k + 1u ? odd_tail : raw.u[k].y;
            raw.u[k].z = d == 4u * k + 2u ? odd_tail : raw.u[k].z;
            raw.u[k].w = d == 4u * k + 3u ? odd_tail : raw.u[k].w;
        }
    }
    __device__ __forceinline__ void fill_signs(uint64_t p, const BucketView& bv, uint32_t which) {
        fill_sign_table<!BF16, BF16>(sh.sign[which], (p - bv.chunk0) << kChunkLog2, bv.key0, bv.key1, t);
    }

    // Front half of an item: bring the input into registers (layout L1), rotate, publish
    // this wave's share of the chunk's range, and bring the chunk into the quantizer's
    // layout.  The direct form also fills the sign table of the workgroup's next item,
    // which is read only after the barriers of this item's exchanges.
    __device__ __forceinline__ void front(float (&v)[kRegs], uint64_t p) {
        const bool more = !ONE && p + dp < a.chunks;
        if constexpr (kDirect) {
            if constexpr (ODD) put_odd_tail(p);
            units_to_l1<kUnits, true>(sh.sign[parity], raw.u, v, tp);
        } else {
            load(p, cur);
            uint4* stage = reinterpret_cast<uint4*>(sh.xb) + 512u * wave;
#pragma unroll
            for (int j = 0; j < kUnits; ++j) stage[lay14::stage_unit((uint32_t)j * 64u + lane)] = raw.u[j];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            uint4 unit[kUnits];
#pragma unroll
            for (int k = 0; k < kUnits; ++k) unit[k] = stage[lay14::stage_unit(8u * block + k)];
            units_to_l1<kUnits, true>(sh.sign[parity], unit, v, tp);
        }
        // the conversion is complete before the registers of `raw` are loaded again: without
        // this the compiler moves it below the loads and copies `raw` out of their way
#pragma unroll
        for (int i = 0; i < kRegs; ++i) asm volatile("" : "+v"(v[i]));
        asm volatile("" ::: "memory");
        if (BATCH && more && p + dp >= boundary) nxt = view_of(p + dp);   // rarely: a new bucket
        if (kDirect && !ONE) load(p + dp, nxt);
        if (more) fill_signs(p + dp, nxt, parity ^ 1u);
        parity ^= 1u;
        rotate_lanes_to_l3<true>(sh, v, lane, block, wave);
        // One word per wave, value | valid bit (non-negative floats order like their bit
        // patterns and leave bit 31 free).  The words travel between workgroups only
        // through device-scope stores and loads, which are served at the memory side, so
        // no cache write-back or invalidate is needed.  The slots start zeroed.
        if constexpr (MINMAX) {
            // (the scaling by 2^-7 is exact and monotone: it commutes with min and max)
            MinMax r = thread_minmax(v);
            if (odd_parity4((lane & 3u) | ((wave >> 1) << 2))) r = MinMax{-r.hi, -r.lo};   // (i5, i6, i7, i8)
            const uint32_t khi = wave_umax(order_key(rotated_end(r.hi)));
            const uint32_t klo = wave_umax(order_key(-rotated_end(r.lo)));
            // one 8-byte word per wave, (key of the maximum) << 32 | key of the negated minimum:
            // an aligned 8-byte store is one transaction, so a reader sees both or neither
            if (lane == 0)
                __hip_atomic_store(pairs(p) + kWaves * w + wave, ((uint64_t)khi << 32) | klo, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        } else if constexpr (WGWORD) {
            const float m = wave_absmax(v) * kInvSqrtC;
            if (lane == 0) sh.red[wave] = m;
            // l3_to_l4e_lanes with the publication behind a barrier in front
            __syncthreads();
            set_prio<true, kPrioExchange>();
            if (wave == 0 && lane == 0) {
                float mw = fmaxf(fmaxf(fmaxf(sh.red[0], sh.red[1]), fmaxf(sh.red[2], sh.red[3])),
                                 fmaxf(fmaxf(sh.red[4], sh.red[5]), fmaxf(sh.red[6], sh.red[7])));
                __hip_atomic_store(&a.slots[p * nwords + w], __float_as_uint(mw) | 0x80000000u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            x3e_store(sh, v, lane, wave);
            __syncthreads();
            x3e_load(sh, v, block, wave);
            set_prio<true, kPrioTail>();
            return;
        } else {
            const float m = wave_absmax(v) * kInvSqrtC;
            if (lane == 0)
                __hip_atomic_store(&a.slots[p * nwords + kWaves * w + wave],
                                   __float_as_uint(m) | 0x80000000u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        l3_to_l4e_lanes<true>(sh, v, lane, block, wave);
    }

    // Back half: wait until every wave of every worker of the chunk has published, take
    // the largest value as the shared scale, quantize and store.  The wait is bounded:
    // on time-out the error word is set and the wave carries on.
    template <int BITS>
    __device__ __forceinline__ void back(const float (&v)[kRegs], uint64_t p) {
        const uint32_t* slot = a.slots + p * nwords;
        uint32_t mx = 0u, mx2 = 0u;   // mx2: MINMAX only, the negated minima
        bool done = false;
        bool polls = true;
        if constexpr (WGWORD) {
            if (WORDS == Words::OneReader) polls = __builtin_amdgcn_readfirstlane((int)wave) == 0;
            if (polls) {
                constexpr int kFew = BF16 && BITS <= 4 ? kFirstPollSleepFewRounds : kFirstPollSleep;
                if (a.chunks <= kFewRounds * (uint64_t)dp) __builtin_amdgcn_s_sleep(kFew);
                else if (WORDS == Words::PerGroup) __builtin_amdgcn_s_sleep(kFirstPollSleepPerGroup);
                else if (p < kLateRound * (uint64_t)dp) __builtin_amdgcn_s_sleep(kFirstPollSleep);
                else __builtin_amdgcn_s_sleep(kFirstPollSleepLate);
            }
        } else {
            if (ONE && a.crowded) __builtin_amdgcn_s_sleep(kFirstPollSleepOneCrowded);
            else __builtin_amdgcn_s_sleep(ONE ? kFirstPollSleepOne : kFirstPollSleep);
        }
        for (uint32_t spins = 0; polls; ++spins) {
            if constexpr (MINMAX) {
                const uint32_t half = kWaves * a.W;
                const uint64_t* pair = pairs(p);
                bool all_valid = true;
                mx = mx2 = 0u;
                for (uint32_t base = 0; base < half; base += 64u) {
                    const uint32_t i = base + lane;
                    if (i < half) {
                        const uint64_t v = __hip_atomic_load(&pair[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const uint32_t vh = (uint32_t)(v >> 32), vl = (uint32_t)v;
                        all_valid = all_valid && v != 0ull;   // (neither key is ever zero)
                        mx = vh > mx ? vh : mx;
                        mx2 = vl > mx2 ? vl : mx2;
                    }
                }
                done = __all(all_valid);
            } else {
                uint32_t all_valid = 0x80000000u;
                mx = 0u;
                for (uint32_t base = 0; base < nwords; base += 64u) {
                    const uint32_t i = base + lane;
                    const uint32_t val =
                        i < nwords ? __hip_atomic_load(&slot[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                   : 0x80000000u;
                    all_valid &= val;
                    const uint32_t mag = val & 0x7FFFFFFFu;
                    mx = mag > mx ? mag : mx;
                }
                done = __all(all_valid != 0u);
            }
            if (done || spins >= a.max_spins) break;
            __builtin_amdgcn_s_sleep(WORDS == Words::OneReader ? kPollSleepOneReader : kPollSleep);
        }
        // Every earlier vector-memory operation of the wave has completed (the read of the range
        // words just did), among them the loads of the next item's input.  Passing those
        // registers through an empty asm tells the compiler so: the next item then starts
        // without a wait on them, which would also wait for the stores issued below.
        // (OneReader: a wave that has not polled waits for them here.)
        if (kDirect && !ONE) {
#pragma unroll
            for (int j = 0; j < kUnits; ++j)
                asm volatile("" : "+v"(raw.u[j].x), "+v"(raw.u[j].y), "+v"(raw.u[j].z), "+v"(raw.u[j].w));
        }
        if (polls && !done && lane == 0)
            __hip_atomic_store(a.error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // The workspace leaves the kernel as it entered it, all zero.  A peer's wave
        // publishes for this chunk only after the barriers of this item's rotation,
        // which every wave of its workgroup reaches only after reading the words of
        // the workgroup's previous chunk; with all of this chunk's words seen, nobody
        // will read the previous chunk's words again, and this wave clears its own.
        if (done && prev != kNone && lane == 0 && (!WGWORD || wave == 0)) {
            if constexpr (MINMAX)
                __hip_atomic_store(pairs(prev) + kWaves * w + wave, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else
                __hip_atomic_store(&a.slots[(uint64_t)prev * nwords + kWordsPerWorker * w + (WGWORD ? 0u : wave)],
                                   0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        uint32_t sbits = wave_umax(mx);
        if constexpr (WORDS == Words::OneReader) {   // (red is written again behind the next item's first barrier)
            if (polls && lane == 0) sh.red[0] = __uint_as_float(sbits);
            __syncthreads();
            sbits = __float_as_uint(sh.red[0]);
        }
        prev = (uint32_t)p;
        const uint64_t pl = p - cur.chunk0;   // the chunk's number inside its bucket
        const float sgn = odd_parity4(block) ? -1.0f : 1.0f;   // the thread's values are negated
        if constexpr (MINMAX) {
            // (after an expired wait a word may be missing; zero then stands for "nothing seen")
            const uint32_t lbits = wave_umax(mx2);
            const float hi = sbits != 0u ? order_value(sbits) : 0.0f;
            const float lo = lbits != 0u ? -order_value(lbits) : 0.0f;
            float* range = global_ptr<float>(reinterpret_cast<uint64_t>(cur.scale));
            if (w == 0 && t == 0) {
                range[2 * pl] = lo;
                range[2 * pl + 1] = hi;
            }
            // (no clamp: lo and hi are the chunk's own extremes, see quantize_pack)
            quantize_store_range<BITS, true, false>(v, lo, hi, a.levels, pl << kChunkLog2, w, cur.key0, cur.key1,
                                             global_ptr<uint8_t>(reinterpret_cast<uint64_t>(cur.payload)), tp,
                                             kInvSqrtC * sgn, drawn_bytes());
            return;
        }
        const float s = __uint_as_float(sbits);
        // (the view's pointers are re-tagged as global here: in a batched launch they come out of
        // the look-up's register barrier as plain addresses)
        if (w == 0 && t == 0) global_ptr<float>(reinterpret_cast<uint64_t>(cur.scale))[pl] = s;
        quantize_store<BITS, false, true>(v, s, a.levels, pl << kChunkLog2, w, cur.key0, cur.key1,
                                          global_ptr<uint8_t>(reinterpret_cast<uint64_t>(cur.payload)), tp, sgn,
                                          drawn_bytes());
    }

    // After the workgroup's last item: its words have no later chunk to vouch for them, so
    // the workgroups of the chunk count themselves off and the last one clears the words
    // of all of them, and the counter.
    __device__ __forceinline__ void finish() {
        if (prev == kNone) return;
        __syncthreads();   // every wave of this workgroup has read the chunk's words
        if (wave != 0) return;
        uint32_t arrived = 0u;
        if (lane == 0)
            arrived = __hip_atomic_fetch_add(&a.done[prev], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        arrived = (uint32_t)__builtin_amdgcn_readfirstlane((int)arrived);
        if (arrived == a.W - 1u) {
            uint32_t* words = a.slots + (uint64_t)prev * nwords;
            for (uint32_t i = lane; i < nwords; i += 64u)
                __hip_atomic_store(&words[i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0)
                __hip_atomic_store(&a.done[prev], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
};

constexpr int kStaggerSleeps = 6;   // late start of half the grid, in units of s_sleep 16 (1024 clocks)

// Items are (chunk, worker) pairs; workgroup g of a grid of G (a multiple of W) takes worker
// g mod W of chunks g / W, g / W + G / W, ...  The peers of an item are therefore items of
// the same round of other workgroups, and with every workgroup resident no wait is circular.
template <bool BF16, int BITS, bool ODD, bool BATCH, bool MINMAX = false, Words WORDS = Words::PerWave, bool ONE = false>
__global__ __launch_bounds__(kThreads, kWavesPerSimd) void encode_all_kernel(const EncodeAllArgs a,
                                                                 const FusedWorkerPtrs ptrs,
                                                                 const BatchArgs batch) {
    __shared__ Shared sh;
    using Ctx = EncodeAllCtx<BF16, ODD, BATCH, MINMAX, WORDS, ONE>;
    const uint32_t t = threadIdx.x;
    const uint32_t p0 = blockIdx.x / a.W;
    const uint32_t block = lanes::block_of_lane(t & 63u);
    Ctx c{a, ptrs, batch, sh, {}, {}, t, t & 63u, t >> 6, (MINMAX ? 2u : 1u) * Ctx::kWordsPerWorker * a.W, block,
          (t & ~63u) | block, blockIdx.x - p0 * a.W, gridDim.x / a.W, 0u, Ctx::kNone, 0u, 0u, {}, {}};
    if (p0 >= a.chunks) return;
    // With more than one round of items, the second half of the grid starts about 2.6 us late
    // (6 x 1024 clocks; the halves are cut between chunks, so all workgroups of a chunk lie in
    // the same half and nobody waits longer for a peer).  Measured, 50 buckets of 1600 chunks with a decode launch in between: 4 to 7
    // such units shorten the step by 1.3 to 3 %, 9 and more lengthen it, quarters or eighths
    // of the grid in steps do no better.
    if (!ONE && a.chunks > c.dp && p0 >= (c.dp >> 1))
        for (int i = 0; i < kStaggerSleeps; ++i) __builtin_amdgcn_s_sleep(16);
    c.cur = c.nxt = c.view_of(p0);
    if (Ctx::kDirect) c.load(p0, c.cur);
    c.fill_signs(p0, c.cur, 0u);
    if constexpr (ONE) c.drawn.draw(((uint64_t)p0 << kChunkLog2) + 32u * c.tp, c.w, a.key0, a.key1);   // while the input is on its way
    __syncthreads();
    // the first chunk's input has arrived before the loop is entered, as every later
    // chunk's has by the time its item starts (see the end of the wait in back())
    if (Ctx::kDirect) {
#pragma unroll
        for (int j = 0; j < Ctx::kUnits; ++j)
            asm volatile("" : "+v"(c.raw.u[j].x), "+v"(c.raw.u[j].y), "+v"(c.raw.u[j].z), "+v"(c.raw.u[j].w));
    }
    for (uint64_t p = p0; p < a.chunks; p += c.dp) {
        float v[kRegs];
        c.front(v, p);
        c.template back<BITS>(v, p);
        if (BATCH) c.cur = c.nxt;
        if (ONE) break;
    }
    c.finish();
}

// Copies `count` 32-bit words that arrive as kernel arguments to device memory: how the
// batched calls put their per-bucket records where the kernels can read them, without a
// host-to-device copy (which would need a staging allocation or pinned memory).
struct WordBlob {
    uint32_t w[kBlobWords];
};
__global__ __launch_bounds__(256) void write_words_kernel(uint32_t* dst, const WordBlob blob, uint32_t count) {
    for (uint32_t i = threadIdx.x; i < count; i += 256u) dst[i] = blob.w[i];
}

// Fill with zeros (a kernel, not a memset node, so that callers can capture it in a
// graph).  Words before the first and after the last 16-byte boundary are written one
// by one by the first block; the aligned middle goes out as 16-byte stores.
__global__ __launch_bounds__(256) void zero_words_kernel(uint32_t* dst, uint64_t words) {
    const uint64_t addr = reinterpret_cast<uint64_t>(dst);
    uint64_t head = ((16u - (addr & 15u)) & 15u) / 4u;   // dst is 4-byte aligned
    if (head > words) head = words;
    const uint64_t vecs = (words - head) / 4u;
    const uint64_t tail0 = head + 4u * vecs;
    if (blockIdx.x == 0) {
        if (threadIdx.x < head) dst[threadIdx.x] = 0u;
        if (tail0 + threadIdx.x < words) dst[tail0 + threadIdx.x] = 0u;
    }
    uint4* mid = reinterpret_cast<uint4*>(dst + head);
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < vecs;
         i += (uint64_t)gridDim.x * blockDim.x)
        mid[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ void copy_word_kernel(const uint32_t* src, uint32_t* dst) { *dst = *src; }

// The same number, of which the compiler no longer knows that it is the same for every item of a
// persistent kernel: addresses that follow from it are computed anew instead of being kept in
// registers (some 40 of the decoders' 128, with spills on their account) across the loop.
__device__ __forceinline__ uint32_t this_item(uint32_t x) {
    asm volatile("" : "+v"(x));
    return x;
}

// ------------------------------------------------------------- aggregate_decode
// One chunk per work item, persistent grid.  Thread t owns coordinates 32 t .. 32 t + 31
// (layout L1): 4 * BITS payload bytes (BITS dwords) per worker.
// Called from inside the rotation of the current chunk: the first four worker groups of the workgroup's
// NEXT chunk are loaded, two at a time, and the first two added (8 bits: the first three, one at a time).
template <class Sum>
struct NextChunkLoads {
    static constexpr uint32_t kAdded = 2u;
    Sum& sum;
    uint64_t byte0;
    bool active;
    template <int K>
    __device__ __forceinline__ void at() {
        if (!active) return;
        if constexpr (Sum::kOneAhead) {
            if (K > 0) sum.template add<0>(K - 1);
            sum.template issue<0>(byte0, K);
        } else if (K == 0) {
            sum.begin(byte0);
        } else if ((uint32_t)K - 1u < sum.groups()) {
            sum.template add<(K - 1) & 1>(K - 1);
            sum.template issue<(K - 1) & 1>(byte0, K + 1);
        }
    }
};

// The bucket a decode item belongs to (uniform).  A single-bucket call has one for good; a
// batched call looks it up in the records as its chunks move from bucket to bucket.
struct DecodeView {
    uint64_t n, chunk0;
    uint32_t key0, key1;
    const float* scale;
    float* out;
    ConstU64Ptr pp;      // the bucket's W payload pointers
};

// RANGED: `scale` holds (lo, hi) pairs of the min/max grid instead of the symmetric scale.
// ONCE: how payloads are read (load_payload_words).
template <int BITS, bool BATCH, bool RANGED = false, bool WIDE = false, bool ONCE = BITS != 8>
__global__ __launch_bounds__(kThreads, kWavesPerSimd) void aggregate_decode_kernel(const AggDecodeArgs a,
                                                                       const FusedPayloadPtrs ptrs,
                                                                       const BatchArgs batch) {
    __shared__ Shared sh;
    using Sum = PayloadSum<BITS, BATCH, WIDE, ONCE>;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t block = lay14::block_of_lane(lane), tp = (t & ~63u) | block;   // the thread's 32 coordinates
    const float norm = l4d_negated(lane, wave) ? -kInvSqrtC : kInvSqrtC;
    const float Lf = (float)((1u << BITS) - 1u);
    const float Wf = (float)a.W;
    const uint64_t thread_byte = (uint64_t)tp * (4u * BITS);

    uint32_t bidx = 0u;
    uint64_t boundary = 0u;   // first chunk of the bucket after bidx
    auto view_of = [&](uint64_t p) -> DecodeView {
        if constexpr (BATCH) {
            while (bidx + 1u < batch.count && p >= batch_record(batch, bidx + 1u)->chunk0) ++bidx;
            ConstRecordPtr r = batch_record(batch, bidx);
            boundary = bidx + 1u < batch.count ? batch_record(batch, bidx + 1u)->chunk0 : ~0ull;
            ConstU64Ptr pp = (ConstU64Ptr)(r + 1) + a.W;   // the payload pointers follow the gradient pointers
            DecodeView dv{r->n, r->chunk0, r->key0, r->key1, r->scale, r->out, pp};
            // the record has arrived before the look-up returns (see EncodeAllCtx::view_of)
            asm volatile("" : "+s"(dv.n), "+s"(dv.chunk0), "+s"(dv.key0), "+s"(dv.key1), "+s"(dv.scale),
                         "+s"(dv.out), "+s"(boundary), "+s"(bidx));
            return dv;
        } else {
            return DecodeView{a.n, 0u, a.key0, a.key1, a.scale, a.out, nullptr};
        }
    };

    if (blockIdx.x >= a.chunks) return;
    DecodeView cur = view_of(blockIdx.x);
    Sum sum{ptrs, cur.pp, a.W};
    sum.clear();
    {   // the first chunk's payload, without overlap
        sum.all((((blockIdx.x - cur.chunk0) << kChunkLog2) * BITS) / 8u + thread_byte);
    }
    for (uint64_t p = blockIdx.x; p < a.chunks; p += gridDim.x) {
        const uint64_t pl = p - cur.chunk0;      // the chunk's number inside its bucket
        const uint64_t g0 = pl << kChunkLog2;
        const uint64_t left = cur.n - g0;
        const uint32_t valid = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;
        __syncthreads();   // the previous item's last reads of the buffer and sign table are done
        fill_sign_table<true, false>(sh.sign[0], g0, cur.key0, cur.key1, t);

        // sums -> rotated-domain estimate of the mean, layout L1
        // symmetric grid: yhat = S q - s;  min/max grid: yhat = S q + lo = S q - (-lo)
        const float* scale = global_ptr<const float>(reinterpret_cast<uint64_t>(cur.scale));
        const float s = RANGED ? -scale[2 * pl] : scale[pl];
        const float step = (RANGED ? scale[2 * pl + 1] + s : s + s) / Lf;
        const float qf = step / Wf;
        float v[kRegs];
        uint32_t S[kRegs];
        sum.unpack(S);
#pragma unroll
        for (int r = 0; r < kRegs; ++r) v[r] = (float)S[r] * qf - s;

        if (!BATCH && a.sums) {   // the caller also wants the integer aggregate
            if (BITS == 8 || WIDE) store_sums16(S, static_cast<uint16_t*>(a.sums) + g0 + 32u * tp);
            else store_sums8(S, static_cast<uint8_t*>(a.sums) + g0 + 32u * tp);
        }

        // the next chunk's payload arrives while this one rotates
        const uint64_t pn = p + gridDim.x;
        const bool more = pn < a.chunks;
        DecodeView nxt = cur;
        if (BATCH && more && pn >= boundary) nxt = view_of(pn);   // rarely: a new bucket
        sum.pp = nxt.pp;
        NextChunkLoads<Sum> next{sum, (((pn - nxt.chunk0) << kChunkLog2) * BITS) / 8u + thread_byte, more};
        sum.clear();
        const uint32_t ti = this_item(t), li = ti & 63u;
        rotate_lanes_to_l4d(sh, v, li, block, wave, next);   // (its barrier also orders the sign table)
        // Many groups and 8 bits: in front of the stores, behind which their loads would queue (4 bits, 64 workers x
        // 16.8 M coordinates 116.5 -> 109.1 us, on one of three devices 108.8 -> 108.9; 32 x 16.8 M 62.0 -> 61.0).
        // Otherwise behind them: in front they take the registers that let the stores' addresses overlap
        // (8 workers x 67 M, 4 bits 98 us, in front 105).
        constexpr bool kFront = WIDE || Sum::kOneAhead;
        if (kFront && more) {
            if constexpr (Sum::kOneAhead) sum.rest_one_ahead(next.byte0, next.kAdded);
            else sum.rest(next.byte0, next.kAdded);
        }
        store_signed_l4d(sh.sign[0], v, global_ptr<float>(reinterpret_cast<uint64_t>(cur.out)) + g0, valid,
                         kFront ? this_item(ti) : ti, norm);
        if (!kFront && more) sum.rest(next.byte0, next.kAdded);   // (its first loads were issued in front of the stores: no wait for them)
        cur = nxt;
    }
}

// The same for a launch of at most one chunk per workgroup: one chunk's chain.  There is no next chunk to keep registers
// for, so the payloads are summed without a condition inside the loop (all_alone), and the scale is read in front of
// them.  A pass with the encoder, 4 bits, us, kernel above -> this: 2 workers x 50257 13.4 -> 12.1, 8 x 50257 14.3 -> 13.4,
// 8 x 2^19 14.9 -> 14.0, 8 x 2^21 25.1 -> 24.2, 16 x 50257 15.7 -> 14.0, 64 x 50257 26.5 -> 22.0, 64 x 2^21 132.5 -> 129.5;
// 8 bits, 8 x 2^20 23.2 -> 22.0, 64 x 2^20 92.6 -> 85.5; 2 bits, 64 x 2^18 34.9 -> 28.5.  (All payloads of 8 or 16 workers in
// flight, with the sign table computed meanwhile, was 2 % slower; only the sign table, no difference.)
template <int BITS, bool RANGED, bool WIDE, bool ONCE>
__global__ __launch_bounds__(kThreads, kWavesPerSimd) void aggregate_decode_one_kernel(const AggDecodeArgs a,
                                                                           const FusedPayloadPtrs ptrs) {
    __shared__ Shared sh;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t block = lay14::block_of_lane(lane), tp = (t & ~63u) | block;   // the thread's 32 coordinates
    const uint64_t p = blockIdx.x, g0 = p << kChunkLog2, left = a.n - g0;
    const uint32_t valid = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;
    const float s = RANGED ? -a.scale[2 * p] : a.scale[p];
    const float step = (RANGED ? a.scale[2 * p + 1] + s : s + s) / (float)((1u << BITS) - 1u);
    const float qf = step / (float)a.W;
    PayloadSum<BITS, false, WIDE, ONCE> sum{ptrs, nullptr, a.W};
    sum.clear();
    sum.all_alone((g0 * BITS) / 8u + tp * (4u * BITS));
    fill_sign_table<true, false>(sh.sign[0], g0, a.key0, a.key1, t);
    float v[kRegs];
    uint32_t S[kRegs];
    sum.unpack(S);
#pragma unroll
    for (int r = 0; r < kRegs; ++r) v[r] = (float)S[r] * qf - s;
    if (a.sums) {
        if (BITS == 8 || WIDE) store_sums16(S, static_cast<uint16_t*>(a.sums) + g0 + 32u * tp);
        else store_sums8(S, static_cast<uint8_t*>(a.sums) + g0 + 32u * tp);
    }
    NoHook none;
    rotate_lanes_to_l4d(sh, v, lane, block, wave, none);   // (its barrier also orders the sign table)
    store_signed_l4d(sh.sign[0], v, a.out + g0, valid, t, l4d_negated(lane, wave) ? -kInvSqrtC : kInvSqrtC);
}

// ------------------------------------------------- saturating aggregate + decode
// Same shape as aggregate_decode_kernel, but the W payloads are combined coordinate by
// coordinate with Sat in worker order (a <- clamp(a + z_w, -M, M), z = idx - M, starting
// from a = 0, which leaves a = z_0 after the first worker), so the running value never
// needs more than BITS bits.  Optionally stores the packed aggregate (a + M) and counts
// the coordinates with at least one clipped step.
// Called from inside the rotation of the current chunk: loads the first two worker groups (8 bits: the
// first) of the workgroup's next chunk.
template <class Loads>
struct NextSatLoads {
    Loads& loads;
    uint64_t byte0;
    bool active;
    template <int K>
    __device__ __forceinline__ void at() {
        if (K == 0 && active) loads.begin_ahead(byte0);
    }
};

// Saturating sums of the thread's 32 coordinates, a <- clamp(a + z, -M, M) with z = idx - M, worker after worker.
// 2 and 4 bits: bit by bit.  A worker's payload words are transposed into planes (plane b holds bit b of all 32
// coordinates, BITS log2(BITS) swaps of halves), and a runs in planes of its two's complement: z = (idx - 2^(BITS-1)) + 1,
// the index with its top bit flipped and a carry in; a sum beyond the BITS bits shows in the signs, and the one value
// below -M that fits them becomes -M.  31 operations for a worker's 32 coordinates at 4 bits, 9 at 2, where
// extract, add and clamp took 96.
// A pass with the encoder, us, before -> this: 8 workers x 15.5 M 4 bits 121.8 -> 116.6, 2 bits 120.5 -> 112.0; x 2^19
// 17.0 -> 14.9 and 16.9 -> 14.3; x 2^16 15.6 -> 13.4; 2 workers the same.
// 8 bits: two coordinates to an operation, t = a + M >= 0 in 16-bit halves, min(t + idx, 3 M) and a saturating
// subtraction of M: x 2^19 17.8 -> 17.3, 2 workers x 2^20 13.5 -> 13.6.
template <int BITS, bool COUNT>
struct SatSum {
    static_assert(BITS == 2 || BITS == 4, "planes");
    uint32_t a[BITS];
    uint32_t clip;   // COUNT: coordinates with a clipped step
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int b = 0; b < BITS; ++b) a[b] = 0u;
        clip = 0u;
    }
    // Words of nibbles (pairs of bits) <-> planes: bit b of field k of word j is bit BITS k + j of plane b.
    static __device__ __forceinline__ void swap_fields(uint32_t& x, uint32_t& y, uint32_t low, int shift) {
        const uint32_t u = (x & low) | ((y << shift) & ~low);
        y = ((x >> shift) & low) | (y & ~low);
        x = u;
    }
    static __device__ __forceinline__ void transpose(uint32_t (&w)[BITS]) {
        if constexpr (BITS == 4) {
            swap_fields(w[0], w[2], 0x33333333u, 2);
            swap_fields(w[1], w[3], 0x33333333u, 2);
            swap_fields(w[0], w[1], 0x55555555u, 1);
            swap_fields(w[2], w[3], 0x55555555u, 1);
        } else {
            swap_fields(w[0], w[1], 0x55555555u, 1);
        }
    }
    static __device__ __forceinline__ uint32_t majority(uint32_t x, uint32_t y, uint32_t z) {
        return __builtin_amdgcn_bitop3_b32(x, y, z, 0xE8);
    }
    __device__ __forceinline__ void add(const PayloadWords<BITS>& payload) {
        uint32_t i[BITS];
#pragma unroll
        for (int b = 0; b < BITS; ++b) i[b] = payload.w[b];
        transpose(i);
        const uint32_t s0 = ~(a[0] ^ i[0]), c0 = a[0] | i[0];
        if constexpr (BITS == 4) {
            const uint32_t s1 = xor3(a[1], i[1], c0), c1 = majority(a[1], i[1], c0);
            const uint32_t s2 = xor3(a[2], i[2], c1), c2 = majority(a[2], i[2], c1);
            const uint32_t s3 = ~xor3(a[3], i[3], c2);
            const uint32_t over = ~a[3] & i[3] & s3, under = a[3] & ~i[3] & ~s3;   // > 7, < -8
            const uint32_t low = s3 & ~s2 & ~s1;                                   // -8 or -7 (or over)
            if (COUNT) clip |= over | under | (low & ~s0);
            a[0] = (s0 | over | under) | low;
            a[1] = (s1 & ~under) | over;
            a[2] = (s2 & ~under) | over;
            a[3] = (s3 & ~over) | under;
        } else {
            const uint32_t s1 = ~xor3(a[1], i[1], c0);
            const uint32_t over = ~a[1] & i[1] & s1;                               // > 1; -2 is the lowest sum
            if (COUNT) clip |= over | (s1 & ~s0);
            a[0] = s0 | s1;
            a[1] = s1 & ~over;
        }
    }
    // a + M, packed like a payload.
    __device__ __forceinline__ void pack(uint32_t (&pk)[BITS]) const {
        // (a + 2^(BITS-1)) - 1: the top bit flipped, then a borrow
        pk[0] = ~a[0];
        if constexpr (BITS == 4) {
            const uint32_t b1 = ~a[1] & pk[0], b2 = ~a[2] & b1;
            pk[1] = a[1] ^ pk[0];
            pk[2] = a[2] ^ b1;
            pk[3] = ~a[3] ^ b2;
        } else {
            pk[1] = ~a[1] ^ pk[0];
        }
        transpose(pk);
    }
    __device__ __forceinline__ uint32_t clipped() const { return (uint32_t)__popc(clip); }
};
template <bool COUNT>
struct SatSum<8, COUNT> {
    typedef uint16_t Pair __attribute__((ext_vector_type(2)));
    static constexpr uint16_t M = 127;
    Pair t[16];   // a + M, 0 .. 2 M: of coordinates 4 d, 4 d + 2 in t[2 d], of 4 d + 1, 4 d + 3 in t[2 d + 1]
    uint32_t clip[COUNT ? 16 : 1];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            t[k] = Pair{M, M};
            if (COUNT) clip[k] = 0u;
        }
    }
    __device__ __forceinline__ void add(const PayloadWords<8>& payload) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t w = payload.w[k >> 1];
            const Pair idx = __builtin_bit_cast(Pair, (k & 1) ? __builtin_amdgcn_perm(0u, w, 0x0C030C01u) : w & 0x00FF00FFu);
            const Pair raw = t[k] + idx;
            t[k] = __builtin_elementwise_sub_sat(__builtin_elementwise_min(raw, Pair{3 * M, 3 * M}), Pair{M, M});
            if (COUNT) clip[k] |= __builtin_bit_cast(uint32_t, raw) ^ __builtin_bit_cast(uint32_t, (Pair)(t[k] + Pair{M, M}));
        }
    }
    __device__ __forceinline__ void pack(uint32_t (&pk)[8]) const {
#pragma unroll
        for (int d = 0; d < 8; ++d)
            pk[d] = __builtin_bit_cast(uint32_t, t[2 * d]) | (__builtin_bit_cast(uint32_t, t[2 * d + 1]) << 8);
    }
    // a of all coordinates
    __device__ __forceinline__ void values(float (&v)[kRegs]) const {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t a = __builtin_bit_cast(uint32_t, (Pair)(t[k] - Pair{M, M}));
            const int r = 4 * (k >> 1) + (k & 1);
            asm("v_cvt_f32_i32_sdwa %0, sext(%1) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0" : "=v"(v[r]) : "v"(a));
            asm("v_cvt_f32_i32_sdwa %0, sext(%1) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1" : "=v"(v[r + 2]) : "v"(a));
        }
    }
    __device__ __forceinline__ uint32_t clipped() const {
        uint32_t count = 0u;
        if constexpr (COUNT) {
#pragma unroll
            for (int k = 0; k < 16; ++k) count += ((clip[k] & 0xFFFFu) != 0u ? 1u : 0u) + ((clip[k] >> 16) != 0u ? 1u : 0u);
        }
        return count;
    }
};

template <int BITS, bool COUNT, bool ONCE = BITS != 8>
__global__ __launch_bounds__(kThreads, kWavesPerSimd) void sat_aggregate_decode_kernel(
    const SatAggDecodeArgs a, const FusedPayloadPtrs ptrs) {
    __shared__ Shared sh;
    constexpr int M = (1 << (BITS - 1)) - 1;
    constexpr int kGroup = BITS == 8 ? 2 : 4;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t block = lay14::block_of_lane(lane), tp = (t & ~63u) | block;   // the thread's 32 coordinates
    const float norm = l4d_negated(lane, wave) ? -kInvSqrtC : kInvSqrtC;
    const float Lf = (float)(2 * M);
    const float Wf = (float)a.W;
    uint32_t clipped_total = 0u;
    const uint64_t thread_byte = (uint64_t)tp * (4u * BITS);

    using Loads = PayloadLoads<BITS, false, kGroup, ONCE>;
    Loads loads{ptrs, nullptr, a.W, {}};
    if (blockIdx.x < a.chunks) loads.begin_ahead((((uint64_t)blockIdx.x << kChunkLog2) * BITS) / 8u + thread_byte);
    for (uint64_t p = blockIdx.x; p < a.chunks; p += gridDim.x) {
        const uint64_t g0 = p << kChunkLog2;
        const uint64_t left = a.n - g0;
        const uint32_t valid = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;
        __syncthreads();   // the previous item's last reads of the buffer and sign table are done
        fill_sign_table<true, false>(sh.sign[0], g0, a.key0, a.key1, t);

        SatSum<BITS, COUNT> sum;
        sum.clear();
        const uint64_t byte0 = (g0 * BITS) / 8u + thread_byte;
        auto combine = [&](const PayloadWords<BITS>(&x)[kGroup], uint32_t w0) {
#pragma unroll
            for (int j = 0; j < kGroup; ++j)
                if (w0 + j < a.W) sum.add(x[j]);
        };
        if constexpr (Loads::kOneAhead) {
            for (uint32_t g = 0; g < loads.groups(); ++g) {
                if (g != 0u) loads.template issue<0>(byte0, g);
                combine(loads.x[0], g * kGroup);
            }
        } else {
            for (uint32_t g = 0; g < loads.groups(); g += 2u) {
                combine(loads.x[0], g * kGroup);
                loads.template issue<0>(byte0, g + 2u);
                if (g + 1u < loads.groups()) combine(loads.x[1], (g + 1u) * kGroup);
                loads.template issue<1>(byte0, g + 3u);
            }
        }
        if (COUNT) clipped_total += sum.clipped();
        uint32_t index[BITS];   // 2 and 4 bits: a + M, packed
        if constexpr (BITS != 8) sum.pack(index);
        if (a.aggregate) {
            uint32_t pk[BITS];
            if constexpr (BITS == 8) sum.pack(pk);
            store_packed<BITS>(BITS == 8 ? pk : index, a.aggregate + byte0);
        }

        // aggregate -> rotated-domain estimate of the mean, layout L1
        const float s = a.scale[p];
        const float step = (s + s) / Lf;
        const float qf = step / Wf;
        float v[kRegs];
        if constexpr (BITS == 8) sum.values(v);
#pragma unroll
        for (int r = 0; r < kRegs; ++r) {
            if constexpr (BITS != 8) {
                const uint32_t field = (index[r * BITS >> 5] >> (r * BITS & 31)) & ((1u << BITS) - 1u);
                v[r] = (float)field - (float)M;
            }
            v[r] = v[r] * qf;   // (v[r] is a whole number: one rounding)
        }
        // the next chunk's first payloads arrive while this one rotates
        const uint64_t pn = p + gridDim.x;
        NextSatLoads<Loads> next{loads, ((pn << kChunkLog2) * BITS) / 8u + thread_byte, pn < a.chunks};
        const uint32_t ti = this_item(t), li = ti & 63u;
        rotate_lanes_to_l4d(sh, v, li, block, wave, next);   // (its barrier also orders the sign table)
        store_signed_l4d(sh.sign[0], v, a.out + g0, valid, ti, norm);
    }
    if (COUNT) {   // one atomic per wave
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) clipped_total += __shfl_xor(clipped_total, off, 64);
        if (lane == 0 && clipped_total != 0u) atomicAdd(a.overflow, (unsigned long long)clipped_total);
    }
}

// ------------------------------------------------------------------ aggregate only
// Streaming sum of W payloads: each thread owns 16 payload bytes per worker.
template <int BITS, typename SumT>
__global__ __launch_bounds__(256) void aggregate_fast_kernel(const FusedPayloadPtrs ptrs, uint32_t W,
                                                             uint64_t vecs, SumT* sums) {
    constexpr bool kWide = BITS != 8 && sizeof(SumT) == 2;   // 16-bit lanes for 2- and 4-bit payloads
    constexpr int kLanes = BITS == 8 ? 2 : (kWide ? 16 : 8) / BITS;
    constexpr uint32_t kMask = BITS == 8 ? 0x00FF00FFu
                               : kWide   ? (BITS == 4 ? 0x000F000Fu : 0x00030003u)
                                         : (BITS == 4 ? 0x0F0F0F0Fu : 0x03030303u);
    constexpr int kCoords = 128 / BITS;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < vecs;
         i += (uint64_t)gridDim.x * blockDim.x) {
        uint32_t acc[4][kLanes];
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int q = 0; q < kLanes; ++q) acc[d][q] = 0u;
        for (uint32_t w0 = 0; w0 < W; w0 += 8) {
            uint4 x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (w0 + j < W) x[j] = reinterpret_cast<const uint4*>(ptrs.p[w0 + j])[i];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (w0 + j < W) {
                    const uint32_t ww[4] = {x[j].x, x[j].y, x[j].z, x[j].w};
#pragma unroll
                    for (int d = 0; d < 4; ++d)
#pragma unroll
                        for (int q = 0; q < kLanes; ++q) acc[d][q] += (ww[d] >> (BITS * q)) & kMask;
                }
        }
        SumT* dst = sums + i * kCoords;
        if constexpr (kWide) {   // lane q = coordinates q (low half) and q + kLanes (high half) of the dword
            constexpr int per = 32 / BITS;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t o[per / 2];   // pairs of consecutive coordinates
#pragma unroll
                for (int c = 0; c < per; c += 2) {
                    const uint32_t lo = c < kLanes ? (acc[d][c] & 0xFFFFu) : (acc[d][c - kLanes] >> 16);
                    const uint32_t hi = c + 1 < kLanes ? (acc[d][c + 1] & 0xFFFFu) : (acc[d][c + 1 - kLanes] >> 16);
                    o[c / 2] = lo | (hi << 16);
                }
#pragma unroll
                for (int k = 0; k < per / 8; ++k)
                    reinterpret_cast<uint4*>(dst + per * d)[k] = make_uint4(o[4 * k], o[4 * k + 1], o[4 * k + 2], o[4 * k + 3]);
            }
        } else if (BITS == 8) {   // u16 sums: (even, odd) pairs
            uint32_t o[8];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                o[2 * d] = __builtin_amdgcn_perm(acc[d][1], acc[d][0], 0x05040100u);
                o[2 * d + 1] = __builtin_amdgcn_perm(acc[d][1], acc[d][0], 0x07060302u);
            }
            reinterpret_cast<uint4*>(dst)[0] = make_uint4(o[0], o[1], o[2], o[3]);
            reinterpret_cast<uint4*>(dst)[1] = make_uint4(o[4], o[5], o[6], o[7]);
        } else if (BITS == 4) {   // u8 sums: lane 0 = even coordinates, lane 1 = odd
            uint32_t o[8];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                o[2 * d] = __builtin_amdgcn_perm(acc[d][1], acc[d][0], 0x05010400u);
                o[2 * d + 1] = __builtin_amdgcn_perm(acc[d][1], acc[d][0], 0x07030602u);
            }
            reinterpret_cast<uint4*>(dst)[0] = make_uint4(o[0], o[1], o[2], o[3]);
            reinterpret_cast<uint4*>(dst)[1] = make_uint4(o[4], o[5], o[6], o[7]);
        } else {                  // 2 bits: lane q byte b = coordinate 4 b + q of the dword's 16
            uint32_t o[16];
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    uint32_t v = 0u;
#pragma unroll
                    for (int q = 0; q < 4; ++q) v |= ((acc[d][q] >> (8 * b)) & 0xFFu) << (8 * q);
                    o[4 * d + b] = v;
                }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                reinterpret_cast<uint4*>(dst)[k] = make_uint4(o[4 * k], o[4 * k + 1], o[4 * k + 2], o[4 * k + 3]);
        }
    }
}

// Workgroups of `kernel` that are resident at once on the whole device.
template <auto kernel>
uint32_t resident_grid() {
    return thc::resident_grid<kernel>(kThreads);
}

// More than 32 workers, dp chunks per round: one reader per workgroup, except for short items (bf16, up to 4 bits) in five to seven
// rounds of an even number of chunks, where the late half of the grid is the other workgroup of every CU, so
// that the two are half an item apart anyway and one wave's hand-over only adds to the item.  4 bits, every wave |
// one reader, us: 64 workers x 40 chunks 37.3 | 40.6, x 56 52.6 | 53.3, x 64 61.8 | 60.0; 48 x 60 42.2 | 46.1, 40 x 72 42.7 | 46.5;
// an odd number of chunks, 56 x 45 42.2 | 41.0, 44 x 66 48.6 | 46.9, 33 x 90 48.3 | 46.3; bf16 8 bits, 64 x 48 56.0 | 50.9.
inline bool one_reader(const EncodeAllArgs& a, uint64_t dp, bool short_item) {
    return !(short_item && (dp & 1u) == 0u && a.chunks > kFewRounds * dp && a.chunks < kLateRound * dp);
}

// Grid of an encoder, whose workgroups wait for one another and have to be resident all at once: what the device keeps of
// the very kernel that is launched (its forms differ in registers), and, as every workgroup keeps one worker, a whole
// number of chunks per round.  0: not even the workgroups of one chunk.
template <auto kernel>
uint32_t agreeing_grid(const EncodeAllArgs& a) {
    const uint64_t total = a.chunks * a.W;
    uint64_t G = resident_grid<kernel>();
    if (G > total) G = total;
    return (uint32_t)(G - G % a.W);
}
template <auto kernel>
hipError_t launch_agreeing(EncodeAllArgs a, const FusedWorkerPtrs& ptrs, const BatchArgs& batch, hipStream_t stream) {
    const uint32_t G = agreeing_grid<kernel>(a);
    if (G == 0) return hipErrorInvalidConfiguration;
    a.crowded = 4ull * G > 3ull * resident_grid<kernel>();
    hipLaunchKernelGGL(kernel, dim3(G), dim3(kThreads), 0, stream, a, ptrs, batch);
    return hipGetLastError();
}
// The form of one item per workgroup where that is a launch of it, the persistent one otherwise.
template <bool BF16, int BITS, bool ODD, bool MINMAX, Words WORDS>
hipError_t launch_one_or_persistent(const EncodeAllArgs& a, const FusedWorkerPtrs& ptrs, hipStream_t stream) {
    constexpr auto one = encode_all_kernel<BF16, BITS, ODD, false, MINMAX, WORDS, true>;
    if (agreeing_grid<one>(a) == a.chunks * a.W) return launch_agreeing<one>(a, ptrs, BatchArgs{}, stream);
    return launch_agreeing<encode_all_kernel<BF16, BITS, ODD, false, MINMAX, WORDS>>(a, ptrs, BatchArgs{}, stream);
}

template <bool BF16, int BITS, bool ODD, bool BATCH>
hipError_t launch_encode_all_t(const EncodeAllArgs& a, const FusedWorkerPtrs& ptrs, const BatchArgs& batch,
                               hipStream_t stream) {
    if constexpr (BATCH) {
        return launch_agreeing<encode_all_kernel<BF16, BITS, ODD, true>>(a, ptrs, batch, stream);
    } else {
        if (a.W > kPerGroupMaxWorkers) {
            const uint64_t dp = agreeing_grid<encode_all_kernel<BF16, BITS, ODD, false, false, Words::OneReader>>(a) / a.W;
            if (one_reader(a, dp, BF16 && BITS <= 4))
                return launch_one_or_persistent<BF16, BITS, ODD, false, Words::OneReader>(a, ptrs, stream);
        }
        if (a.W > kPerWaveMaxWorkers)
            return launch_one_or_persistent<BF16, BITS, ODD, false, Words::PerGroup>(a, ptrs, stream);
        return launch_one_or_persistent<BF16, BITS, ODD, false, Words::PerWave>(a, ptrs, stream);
    }
}

template <bool BATCH>
hipError_t launch_encode_all_pick(const EncodeAllArgs& a, const FusedWorkerPtrs& ptrs, const BatchArgs& batch,
                                  bool bf16, bool odd, uint32_t bits, hipStream_t stream) {
    if (bf16 && odd) {   // an odd count of bf16 somewhere: the last coordinate comes by itself
        if (bits == 2) return launch_encode_all_t<true, 2, true, BATCH>(a, ptrs, batch, stream);
        if (bits == 4) return launch_encode_all_t<true, 4, true, BATCH>(a, ptrs, batch, stream);
        return launch_encode_all_t<true, 8, true, BATCH>(a, ptrs, batch, stream);
    }
    if (bf16) {
        if (bits == 2) return launch_encode_all_t<true, 2, false, BATCH>(a, ptrs, batch, stream);
        if (bits == 4) return launch_encode_all_t<true, 4, false, BATCH>(a, ptrs, batch, stream);
        return launch_encode_all_t<true, 8, false, BATCH>(a, ptrs, batch, stream);
    }
    if (bits == 2) return launch_encode_all_t<false, 2, false, BATCH>(a, ptrs, batch, stream);
    if (bits == 4) return launch_encode_all_t<false, 4, false, BATCH>(a, ptrs, batch, stream);
    return launch_encode_all_t<false, 8, false, BATCH>(a, ptrs, batch, stream);
}

template <int BITS, bool BATCH, bool RANGED, bool WIDE, bool ONCE = BITS != 8>
hipError_t launch_aggregate_decode_t(const AggDecodeArgs& a, const FusedPayloadPtrs& ptrs, const BatchArgs& batch,
                                        hipStream_t stream) {
    uint32_t G = resident_grid<aggregate_decode_kernel<BITS, BATCH, RANGED, WIDE, ONCE>>();
    if (G == 0) return hipErrorInvalidValue;
    if constexpr (!BATCH) {   // every chunk has a workgroup of its own (one round)
        if (a.chunks <= G) {
            hipLaunchKernelGGL((aggregate_decode_one_kernel<BITS, RANGED, WIDE, ONCE>), dim3((uint32_t)a.chunks),
                               dim3(kThreads), 0, stream, a, ptrs);
            return hipGetLastError();
        }
    }
    if (G > a.chunks) G = (uint32_t)a.chunks;
    hipLaunchKernelGGL((aggregate_decode_kernel<BITS, BATCH, RANGED, WIDE, ONCE>), dim3(G), dim3(kThreads), 0, stream,
                       a, ptrs, batch);
    return hipGetLastError();
}
// 4-bit payloads of so many workers that the sums need 16 bits.
// (2-bit payloads would need more than 85 workers, beyond what the one-launch forms take)
__host__ inline bool wide_sums(uint32_t W, uint32_t bits) { return bits == 4u && W * 15u > 255u; }

template <bool BATCH, bool RANGED>
hipError_t launch_aggregate_decode_pick(const AggDecodeArgs& a, const FusedPayloadPtrs& ptrs, const BatchArgs& batch,
                                        uint32_t bits, hipStream_t stream) {
    if (a.chunks == 0) return hipSuccess;
    if (wide_sums(a.W, bits)) return launch_aggregate_decode_t<4, BATCH, RANGED, true>(a, ptrs, batch, stream);
    if (bits == 2) return launch_aggregate_decode_t<2, BATCH, RANGED, false>(a, ptrs, batch, stream);
    if (bits == 4) return launch_aggregate_decode_t<4, BATCH, RANGED, false>(a, ptrs, batch, stream);
    if (stream_payloads(a.W, a.chunks << kChunkLog2)) return launch_aggregate_decode_t<8, BATCH, RANGED, false, true>(a, ptrs, batch, stream);
    return launch_aggregate_decode_t<8, BATCH, RANGED, false, false>(a, ptrs, batch, stream);
}

}  // namespace
}  // namespace k14

uint32_t encode_all_slot_words(uint32_t W) { return k14::kWaves * W; }

// Workgroups of the one-pass encoder that the device keeps resident at once.
static uint32_t encode_all_resident(bool bf16, uint32_t bits) {
    using namespace k14;
    if (bf16) return bits == 2 ? resident_grid<encode_all_kernel<true, 2, false, false>>()
                   : bits == 4 ? resident_grid<encode_all_kernel<true, 4, false, false>>()
                               : resident_grid<encode_all_kernel<true, 8, false, false>>();
    return bits == 2 ? resident_grid<encode_all_kernel<false, 2, false, false>>()
         : bits == 4 ? resident_grid<encode_all_kernel<false, 4, false, false>>()
                     : resident_grid<encode_all_kernel<false, 8, false, false>>();
}

bool encode_all_fused_applicable(const EncodeAllArgs& a, const FusedWorkerPtrs& ptrs, uint32_t chunk_log2,
                                 bool bf16, uint32_t bits) {
    if (chunk_log2 != 14 || a.W > (uint32_t)kMaxFusedWorkers) return false;
    if (a.chunks * a.W >= 0x7FFFFFFFull) return false;
    // the W workgroups of a chunk wait for one another: all of them must be resident
    if (encode_all_resident(bf16, bits) < a.W) return false;
    for (uint32_t w = 0; w < a.W; ++w)
        if ((reinterpret_cast<uintptr_t>(ptrs.grad[w]) & 15u) || (reinterpret_cast<uintptr_t>(ptrs.payload[w]) & 15u))
            return false;
    return true;
}

hipError_t launch_zero_words(uint32_t* dst, uint64_t words, hipStream_t stream) {
    if (words == 0) return hipSuccess;
    const uint64_t blocks = (words / 4u + 255u) / 256u;
    hipLaunchKernelGGL(k14::zero_words_kernel, dim3((uint32_t)(blocks < 1u ? 1u : (blocks > 8192u ? 8192u : blocks))),
                       dim3(256), 0, stream, dst, words);
    return hipGetLastError();
}

hipError_t launch_copy_word(const uint32_t* src, uint32_t* dst, hipStream_t stream) {
    hipLaunchKernelGGL(k14::copy_word_kernel, dim3(1), dim3(1), 0, stream, src, dst);
    return hipGetLastError();
}

hipError_t launch_encode_all_fused(const EncodeAllArgs& a, const FusedWorkerPtrs& ptrs, bool bf16,
                                   uint32_t bits, hipStream_t stream) {
    return k14::launch_encode_all_pick<false>(a, ptrs, BatchArgs{}, bf16, (a.n & 1u) != 0u, bits, stream);
}

// The min/max grid through the same kernel: a.scale receives (lo, hi) pairs and a.slots has
// twice the words per chunk.  Launches of one round take the form without a next item here too (with the decoder and the
// clearing launch, us: 8 workers x 100000 16.7 -> 14.8, 8 x 2^20 23.7 -> 22.3, 16 x 0.5 M fp32 30.2 -> 26.0, 32 x 2^18 33.8 -> 30.9).
// Its pauses, 8 | 24, with the decoder: 8 workers x 40 chunks bf16 19.8 | 19.4, fp32 19.6 | 20.5, x 50 21.2 | 20.0, 20.7 | 20.9, x 64 23.0 | 20.4,
// 23.9 | 21.8; 16 x 24 fp32 24.0 | 25.0, x 28 25.5 | 26.2, x 32 29.5 | 26.3: the line of the symmetric grid serves.  (By itself, with no
// decoder between, the fp32 encoder of a full launch takes 16.7 us with the longer pause and 14.5 with the shorter one, 8 x 64.)
hipError_t launch_encode_all_ranged(const EncodeAllArgs& a, const FusedWorkerPtrs& ptrs, bool bf16,
                                    uint32_t bits, hipStream_t stream) {
    using namespace k14;
    const bool odd = (a.n & 1u) != 0u;
#define THC_RANGED(BF, B, O) return launch_one_or_persistent<BF, B, O, true, Words::PerWave>(a, ptrs, stream)
    if (a.chunks == 0) return hipSuccess;
    if (bf16 && odd) {
        if (bits == 2) THC_RANGED(true, 2, true);
        if (bits == 4) THC_RANGED(true, 4, true);
        THC_RANGED(true, 8, true);
    }
    if (bf16) {
        if (bits == 2) THC_RANGED(true, 2, false);
        if (bits == 4) THC_RANGED(true, 4, false);
        THC_RANGED(true, 8, false);
    }
    if (bits == 2) THC_RANGED(false, 2, false);
    if (bits == 4) THC_RANGED(false, 4, false);
    THC_RANGED(false, 8, false);
#undef THC_RANGED
}

hipError_t launch_encode_all_batch(const EncodeAllArgs& a, const BatchArgs& batch, bool bf16, bool any_odd,
                                   uint32_t bits, hipStream_t stream) {
    return k14::launch_encode_all_pick<true>(a, FusedWorkerPtrs{}, batch, bf16, any_odd, bits, stream);
}

hipError_t launch_write_words(uint32_t* dst, const uint32_t* host_words, uint32_t count, hipStream_t stream) {
    // the words travel as kernel arguments, kBlobWords at a time
    for (uint32_t done = 0; done < count; done += (uint32_t)kBlobWords) {
        k14::WordBlob blob;
        const uint32_t now = count - done < (uint32_t)kBlobWords ? count - done : (uint32_t)kBlobWords;
        for (uint32_t i = 0; i < now; ++i) blob.w[i] = host_words[done + i];
        hipLaunchKernelGGL(k14::write_words_kernel, dim3(1), dim3(256), 0, stream, dst + done, blob, now);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

bool aggregate_decode_fused_applicable(uint32_t W, uint32_t chunk_log2, uint32_t bits) {
    if (chunk_log2 != 14 || W > (uint32_t)kMaxFusedPayloads) return false;
    // packed accumulators: 8-bit lanes for 2- and 4-bit payloads, 16-bit lanes for 8-bit.
    // The kernel stores the sums at the width of its lanes, so the shape qualifies only
    // when that is also the width the caller's buffer has (one worker of 8-bit payloads
    // has one-byte sums and takes the unfused path).
    static_assert(kMaxFusedPayloads * 3 <= 255, "2-bit payloads have narrow lanes only");
    const uint32_t top = W * ((1u << bits) - 1u);
    return bits == 8 ? (top > 255u && top <= 65535u) : top <= 65535u;
}

hipError_t launch_aggregate_decode_fused(const AggDecodeArgs& a, const FusedPayloadPtrs& ptrs,
                                         uint32_t bits, hipStream_t stream) {
    return k14::launch_aggregate_decode_pick<false, false>(a, ptrs, BatchArgs{}, bits, stream);
}

// a.scale holds (lo, hi) pairs.
hipError_t launch_aggregate_decode_ranged(const AggDecodeArgs& a, const FusedPayloadPtrs& ptrs,
                                          uint32_t bits, hipStream_t stream) {
    return k14::launch_aggregate_decode_pick<false, true>(a, ptrs, BatchArgs{}, bits, stream);
}

hipError_t launch_aggregate_decode_batch(const AggDecodeArgs& a, const BatchArgs& batch, uint32_t bits,
                                         hipStream_t stream) {
    return k14::launch_aggregate_decode_pick<true, false>(a, FusedPayloadPtrs{}, batch, bits, stream);
}

bool sat_aggregate_decode_fused_applicable(uint32_t W, uint32_t chunk_log2) {
    return chunk_log2 == 14 && W <= (uint32_t)kMaxFusedPayloads;
}

hipError_t launch_sat_aggregate_decode_fused(const SatAggDecodeArgs& a, const FusedPayloadPtrs& ptrs,
                                             uint32_t bits, hipStream_t stream) {
    using namespace k14;
    if (a.chunks == 0) return hipSuccess;
    uint32_t G = 0;
#define THC_SATDEC(...)                                                                            \
    do {                                                                                          \
        G = resident_grid<sat_aggregate_decode_kernel<__VA_ARGS__>>();                            \
        if (G == 0) return hipErrorInvalidValue;                                                  \
        if ((uint64_t)G > a.chunks) G = (uint32_t)a.chunks;                                       \
        hipLaunchKernelGGL((sat_aggregate_decode_kernel<__VA_ARGS__>), dim3(G), dim3(kThreads), 0, stream, \
                           a, ptrs);                                                              \
    } while (0)
    const bool once = bits == 8 && stream_payloads(a.W, a.chunks << kChunkLog2);
    if (a.overflow) {
        if (bits == 2) THC_SATDEC(2, true);
        else if (bits == 4) THC_SATDEC(4, true);
        else if (once) THC_SATDEC(8, true, true);
        else THC_SATDEC(8, true);
    } else {
        if (bits == 2) THC_SATDEC(2, false);
        else if (bits == 4) THC_SATDEC(4, false);
        else if (once) THC_SATDEC(8, false, true);
        else THC_SATDEC(8, false);
    }
#undef THC_SATDEC
    return hipGetLastError();
}

bool aggregate_fast_applicable(uint32_t W, uint32_t bits, uint32_t sum_bytes, uint64_t payload_bytes) {
    if (W > (uint32_t)kMaxFusedPayloads || (payload_bytes & 15u)) return false;
    return (bits != 2 && sum_bytes == 2) || (bits != 8 && sum_bytes == 1);
}

hipError_t launch_aggregate_fast(const FusedPayloadPtrs& ptrs, uint32_t W, uint32_t bits,
                                 uint64_t payload_bytes, void* sums, hipStream_t stream) {
    using namespace k14;
    const uint64_t vecs = payload_bytes / 16u;
    if (vecs == 0) return hipSuccess;
    const int cus = device_cus();
    uint64_t blocks = (vecs + 255u) / 256u;
    const uint64_t cap = (uint64_t)(cus > 0 ? cus : 256) * 16u;
    if (blocks > cap) blocks = cap;
    const dim3 grid((uint32_t)blocks), block(256);
    if (wide_sums(W, bits))   // 4-bit payloads of more than 17 workers: the sums take 16 bits
        hipLaunchKernelGGL((aggregate_fast_kernel<4, uint16_t>), grid, block, 0, stream, ptrs, W, vecs,
                           static_cast<uint16_t*>(sums));
    else if (bits == 2)
        hipLaunchKernelGGL((aggregate_fast_kernel<2, uint8_t>), grid, block, 0, stream, ptrs, W, vecs,
                           static_cast<uint8_t*>(sums));
    else if (bits == 4)
        hipLaunchKernelGGL((aggregate_fast_kernel<4, uint8_t>), grid, block, 0, stream, ptrs, W, vecs,
                           static_cast<uint8_t*>(sums));
    else
        hipLaunchKernelGGL((aggregate_fast_kernel<8, uint16_t>), grid, block, 0, stream, ptrs, W, vecs,
                           static_cast<uint16_t*>(sums));
    return hipGetLastError();
}

}  // namespace thc
