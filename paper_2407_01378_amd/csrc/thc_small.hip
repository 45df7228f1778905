// Tuned kernels for chunks of 2^5 .. 2^13 coordinates, same results as the generic ones.
//
// Encode.  A wave holds 2^11 coordinates of one worker, 32 per thread, in registers; a workgroup the same coordinates
// of ALL workers at once where they fit 16 waves (16 workers up to chunks of 2^11, 8 at 2^12, 4 at 2^13), so the shared
// range of a chunk is a maximum over a few words in LDS behind one barrier and no workgroup waits for another.  More
// workers, by size (rounds_are_better, with figures): either they are spread over workgroups of up to 8 waves that agree on the
// range through the workspace (the protocol of thc_fused14.hip: persistent grid, an item's workgroups side by side, bounded waits),
// and every gradient is read and rotated once; or one workgroup takes them in rounds, all but the last of which it rotates a
// second time.  Spread is the better one in launches that leave CUs without an item and wherever an item's rotation is long: us with the
// decoder, rounds -> spread: 8 workers x 50257, chunk 2^13 25.6 -> 15.0, 8 x 2^20 26.6 -> 20.2, 8 x 2.4 M fp32 51.4 -> 33.8, 16 x 0.75 M
// fp32 52.4 -> 28.6; 32 x 0.34 M, chunk 2^12, 8 bits 45.3 -> 28.1; 64 x 0.53 M fp32, chunk 2^10 82 -> 47.4, 32 x 2^17 22.2 -> 16.1; 64 x 2^15,
// chunk 2^8, 2 bits 34.0 -> 15.9; rounds where the items fill the CUs and the rotation is short.  (Where 16 waves do, spread over
// two workgroups is slower: 16 x 2^23, chunk 2^10 110 and 130 us.)  The rotation
// stays inside the wave up to chunks of 2^11: 5 stages between registers, 4 between lanes by
// data-parallel primitives and 2 after a swap of a lane bit into the registers (thc_lanes.h).
// Chunks of 2^12 and 2^13 span two and four waves, which trade half of their registers through LDS
// before each further stage.  Bound by vector-ALU issue while its rounds are full (8 workers, chunk 2^12, 8 bits: 27.3
// operations per worker-coordinate by the counters; one workgroup of 16 waves per CU, a round of 256 items 6 us:
// 1280 items 38.8 us, 1536 42.8, of which the operations are 35.0); a last round that is nearly empty takes as long as
// a full one (1600 items 48.2 us, 1792 48.7; with wave priorities 1600 47.0), and a launch of one item per workgroup is the item's own chain of loads,
// stages and barriers (4 workers x 2^20 fp32, chunk 2^10: 6.5 us, and 5.9 of the decoder, in a loop of each and in a trace).
//   Measured, encode + aggregate + decode: 8 workers x 6.5 M bf16, chunk 2^12, 8 bits: 762 -> 67 us
//   (3.7 TB/s); 4 workers x 1 M fp32, chunk 2^10: 178 -> 12.8 us.  Before: one range and one encode
//   launch per worker of the generic kernels, which load element by element and take a
//   barrier per stage above 2^4.
//
// Decode.  A workgroup of four waves owns 2^13 coordinates (fewer, down to the 2^11 of a wave or a chunk, where
// that spreads a short gradient over the CUs: small_decode_log2); a thread sums the workers' payload
// words of its 32 coordinates, five stages run in registers, the wave re-shuffles through its
// own 8 KB of LDS, the rest of the stages follow, and the result leaves in 128-byte lines.
// Bound by memory.
#include "thc_core14.h"
#include "thc_internal.h"
#include "thc_lanes.h"
#include "thc_payload.h"
#include "thc_resident.h"

#pragma clang fp contract(off)

namespace thc {
namespace k14 {
namespace {

constexpr uint32_t kWaveLog2 = 11;               // coordinates of a wave
constexpr uint32_t kWaveCoords = 1u << kWaveLog2;
constexpr uint32_t kMaxWaves = 16;
constexpr uint32_t kPreferredWaves = 8;          // two workgroups of 8 waves fill a CU at 128 registers
// Pauses of the wait for the peers' words, in units of 64 clocks: in front of the first read, and between reads.  Many
// workgroups publish further apart, and their reads load the path the words travel on.  Encoder, us, 16 and 4 | 24 and 4 |
// 40 and 8: 64 workers x 2^22, chunk 2^12 (16 workgroups) 237 | 233 | 225, 64 x 2^21 fp32, 2^13 (32) 173 | 170 | 164; 64 x 4 M, 2^8 (8)
// 24 and 4 175, 40 and 8 185, 48 x 2.5 M (6) 86.9 and 89.1; 20 x 4 M, 2^11 (3) 74.4 | 70.3, 32 x 8.4 M, 2^9 (4) 185 | 189.
constexpr int kFirstPollSleep = 24, kPollSleep = 4;
constexpr int kFirstPollSleepMany = 40, kPollSleepMany = 8;   // more than kFewParts workgroups
constexpr uint32_t kFewParts = 8;

// What a launch does: encode all workers of a workgroup onto their common range; only the range of one
// worker; encode one worker onto a range handed in; encode all workers, who are spread over several workgroups; encode
// all workers in one workgroup, in rounds of them.
enum class SmallOp : int { EncodeAll = 0, Absmax = 1, EncodeOnto = 2, EncodeSpread = 3, EncodeRounds = 4 };

struct SmallArgs {
    uint64_t n, padded;
    uint64_t items;           // workgroup-sized pieces of the gradient: `regions` units each
    uint32_t l;               // chunk_log2
    uint32_t W;
    uint32_t worker0;         // number of the first worker in the random stream
    uint32_t key0, key1;
    uint32_t levels;
    float norm;               // c^(-1/2)
    float* scale_out;         // may be null
    const float* scale_in;    // EncodeOnto
    uint32_t* error;          // EncodeAll: may be null, four words that a good run leaves zero; EncodeSpread: set if a wait expires
    // shape of a workgroup: wave = (region * groups + group) * 2^wpw_log2 + part; a unit is the
    // 2^max(11, l) coordinates of one worker that its 2^wpw_log2 waves hold, a group is one worker
    uint32_t wpw_log2, groups, regions;
    // EncodeSpread: workgroups of an item (each has `groups` of the workers), a word per chunk for each of them and one
    // counter per chunk, all zero before and after.  EncodeRounds: rounds, of `groups` workers each
    uint32_t parts;
    uint32_t max_spins;
    uint32_t* slots;
    uint32_t* done;
};

// Coordinate ranges by chunk size: CLASS 0: l <= 9, 1: l = 10, 11, 2: l = 12, 13.
constexpr int class_of(uint32_t l) { return l <= 9 ? 0 : l <= 11 ? 1 : 2; }

template <bool BF16, int CLASS, int BITS, SmallOp OP>
__global__ __launch_bounds__(64 * kMaxWaves) void small_encode_kernel(const SmallArgs a, const FusedWorkerPtrs ptrs) {
    constexpr int kUnits = BF16 ? 4 : 8;
    constexpr int kElem = BF16 ? 2 : 4;
    // bf16 input is loaded one item ahead.  fp32 (32 registers in flight) when its item starts: ahead, the kernel spills.  Pass
    // with the decoder, us, ahead -> this: 4 workers x 2^20, chunk 2^10 14.9 -> 13.3, 8 x 2^20 20.7 -> 16.4, 8 x 2^22 44.7 -> 38.8,
    // 2 x 2^24 53.4 -> 47.7, 8 x 2^23, chunk 2^12 91.6 -> 78.4; 8 x 2^24, chunk 2^11 166 -> 154.
    constexpr bool kAhead = BF16;
    constexpr bool kRounds = OP == SmallOp::EncodeRounds;
    extern __shared__ uint4 dyn[];
    const uint32_t t = threadIdx.x, lane = t & 63u;
    // (the wave's number is the same for all lanes: kept in a scalar register, so are the
    // addresses that follow from it)
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    const uint32_t waves = blockDim.x >> 6;
    const uint32_t wpw = CLASS == 2 ? 1u << a.wpw_log2 : 1u;
    const uint32_t part = wave & (wpw - 1u);
    const uint32_t rg = CLASS == 2 ? wave >> a.wpw_log2 : wave;
    const uint32_t region = rg / a.groups;
    const uint32_t group = rg - region * a.groups;
    const uint32_t block = lanes::block_of_lane(lane);
    const uint32_t unit_log2 = CLASS == 2 ? a.l : kWaveLog2;

    // LDS: staging of fp32 input / the traded registers, two sign tables, two range tables
    constexpr uint32_t kStage = !BF16 || CLASS == 2 ? 512u : 0u;   // 16-byte units per wave
    const uint32_t sign_words = a.regions * (1u << (unit_log2 - 5u));
    uint4* stage = dyn + kStage * wave;
    uint32_t* sign = reinterpret_cast<uint32_t*>(dyn + kStage * waves);
    // chunks of a unit (one row of range words each), entries of a row: groups x waves of a chunk
    const uint32_t rows_log2 = a.l < kWaveLog2 ? kWaveLog2 - a.l : 0u;
    const uint32_t row = (a.groups * wpw + 3u) & ~3u;
    float* red = reinterpret_cast<float*>(sign + 2u * sign_words);
    const uint32_t red_words = (a.regions << rows_log2) * row;
    if (OP == SmallOp::EncodeAll || OP == SmallOp::EncodeSpread || kRounds) {
        for (uint32_t i = t; i < 2u * red_words; i += blockDim.x) red[i] = 0.0f;   // (the unused end of a row stays zero)
    }
    uint32_t* got = reinterpret_cast<uint32_t*>(red + red_words);   // EncodeSpread: the peers' words, instead of the second table
    // this lane's chunk inside its unit
    const uint32_t chunk = CLASS == 0 ? block >> (a.l - 5u) : (CLASS == 1 && a.l == 10u ? lane >> 5 : 0u);
    float* red_row = red + ((region << rows_log2) + chunk) * row;

    // where the two runs of 16 coordinates lie that the lane holds after the rotation
    uint32_t run0, run1;
    if (CLASS == 0) {
        run0 = block << 5;
        run1 = run0 + 16u;
    } else {   // i4 = lane bit 4, i5..i8 as before, i9 and above as the swaps left them
        const uint32_t mid = ((lane & 16u)) | ((block & 15u) << 5);
        if (CLASS == 1 && a.l == 10u) {          // register bit 4 = i9, lane bit 5 = i10
            run0 = mid | ((lane >> 5) << 10);
            run1 = run0 + 512u;
        } else if (CLASS == 1) {                 // register bit 4 = i10, lane bit 5 = i9
            run0 = mid | ((lane >> 5) << 9);
            run1 = run0 + 1024u;
        } else {                                 // register bit 4 = i(l - 1), part = i10 (and i11)
            run0 = mid | ((lane >> 5) << 9) | (part << 10);
            run1 = run0 + (1u << (a.l - 1u));
        }
    }
    const float sg0 = (block & 1u) ? -1.0f : 1.0f, sg1 = (block & 2u) ? -1.0f : 1.0f,
                sg2 = (block & 4u) ? -1.0f : 1.0f, sg3 = (block & 8u) ? -1.0f : 1.0f;
    const uint32_t lane_stages = CLASS == 0 ? a.l - 5u : 4u;   // how many of i5..i8 are rotated
    const float neg = (__popc(block & ((1u << lane_stages) - 1u)) & 1) ? -1.0f : 1.0f;

    // EncodeSpread: which of an item's workgroups this one is, and the items it takes
    const uint32_t parts = OP == SmallOp::EncodeSpread ? a.parts : 1u;
    const uint32_t first = OP == SmallOp::EncodeSpread ? blockIdx.x / parts : blockIdx.x;
    const uint32_t stride = OP == SmallOp::EncodeSpread ? gridDim.x / parts : gridDim.x;
    const uint32_t mine = OP == SmallOp::EncodeSpread ? blockIdx.x - first * parts : 0u;
    uint32_t w = group + a.groups * mine;   // the worker
    // EncodeRounds: a turn is one worker's unit.  The first `parts` turns find the range; the last of them is quantized where
    // it stands, the ones before it are rotated once more, backwards.
    const uint32_t turns = kRounds ? 2u * a.parts - 1u : 1u;
    auto worker_of = [&](uint32_t turn) { return group + a.groups * (turn < a.parts ? turn : turns - 1u - turn); };
    auto coord0_of = [&](uint64_t item) { return (item * a.regions + region) << unit_log2; };

    Raw<kUnits> raw;
    uint32_t odd_tail = 0u;   // BF16: the last coordinate of an odd count, in the lane that owns it
    auto load = [&](uint64_t item, uint32_t w) {
        const uint64_t g0 = coord0_of(item) + part * kWaveCoords;
        uint64_t left = (item < a.items && w < a.W && g0 < a.n) ? a.n - g0 : 0u;
        if (left > (uint64_t)kWaveCoords) left = kWaveCoords;
        uint64_t addr = reinterpret_cast<uint64_t>(ptrs.grad[w < a.W ? w : 0u]) + (left != 0u ? g0 * kElem : 0u);
        addr = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(addr >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)addr);
        // reads past the range return zero; its check works on dwords, so the last coordinate
        // of an odd count of bf16 is fetched by itself
        const uint32_t bytes = BF16 ? ((uint32_t)left & ~1u) * 2u : (uint32_t)left * 4u;
        __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(addr), 0, bytes, 0x00020000);
        typedef uint32_t u4v __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int j = 0; j < kUnits; ++j) {
            // bf16: the lane's own 64 bytes; fp32: coalesced, dealt out through the wave's LDS
            const uint32_t unit = BF16 ? 4u * block + j : (uint32_t)j * 64u + lane;
            const u4v q = __builtin_amdgcn_raw_buffer_load_b128(rsrc, unit * 16u, 0, 0);
            raw.u[j] = make_uint4(q.x, q.y, q.z, q.w);
        }
        if (BF16 && (left & 1u)) {
            odd_tail = 0u;
            if (block == (uint32_t)left >> 5)
                odd_tail = reinterpret_cast<const uint16_t*>(addr)[left - 1u];
        }
    };
    // the coordinates of the item that exist (for the odd tail), as load() saw them
    auto left_of = [&](uint64_t item) -> uint32_t {
        const uint64_t g0 = coord0_of(item) + part * kWaveCoords;
        const uint64_t left = (item < a.items && w < a.W && g0 < a.n) ? a.n - g0 : 0u;
        return left > (uint64_t)kWaveCoords ? kWaveCoords : (uint32_t)left;
    };
    auto fill_signs = [&](uint64_t item, uint32_t which) {
        if (t < sign_words / 4u) {
            const u32x4 s = sign_block(((item * a.regions) << (unit_log2 - 7u)) + t, a.key0, a.key1);
            uint4 o = make_uint4(s.w[0], s.w[1], s.w[2], s.w[3]);
            if (BF16) o = make_uint4(unshuffle_bits(s.w[0]), unshuffle_bits(s.w[1]), unshuffle_bits(s.w[2]), unshuffle_bits(s.w[3]));
            reinterpret_cast<uint4*>(sign + which * sign_words)[t] = o;
        }
    };

    if (kAhead) load(first, w);
    fill_signs(first, 0u);
    // What the items need of the arguments later, read while the input is on its way: left to the compiler, some of these
    // scalar reads stand where their values are used, behind the barriers, and the wave waits for them there.
    uint64_t payload_at = OP != SmallOp::Absmax ? reinterpret_cast<uint64_t>(ptrs.payload[w < a.W ? w : 0u]) : 0u;
    uint64_t out_at = reinterpret_cast<uint64_t>(a.scale_out), in_at = reinterpret_cast<uint64_t>(a.scale_in);
    uint32_t step = stride;
    asm volatile("" : "+s"(payload_at), "+s"(out_at), "+s"(in_at), "+s"(step));
    uint8_t* payload = global_ptr<uint8_t>(payload_at);
    float* scale_out = global_ptr<float>(out_at);
    const float* scale_in = global_ptr<const float>(in_at);
    __syncthreads();
    uint32_t cur = 0u;
    // EncodeSpread: first chunk and number of chunks of this and of the previous item
    const uint64_t chunks = a.padded >> a.l;
    uint64_t prev0 = 0u;
    uint32_t prev_live = 0u;
    uint32_t turn = 0u, most = 0u;   // most: largest magnitude of the lane's chunk, as a word
    float s = 0.0f;
    for (uint64_t item = first; item < a.items;) {
        const bool ends = !kRounds || turn + 1u == turns;   // the item's last turn
        const uint64_t u0 = coord0_of(item);
        const uint64_t p = (u0 >> a.l) + chunk;
        const bool exists = (p << a.l) < a.padded;
        const uint32_t sx = sign[cur * sign_words + (region << (unit_log2 - 5u)) + part * 64u + block];
        float v[kRegs];
        if constexpr (BF16) {
            if (a.n & 1u) {   // (uniform)
                const uint32_t left = left_of(item);
                if ((left & 1u) && block == left >> 5) {
                    const uint32_t d = (left & 31u) >> 1;   // dword of the lane's 16 that holds it
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        raw.u[k].x = d == 4u * k ? odd_tail : raw.u[k].x;
                        raw.u[k].y = d == 4u * k + 1u ? odd_tail : raw.u[k].y;
                        raw.u[k].z = d == 4u * k + 2u ? odd_tail : raw.u[k].z;
                        raw.u[k].w = d == 4u * k + 3u ? odd_tail : raw.u[k].w;
                    }
                }
            }
            units_to_l1<kUnits, true>(sx, raw.u, v);
        } else {
            if (!kAhead) load(item, w);
#pragma unroll
            for (int j = 0; j < kUnits; ++j) stage[lay14::stage_unit((uint32_t)j * 64u + lane)] = raw.u[j];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            uint4 unit[kUnits];
#pragma unroll
            for (int k = 0; k < kUnits; ++k) unit[k] = stage[lay14::stage_unit(8u * block + k)];
            units_to_l1<kUnits, true>(sx, unit, v);
        }
#pragma unroll
        for (int i = 0; i < kRegs; ++i) asm volatile("" : "+v"(v[i]));   // converted before `raw` is loaded again
        asm volatile("" ::: "memory");
        if (kAhead) load(ends ? item + step : item, kRounds ? worker_of(ends ? 0u : turn + 1u) : w);
        if ((!kRounds || turn == 0u) && item + step < a.items) fill_signs(item + step, cur ^ 1u);

        // (as in the chunk-2^14 encoder: the rotation ahead of the other workgroup's quantizer.  Encoder alone, us: 8 workers
        // x 2^24, chunk 2^13 129 -> 116, 64 x 2^22, chunk 2^12 250 -> 221; one workgroup per CU 48.7 -> 47.0)
        set_prio<true, kPrioRotateEarly>();
        butterflies<0, 5>(v);
        if (CLASS != 0 || a.l > 5u) lanes::lane_stage<0>(v, sg0);
        if (CLASS != 0 || a.l > 6u) lanes::lane_stage<1>(v, sg1);
        if (CLASS != 0 || a.l > 7u) lanes::lane_stage<2>(v, sg2);
        if (CLASS != 0 || a.l > 8u) lanes::lane_stage<3>(v, sg3);
        if constexpr (CLASS != 0) {
            lanes::swap_top_register_bit<16>(v);
            butterflies<4, 5>(v);
            if (CLASS == 2 || a.l > 10u) {
                lanes::swap_top_register_bit<32>(v);
                butterflies<4, 5>(v);
            }
        }
        if constexpr (CLASS == 2) {
            // (two buffers, free again behind the item's last barrier)
            set_prio<OP == SmallOp::EncodeSpread, kPrioRotateLate>();
            float4* buf = reinterpret_cast<float4*>(dyn);
            trade_halves(v, buf + kStage * wave, buf + kStage * (wave ^ 1u), (part & 1u) != 0u, lane);
            butterflies<4, 5>(v);
            if (a.l > 12u) {
                buf += 256;
                trade_halves(v, buf + kStage * wave, buf + kStage * (wave ^ 2u), (part & 2u) != 0u, lane);
                butterflies<4, 5>(v);
            }
            if (kRounds) __syncthreads();   // (the next turn stores into them)
        }

        if (OP != SmallOp::EncodeOnto && (!kRounds || turn < a.parts)) {
            // the chunk's largest magnitude: registers, then the lanes that share the chunk
            float m = 0.0f;
#pragma unroll
            for (int i = 0; i < kRegs; i += 2)
                asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(m), "v"(v[i]), "v"(v[i + 1]));
            uint32_t x = __float_as_uint(m * a.norm);   // non-negative floats order like their bit patterns
            if (CLASS != 0 || a.l > 5u) x = lanes::umax_step<1>(x);
            if (CLASS != 0 || a.l > 6u) x = lanes::umax_step<2>(x);
            if (CLASS != 0 || a.l > 7u) x = lanes::umax_step<7>(x);
            if (CLASS != 0 || a.l > 8u) x = lanes::umax_step<15>(x);
            if constexpr (CLASS != 0) {
                x = lanes::umax_step<16>(x);
                if (CLASS == 2 || a.l > 10u) x = lanes::umax_step<32>(x);
            }
            most = kRounds && turn != 0u && most > x ? most : x;
        }
        const bool leader = CLASS == 0 ? (block & ((1u << (a.l - 5u)) - 1u)) == 0u
                                       : (CLASS == 1 && a.l == 10u ? (lane & 31u) == 0u : lane == 0u);
        if (kRounds && turn + 1u != a.parts) {
            // (the range is not known yet, or it is already)
        } else if (OP == SmallOp::EncodeAll || kRounds) {
            // all workers' waves have published behind the barrier (which also orders the sign
            // table of the next item); the two range tables take turns
            float* at = red_row + cur * red_words;
            if (leader) at[group * wpw + part] = __uint_as_float(most);
            __syncthreads();
            s = 0.0f;
            for (uint32_t i = 0; i < row; i += 4u) {
                const float4 f = *reinterpret_cast<const float4*>(at + i);
                s = fmaxf(fmaxf(s, fmaxf(f.x, f.y)), fmaxf(f.z, f.w));
            }
            if (leader && group == 0u && part == 0u && exists && out_at) scale_out[p] = s;
        } else if (OP == SmallOp::EncodeSpread) {
            // The waves' maxima meet in LDS; the first wave publishes the workgroup's word of every chunk and waits for
            // the peers' (see EncodeAllCtx in thc_fused14.hip, whose protocol this is, in the form with one reader).
            if (leader) red_row[group * wpw + part] = __uint_as_float(most);
            __syncthreads();   // (also orders the sign table of the next item)
            if (wave == 0u) {
                const uint64_t p0 = coord0_of(item) >> a.l;
                const uint32_t live = chunks - p0 < (1ull << rows_log2) ? (uint32_t)(chunks - p0) : 1u << rows_log2;
                uint32_t* words = a.slots + p0 * parts;
                if (lane < live) {
                    const float* at = red + lane * row;
                    float m = 0.0f;
                    for (uint32_t i = 0; i < row; i += 4u) {
                        const float4 f = *reinterpret_cast<const float4*>(at + i);
                        m = fmaxf(fmaxf(m, fmaxf(f.x, f.y)), fmaxf(f.z, f.w));
                    }
                    __hip_atomic_store(&words[lane * parts + mine], __float_as_uint(m) | 0x80000000u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                }
                if (parts > kFewParts) __builtin_amdgcn_s_sleep(kFirstPollSleepMany);
                else __builtin_amdgcn_s_sleep(kFirstPollSleep);
                bool seen = false;
                for (uint32_t spins = 0;; ++spins) {
                    uint32_t valid = 0x80000000u;
                    for (uint32_t base = 0; base < live * parts; base += 64u) {
                        const uint32_t i = base + lane;
                        if (i < live * parts) {
                            const uint32_t val = __hip_atomic_load(&words[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            valid &= val;
                            got[i] = val & 0x7FFFFFFFu;
                        }
                    }
                    seen = __all(valid != 0u);
                    if (seen || spins >= a.max_spins) break;
                    if (parts > kFewParts) __builtin_amdgcn_s_sleep(kPollSleepMany);
                    else __builtin_amdgcn_s_sleep(kPollSleep);
                }
                if (!seen && lane == 0u) __hip_atomic_store(a.error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                // With all of this item's words seen every peer has read the previous item's: nobody will read them
                // again, and this workgroup clears its own.
                if (seen && lane < prev_live)
                    __hip_atomic_store(&a.slots[(prev0 + lane) * parts + mine], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                prev0 = p0;
                prev_live = live;
            }
            __syncthreads();
            // the next item's input has arrived in the meantime; knowing that, the compiler does not wait for it
            // behind the stores below
#pragma unroll
            for (int j = 0; kAhead && j < kUnits; ++j)
                asm volatile("" : "+v"(raw.u[j].x), "+v"(raw.u[j].y), "+v"(raw.u[j].z), "+v"(raw.u[j].w));
            uint32_t x = 0u;
            if (exists)
                for (uint32_t i = 0; i < parts; ++i) x = max(x, got[chunk * parts + i]);
            s = __uint_as_float(x);
            if (leader && mine == 0u && group == 0u && part == 0u && exists) scale_out[p] = s;
        } else if (OP == SmallOp::Absmax) {
            if (CLASS == 2) {
                float* at = red_row + cur * red_words;
                if (leader) at[part] = __uint_as_float(most);
                __syncthreads();
                s = 0.0f;
                for (uint32_t i = 0; i < wpw; ++i) s = fmaxf(s, at[i]);
                if (leader && part == 0u && exists) scale_out[p] = s;
            } else {
                if (leader && exists) scale_out[p] = __uint_as_float(most);
                __syncthreads();   // the next item's sign table
            }
        } else {
            s = exists ? scale_in[p] : 0.0f;
            if (leader && part == 0u && exists && out_at) scale_out[p] = s;
            __syncthreads();       // the next item's sign table
        }

        set_prio<true, kPrioTail>();
        if (OP != SmallOp::Absmax && (!kRounds || turn + 1u >= a.parts) && w < a.W) {
            constexpr bool kClamp = OP == SmallOp::EncodeOnto;
            constexpr bool kOffset = ((1u << BITS) - 2u) > kSingleFmaMaxLevels;
            const float two = s + s;
            const bool ranged = two >= kMinRange;
            const float inv = ranged ? (float)a.levels / two : 0.0f;
            const float base = ((ranged ? !kOffset : (a.levels & 1u) == 0u) ? 0.5f * (float)a.levels : 0.0f) + 0x1p-9f;
            const uint64_t b0 = (u0 + run0) >> 4, b1 = (u0 + run1) >> 4;
            const uint32_t worker = a.worker0 + w;
            uint32_t by[8], pk[BITS];
            // even l: c^(-1/2) is a power of two and moves into the multiplier (see quantize_pack);
            // the condition must hold for every lane, chunks of one wave differ in s
            const bool fold = (a.l & 1u) == 0u && __all(!ranged || (s >= 0x1p-100f && s <= 0x1p100f));
            if (fold) {
                const float sub = -s * (1.0f / a.norm);
                const float mul = inv * a.norm * (kOffset ? 1.0f : neg);
                quantize_half<BITS, kClamp, true, kOffset, true>(v, 0, b0, sub, mul, base, a.levels, worker, a.key0, a.key1, by, 1.0f, neg);
                quantize_half<BITS, kClamp, true, kOffset, true>(v, 1, b1, sub, mul, base, a.levels, worker, a.key0, a.key1, by, 1.0f, neg);
            } else {
                const float norm = a.norm * neg;
                quantize_half<BITS, kClamp, false, kOffset, true>(v, 0, b0, -s, inv, base, a.levels, worker, a.key0, a.key1, by, norm, neg);
                quantize_half<BITS, kClamp, false, kOffset, true>(v, 1, b1, -s, inv, base, a.levels, worker, a.key0, a.key1, by, norm, neg);
            }
            pack_bytes<BITS>(by, pk);
            uint8_t* dst = kRounds ? global_ptr<uint8_t>(reinterpret_cast<uint64_t>(ptrs.payload[w])) : payload;
            if constexpr (CLASS == 0) {   // 32 consecutive coordinates
                if (exists) store_packed<BITS>(pk, dst + b0 * (2u * BITS));
            } else if (exists) {
                uint8_t* d0 = dst + b0 * (2u * BITS);
                uint8_t* d1 = dst + b1 * (2u * BITS);
                if constexpr (BITS == 8) {
                    *reinterpret_cast<uint4*>(d0) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
                    *reinterpret_cast<uint4*>(d1) = make_uint4(pk[4], pk[5], pk[6], pk[7]);
                } else if constexpr (BITS == 4) {
                    *reinterpret_cast<uint2*>(d0) = make_uint2(pk[0], pk[1]);
                    *reinterpret_cast<uint2*>(d1) = make_uint2(pk[2], pk[3]);
                } else {
                    *reinterpret_cast<uint32_t*>(d0) = pk[0];
                    *reinterpret_cast<uint32_t*>(d1) = pk[1];
                }
            }
        }
        if (ends) {
            if (kRounds) __syncthreads();   // (the turns behind the range's barrier read the sign table too)
            item += step;
            cur ^= 1u;
            turn = 0u;
        } else {
            ++turn;
        }
        if (kRounds) w = worker_of(turn);
    }
    if ((OP == SmallOp::EncodeAll || kRounds) && a.error && blockIdx.x == 0 && t < 4u) a.error[t] = 0u;
    if (OP == SmallOp::EncodeSpread && wave == 0u && prev_live != 0u) {
        // the last item's words: its workgroups count themselves off, the last one clears them and the counter
        uint32_t arrived = 0u;
        if (lane == 0u)
            arrived = __hip_atomic_fetch_add(&a.done[prev0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        arrived = (uint32_t)__builtin_amdgcn_readfirstlane((int)arrived);
        if (arrived == parts - 1u) {
            for (uint32_t i = lane; i < prev_live * parts; i += 64u)
                __hip_atomic_store(&a.slots[prev0 * parts + i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0u) __hip_atomic_store(&a.done[prev0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ------------------------------------------------------------------------------ decode
constexpr int kDecodeThreads = 256;    // of a workgroup, at most
constexpr uint32_t kDecodeLog2 = 13;   // its coordinates

struct SmallDecodeArgs {
    uint64_t n, padded;
    uint32_t l, W;
    uint32_t key0, key1;
    float norm;
    const float* scale;
    const void* in;     // stored sums (SRC u8 / u16)
    void* sums;         // SRC payloads: where the integer sums go; may be null
    float* out;
};

// SRC: 0 the workers' payloads, 1 stored u8 sums, 2 stored u16 sums.  WIDE, ONCE: see PayloadSum.
template <int SRC, int BITS, bool WIDE, bool ONCE = BITS != 8>
__global__ __launch_bounds__(kDecodeThreads, 4) void small_decode_kernel(const SmallDecodeArgs a,
                                                                      const FusedPayloadPtrs ptrs) {
    __shared__ float4 xb4[4 * 512];
    __shared__ alignas(16) uint32_t sign[1u << (kDecodeLog2 - 5u)];
    const uint32_t t = threadIdx.x, lane = t & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    const uint64_t base = (uint64_t)blockIdx.x * (blockDim.x * 32u);
    const uint64_t g = base + 32u * t;
    const bool exists = g < a.padded;   // (chunks are whole multiples of a thread's 32 coordinates)
    // A thread beyond the end reads what the first one reads, and stores nothing: loads under a condition have a zero to
    // merge with, and the copy of the first one's result into the merged registers waited for it in front of
    // the second load and of the sign table (stored sums, 12 M coordinates, chunk 2^10, 4 bits: 15.6 us so, 12.0 without).
    const uint64_t from = exists ? g : base;
    const uint32_t l = a.l;
    uint32_t S[kRegs];
    const float s = a.scale[from >> l];
    if constexpr (SRC == 0) {
        PayloadSum<BITS, false, WIDE, ONCE> sum{ptrs, nullptr, a.W};
        sum.clear();
        sum.all_alone((from * BITS) / 8u);
        if (t < blockDim.x / 4u) *reinterpret_cast<u32x4*>(&sign[4 * t]) = sign_block((base >> 7) + t, a.key0, a.key1);
        sum.unpack(S);
        if (a.sums && exists) {
            if (BITS == 8 || WIDE) store_sums16(S, static_cast<uint16_t*>(a.sums) + g);
            else store_sums8(S, static_cast<uint8_t*>(a.sums) + g);
        }
    } else {
        constexpr int kVecs = 2 * SRC;
        uint4 q[kVecs];
#pragma unroll
        for (int k = 0; k < kVecs; ++k)
            q[k] = load_last_use(reinterpret_cast<const uint4*>(static_cast<const uint8_t*>(a.in) + from * SRC) + k);
        if (t < blockDim.x / 4u) *reinterpret_cast<u32x4*>(&sign[4 * t]) = sign_block((base >> 7) + t, a.key0, a.key1);
#pragma unroll
        for (int k = 0; k < kVecs; ++k) {
            const uint32_t x[4] = {q[k].x, q[k].y, q[k].z, q[k].w};
#pragma unroll
            for (int e = 0; e < 16 / SRC; ++e) {
                constexpr int per = 4 / SRC;
                S[16 / SRC * k + e] = (x[e / per] >> (8 * SRC * (e % per))) & (SRC == 1 ? 0xFFu : 0xFFFFu);
            }
        }
    }
    const float qf = ((s + s) / (float)((1u << BITS) - 1u)) / (float)a.W;
    float v[kRegs];
#pragma unroll
    for (int r = 0; r < kRegs; ++r) v[r] = (float)S[r] * qf - s;

    butterflies<0, 5>(v);
    float* reg = reinterpret_cast<float*>(xb4) + wave * 2048u;
#pragma unroll
    for (int q = 0; q < 8; ++q)
        reinterpret_cast<float4*>(reg)[lay14::x1_store(lane, q) >> 2] =
            make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int r = 0; r < kRegs; ++r) v[r] = reg[lay14::x1_load(lane, r)];
    // now register = i5..i9, lane = i0..i4, i10
    if (l > 5u) butterflies<0, 1>(v);
    if (l > 6u) butterflies<1, 2>(v);
    if (l > 7u) butterflies<2, 3>(v);
    if (l > 8u) butterflies<3, 4>(v);
    if (l > 9u) butterflies<4, 5>(v);
    __syncthreads();   // the sign table; every wave has read its part of the buffer
    // where register r's coordinate lies: (lane & 31) + 32 (r & 15) + at + (r >> 4) hi
    uint32_t at = wave * kWaveCoords + ((lane >> 5) << 10), hi = 512u;
    if (l > 10u) {
        lanes::swap_top_register_bit<32>(v);   // register bit 4 = i10, lane bit 5 = i9
        butterflies<4, 5>(v);
        at = wave * kWaveCoords + ((lane >> 5) << 9);
        hi = 1024u;
    }
    if (l > 11u) {
        trade_halves(v, xb4 + 512u * wave, xb4 + 512u * (wave ^ 1u), (wave & 1u) != 0u, lane);
        butterflies<4, 5>(v);
        at = ((wave >> 1) << 12) + ((wave & 1u) << 10) + ((lane >> 5) << 9);
        hi = 2048u;
    }
    if (l > 12u) {
        trade_halves(v, xb4 + 256 + 512u * wave, xb4 + 256 + 512u * (wave ^ 2u), (wave & 2u) != 0u, lane);
        butterflies<4, 5>(v);
        at = (wave << 10) + ((lane >> 5) << 9);
        hi = 4096u;
    }
    float* out = a.out + base + at + (lane & 31u);
    const uint32_t* sw = sign + (at >> 5);
    const uint32_t shift = 31u - (lane & 31u);
    const uint64_t left = a.n - base;   // (the grid covers n: base < n)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 sq = *reinterpret_cast<const uint4*>(sw + (h * hi >> 5) + 4 * q);
            const uint32_t wd[4] = {sq.x, sq.y, sq.z, sq.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 16 * h + 4 * q + e;
                const uint32_t off = h * hi + 32u * (4 * q + e);
                const uint32_t x = xor_masked(__float_as_uint(v[r] * a.norm), wd[e] << shift, 0x80000000u);
                if (at + (lane & 31u) + off < left) __builtin_nontemporal_store(__uint_as_float(x), out + off);
            }
        }
    }
}

// ------------------------------------------------------------------------------ launch
template <bool BF16, int CLASS, int BITS, SmallOp OP>
hipError_t launch_encode_t(const SmallArgs& a, const FusedWorkerPtrs& ptrs, hipStream_t stream) {
    constexpr auto kernel = small_encode_kernel<BF16, CLASS, BITS, OP>;
    const uint32_t wpw = 1u << a.wpw_log2, waves = a.regions * a.groups * wpw;
    const uint32_t unit_log2 = a.l > kWaveLog2 ? a.l : kWaveLog2;
    const uint32_t rows_log2 = a.l < kWaveLog2 ? kWaveLog2 - a.l : 0u;
    const uint32_t lds = waves * (!BF16 || CLASS == 2 ? 8192u : 0u) +
                         2u * 4u * (a.regions << (unit_log2 - 5u)) +
                         2u * 4u * (a.regions << rows_log2) * ((a.groups * wpw + 3u) & ~3u) +
                         (OP == SmallOp::EncodeSpread ? 4u * (a.parts << rows_log2) : 0u);
    if (!allow_lds<kernel>(lds)) return hipErrorInvalidValue;
    uint64_t G = resident_grid<kernel>(64u * waves, lds);
    if (OP == SmallOp::EncodeSpread) G /= a.parts;   // an item's workgroups wait for one another: all of them resident
    if (G == 0) return hipErrorInvalidValue;
    if (G > a.items) G = a.items;
    if (OP == SmallOp::EncodeSpread) G *= a.parts;
    hipLaunchKernelGGL(kernel, dim3((uint32_t)G), dim3(64u * waves), lds, stream, a, ptrs);
    return hipGetLastError();
}

template <bool BF16, int CLASS, SmallOp OP>
hipError_t launch_encode_bits(const SmallArgs& a, const FusedWorkerPtrs& ptrs, uint32_t bits, hipStream_t stream) {
    if (OP == SmallOp::Absmax) return launch_encode_t<BF16, CLASS, 4, SmallOp::Absmax>(a, ptrs, stream);
    if (bits == 2) return launch_encode_t<BF16, CLASS, 2, OP>(a, ptrs, stream);
    if (bits == 4) return launch_encode_t<BF16, CLASS, 4, OP>(a, ptrs, stream);
    return launch_encode_t<BF16, CLASS, 8, OP>(a, ptrs, stream);
}

template <SmallOp OP>
hipError_t launch_encode(SmallArgs& a, const FusedWorkerPtrs& ptrs, bool bf16, uint32_t bits, hipStream_t stream) {
    // Shape of a workgroup.  All workers of a unit side by side, and as many units as fill 8 waves; spread: the workers,
    // evenly, over workgroups of up to 8 waves; rounds: evenly, over as few rounds of up to 16 waves as there can be.
    a.wpw_log2 = a.l > kWaveLog2 ? a.l - kWaveLog2 : 0u;
    const uint32_t most = kMaxWaves >> a.wpw_log2;
    if (OP == SmallOp::EncodeRounds) a.parts = (a.W + most - 1u) / most;
    const uint32_t split = OP == SmallOp::EncodeSpread || OP == SmallOp::EncodeRounds ? a.parts : 1u;
    a.groups = (a.W + split - 1u) / split;
    const uint32_t per_region = a.groups << a.wpw_log2;
    a.regions = split == 1u && per_region < kPreferredWaves ? kPreferredWaves / per_region : 1u;
    const uint32_t unit_log2 = a.l > kWaveLog2 ? a.l : kWaveLog2;
    const uint64_t units = (a.padded + (1ull << unit_log2) - 1u) >> unit_log2;
    // (a few units: spread over the CUs before they share a workgroup)
    while (a.regions > 1u && units <= (uint64_t)device_cus() * (a.regions >> 1)) a.regions >>= 1;
    a.items = (units + a.regions - 1u) / a.regions;
    const int cls = class_of(a.l);
    if (bf16) {
        if (cls == 0) return launch_encode_bits<true, 0, OP>(a, ptrs, bits, stream);
        if (cls == 1) return launch_encode_bits<true, 1, OP>(a, ptrs, bits, stream);
        return launch_encode_bits<true, 2, OP>(a, ptrs, bits, stream);
    }
    if (cls == 0) return launch_encode_bits<false, 0, OP>(a, ptrs, bits, stream);
    if (cls == 1) return launch_encode_bits<false, 1, OP>(a, ptrs, bits, stream);
    return launch_encode_bits<false, 2, OP>(a, ptrs, bits, stream);
}

// More workers than 16 waves: in rounds of them in one workgroup (all rounds but the last are rotated twice, a CU has one
// such workgroup), or spread over `parts` workgroups of half its size that agree on the range.  Rounds of the grid in both
// forms: ceil(items / CUs) and ceil(items / (2 CUs / parts)); one of the first form takes about parts (l + 4 for fp32) / 14 as long
// as one of the second, whose agreement costs more the more chunks an item has (64 at 2^5).  Over 1907 shapes (l = 5 .. 13, 5 .. 64
// workers, 64 .. 2048 items) that picks a form 0.3 % slower than the better one on average, where spread throughout is 3.3 %
// and rounds throughout 19 %.  Encoder, us, rounds | spread, bf16 4 bits: chunk 2^5, 17 workers x 2^19 10.0 | 14.7, 64 x 2^20 53 | 73, 32 x
// 2^22 91 | 113; 2^8, 17 x 2^20 19.4 | 22.1, 32 x 2^20 28.3 | 26.6, 64 x 2^21 102 | 96; 2^8, 17 x 2^18 11.2 | 8.7; 2^11, 32 x 2^21 61 | 56; fp32,
// 2^8, 32 x 2^20 33 | 28.
// Three parts of a grid of the first form that is one nearly full round (the spread form's second round is half empty): 17 workers x
// 2^19, 2^10 12.9 | 14.8, fp32 12.7 | 14.8; 20 x 2^19, 2^10 13.7 | 14.6; 9 x 2^20, 2^12 14.8 | 16.0; at 2^13 the same or slower.
bool rounds_are_better(uint32_t parts, uint32_t l, uint64_t chunks, bool bf16) {
    const uint64_t cus = (uint64_t)device_cus(), groups = 2u * cus / parts;
    if (groups == 0u) return true;   // (the form that waits for nobody)
    const uint32_t unit_log2 = l > kWaveLog2 ? l : kWaveLog2;
    const uint64_t items = ((chunks << l) + (1ull << unit_log2) - 1u) >> unit_log2;
    const uint64_t in_rounds = (items + cus - 1u) / cus, spread = (items + groups - 1u) / groups;
    if (parts == 3u && l <= 12u && items <= cus && 8u * items > 7u * cus) return true;
    return in_rounds * parts * (bf16 ? l : l + 4u) < 14u * spread;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool small_size(uint32_t chunk_log2) { return chunk_log2 >= 5u && chunk_log2 < 14u; }

}  // namespace
}  // namespace k14

bool small_encode_all_applicable(const EncodeAllArgs& a, const FusedWorkerPtrs& ptrs, uint32_t chunk_log2) {
    if (!k14::small_size(chunk_log2) || a.W > (uint32_t)kMaxFusedWorkers) return false;
    for (uint32_t w = 0; w < a.W; ++w)
        if (!k14::aligned16(ptrs.grad[w]) || !k14::aligned16(ptrs.payload[w])) return false;
    return true;
}

// Over how many workgroups the workers of a chunk are spread; more than one: they agree on the range through the workspace.
uint32_t small_encode_parts(uint32_t W, uint32_t chunk_log2, uint64_t chunks, bool bf16) {
    const uint32_t wpw_log2 = chunk_log2 > k14::kWaveLog2 ? chunk_log2 - k14::kWaveLog2 : 0u;
    const uint32_t waves = W << wpw_log2;
    if (waves <= k14::kMaxWaves) return 1u;
    const uint32_t parts = (waves + k14::kPreferredWaves - 1u) / k14::kPreferredWaves;
    return k14::rounds_are_better(parts, chunk_log2, chunks, bf16) ? 1u : parts;
}

hipError_t launch_small_encode_all(const EncodeAllArgs& e, const FusedWorkerPtrs& ptrs, uint32_t chunk_log2, float norm,
                                   bool bf16, uint32_t bits, uint32_t parts, bool clear_error, hipStream_t stream) {
    k14::SmallArgs a{};
    a.n = e.n;
    a.padded = e.chunks << chunk_log2;
    a.l = chunk_log2;
    a.W = e.W;
    a.key0 = e.key0;
    a.key1 = e.key1;
    a.levels = e.levels;
    a.norm = norm;
    a.scale_out = e.scale;
    a.parts = parts;
    if (parts > 1u) {
        a.error = e.error;
        a.max_spins = e.max_spins;
        a.slots = e.slots;
        a.done = e.slots + parts * e.chunks;
        return k14::launch_encode<k14::SmallOp::EncodeSpread>(a, ptrs, bf16, bits, stream);
    }
    a.error = clear_error ? e.error : nullptr;
    const uint32_t wpw_log2 = chunk_log2 > k14::kWaveLog2 ? chunk_log2 - k14::kWaveLog2 : 0u;
    if ((e.W << wpw_log2) > k14::kMaxWaves) return k14::launch_encode<k14::SmallOp::EncodeRounds>(a, ptrs, bf16, bits, stream);
    return k14::launch_encode<k14::SmallOp::EncodeAll>(a, ptrs, bf16, bits, stream);
}

bool small_applicable(Mode mode, const ChunkArgs& c) {
    if (!k14::small_size(c.chunk_log2) || c.no_rotate || c.range_in || c.out_bf16) return false;
    if (mode == Mode::Absmax) return k14::aligned16(c.in);
    if (mode == Mode::Encode) return k14::aligned16(c.in) && k14::aligned16(c.out);
    return mode == Mode::Decode && !c.sat && k14::aligned16(c.in) && (c.padded >> k14::kDecodeLog2) < 0x7FFFFFFFull;
}

// Coordinates of a workgroup (log2): 2^11 per wave, at least a chunk.  Four waves, and fewer where that spreads a
// short gradient over the CUs.  W: payloads that are summed (1 for stored sums).  The lines, in workgroups of four waves on 256
// CUs, and the decoder in us with one | two | four waves (chunk 2^10):
//   more than two for each CU     four
//   more than one                 four; 3 and 4 payloads two: 2.6 M coordinates, 4 at 4 bits 10.6 | 6.0 | 7.3, at 8 bits 11.2 | 7.0 | 8.4;
//                                 2 at 4 bits 10.8 | 7.0 | 6.2, 8 at 4 bits 11.1 | 7.8 | 7.6
//   more than one for two CUs     up to 4 payloads four: 2^21, 1 at 2 bits 6.4 | 7.3 | 6.1, 2 at 4 bits 6.7 | 7.0 | 6.1, 4 at 4
//                                 bits 6.4 | 6.1 | 6.5; more one: 1.3 M, 8 at 4 bits 5.6 | 7.2 | 6.4, 8 at 8 bits 6.5 | 8.0 | 7.2
//   more than one for four CUs    up to 4 payloads two: 2^20, 2 at 4 bits 6.0 | 5.9 | 6.2, 4 at 8 bits 6.7 | 5.9 | 6.2; more one: 8 at 4
//                                 bits 5.5 | 6.4 | 6.4, 16 at 4 bits 6.4 | 6.6 | 6.6
//   more than two                 one: 2^19, 2 at 4 bits 5.3 | 5.8 | 5.9, 16 at 8 bits 6.4 | 8.0 | 7.8
//   up to two (one payload: four) four with up to 8 payloads: every further XCD that takes part costs more than its waves
//                                 save (2^14, 1 at 2 bits 5.3 | 5.2 | 4.9, stored sums 4.9 | 4.6 | 4.5)
static uint32_t small_decode_log2(uint64_t padded, uint32_t l, uint32_t W) {
    const uint64_t groups = (padded + (1ull << k14::kDecodeLog2) - 1u) >> k14::kDecodeLog2, cus = device_cus();
    uint32_t log2 = k14::kDecodeLog2;
    if (groups > cus) {
        if (groups < 2u * cus && (W == 3u || W == 4u)) log2 = k14::kWaveLog2 + 1u;
    } else if (2u * groups > cus) {
        if (W > 4u) log2 = k14::kWaveLog2;
    } else if (4u * groups > cus) {
        log2 = W > 4u ? k14::kWaveLog2 : k14::kWaveLog2 + 1u;
    } else if (groups > (W == 1u ? 4u : 2u) || W > 8u) {
        log2 = k14::kWaveLog2;
    }
    return log2 > l ? log2 : l;
}

static hipError_t small_decode(k14::SmallDecodeArgs& a, const FusedPayloadPtrs& ptrs, int src, uint32_t bits, bool wide,
                               hipStream_t stream) {
    using namespace k14;
    const uint32_t log2 = small_decode_log2(a.padded, a.l, src == 0 ? a.W : 1u);
    const dim3 grid((uint32_t)((a.padded + (1ull << log2) - 1u) >> log2)), block(1u << (log2 - 5u));
    if (grid.x == 0) return hipSuccess;
#define THC_SMALL_DECODE(...) hipLaunchKernelGGL((small_decode_kernel<__VA_ARGS__>), grid, block, 0, stream, a, ptrs)
    if (src == 0) {
        if (wide) THC_SMALL_DECODE(0, 4, true);
        else if (bits == 2) THC_SMALL_DECODE(0, 2, false);
        else if (bits == 4) THC_SMALL_DECODE(0, 4, false);
        else if (stream_payloads(a.W, a.padded, true)) THC_SMALL_DECODE(0, 8, false, true);
        else THC_SMALL_DECODE(0, 8, false);
    } else if (src == 1) {
        if (bits == 2) THC_SMALL_DECODE(1, 2, false);
        else if (bits == 4) THC_SMALL_DECODE(1, 4, false);
        else THC_SMALL_DECODE(1, 8, false);
    } else {
        if (bits == 2) THC_SMALL_DECODE(2, 2, false);
        else if (bits == 4) THC_SMALL_DECODE(2, 4, false);
        else THC_SMALL_DECODE(2, 8, false);
    }
#undef THC_SMALL_DECODE
    return hipGetLastError();
}

hipError_t launch_small(Mode mode, const ChunkArgs& c, hipStream_t stream) {
    if (c.padded == 0) return hipSuccess;
    if (mode == Mode::Decode) {
        k14::SmallDecodeArgs d{c.n, c.padded, c.chunk_log2, c.W, c.key0, c.key1, c.inv_sqrt_c, c.scale_in, c.in, nullptr,
                               static_cast<float*>(c.out)};
        return small_decode(d, FusedPayloadPtrs{}, (int)c.sum_bytes, c.bits, false, stream);
    }
    k14::SmallArgs a{};
    a.n = c.n;
    a.padded = c.padded;
    a.l = c.chunk_log2;
    a.W = 1;
    a.worker0 = c.worker;
    a.key0 = c.key0;
    a.key1 = c.key1;
    a.levels = c.levels;
    a.norm = c.inv_sqrt_c;
    FusedWorkerPtrs ptrs{};
    ptrs.grad[0] = c.in;
    if (mode == Mode::Absmax) {
        a.scale_out = static_cast<float*>(c.out);
        return k14::launch_encode<k14::SmallOp::Absmax>(a, ptrs, c.in_bf16 != 0u, 4, stream);
    }
    ptrs.payload[0] = static_cast<uint8_t*>(c.out);
    a.scale_in = c.scale_in;
    a.scale_out = c.scale_out;
    if (c.scale_in) return k14::launch_encode<k14::SmallOp::EncodeOnto>(a, ptrs, c.in_bf16 != 0u, c.bits, stream);
    return k14::launch_encode<k14::SmallOp::EncodeAll>(a, ptrs, c.in_bf16 != 0u, c.bits, stream);
}

bool small_aggregate_decode_applicable(uint32_t W, uint32_t chunk_log2, uint32_t bits, uint64_t padded) {
    return k14::small_size(chunk_log2) && aggregate_decode_fused_applicable(W, 14, bits) &&
           (padded >> k14::kDecodeLog2) < 0x7FFFFFFFull;
}

hipError_t launch_small_aggregate_decode(const AggDecodeArgs& e, const FusedPayloadPtrs& ptrs, uint32_t chunk_log2,
                                         float norm, uint32_t bits, hipStream_t stream) {
    k14::SmallDecodeArgs d{e.n, e.chunks << chunk_log2, chunk_log2, e.W, e.key0, e.key1, norm, e.scale, nullptr, e.sums,
                           e.out};
    return small_decode(d, ptrs, 0, bits, bits == 4u && e.W * 15u > 255u, stream);
}

}  // namespace thc
