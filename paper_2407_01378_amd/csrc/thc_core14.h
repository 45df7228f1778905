// Device building blocks of the chunk-2^14 kernels: one workgroup of 512 threads (8
// waves) rotates one chunk held 32 coordinates per thread.  Butterfly stages run in
// stride order 1, 2, 4, ..., 8192, every stage one fp32 add and one fp32 subtract per
// pair, so results are bit-identical to the stage-by-stage definition; between the
// three register-resident groups of stages (5 + 5 + 4) the chunk is re-shuffled through
// LDS with the conflict-free maps of thc_layout14.h, and once more into the layout the
// consumer wants (32 consecutive coordinates per thread for the quantizer, 4 per lane
// for coalesced fp32 stores).
#pragma once

#include <type_traits>

#include "thc_device.h"
#include "thc_lanes.h"
#include "thc_layout14.h"

#pragma clang fp contract(off)

namespace thc {
namespace k14 {

constexpr int kThreads = 512;
constexpr int kChunkLog2 = 14;
constexpr int kChunk = 1 << kChunkLog2;
constexpr int kRegs = 32;                 // coordinates per thread
constexpr float kInvSqrtC = 0.0078125f;   // 2^-7, exact

// Wave priorities (s_setprio) by phase.  Two workgroups share a CU; a wave inside the
// rotation alternates short bursts of arithmetic with LDS exchanges and barriers, while
// the phase after the rotation (quantize and pack, or scale and store) is one long run of
// independent arithmetic.  Letting the rotation go first keeps its LDS and barrier
// latencies off the critical path and leaves the long run to fill the gaps; measured on
// the encode kernel this is worth 9 %.
constexpr int kPrioRotateEarly = 1;   // stages before the second exchange
constexpr int kPrioRotateLate = 2;    // stages after it
constexpr int kPrioExchange = 3;      // issuing LDS stores / loads of an exchange
constexpr int kPrioTail = 0;          // everything after the last exchange
// The memory-bound decode kernels run every phase at the default priority (PRIO = false):
// there the same scheme delays the next item's loads and costs 15 %.
template <bool PRIO, int LEVEL>
__device__ __forceinline__ void set_prio() {
    if constexpr (PRIO) __builtin_amdgcn_s_setprio(LEVEL);
}

struct alignas(16) SignTable {
    uint32_t sgn[kChunk / 32];   // sign diagonal of a chunk, bit (i mod 32) of word i / 32
    uint32_t sgx[kChunk / 32];   // the same words with even bits gathered in the low half,
                                 // odd bits in the high half (for bf16 pairs)
};
struct alignas(16) Shared {
    float xb[kChunk];            // exchange buffer, 64 KB
    SignTable sign[2];           // persistent kernels fill the next chunk's table ahead of time
    float red[8];                // one slot per wave for workgroup-wide reductions
};

// Butterflies on register-index bits [LO, HI): v[i], v[i+h] <- v[i] + v[i+h], v[i] - v[i+h].
template <int LO, int HI>
__device__ __forceinline__ void butterflies(float (&v)[kRegs]) {
#pragma unroll
    for (int b = LO; b < HI; ++b) {
        const int h = 1 << b;
#pragma unroll
        for (int i = 0; i < kRegs; ++i) {
            if ((i & h) == 0) {
                const float lo = v[i], hi = v[i + h];
                v[i] = lo + hi;
                v[i + h] = lo - hi;
            }
        }
    }
}

// Even bits of x to the low half, odd bits to the high half (bit 2p -> p, 2p+1 -> 16+p).
__device__ __forceinline__ uint32_t unshuffle_bits(uint32_t x) {
    uint32_t t;
    t = (x ^ (x >> 1)) & 0x22222222u; x ^= t ^ (t << 1);
    t = (x ^ (x >> 2)) & 0x0C0C0C0Cu; x ^= t ^ (t << 2);
    t = (x ^ (x >> 4)) & 0x00F000F0u; x ^= t ^ (t << 4);
    t = (x ^ (x >> 8)) & 0x0000FF00u; x ^= t ^ (t << 8);
    return x;
}

// 128 threads (two waves; which two is chosen by `turn`, so that persistent kernels can
// spread this work over the SIMDs from item to item) compute the 16384 sign bits of the
// chunk that starts at coordinate g0 (a multiple of 16384).  SGN / SGX select the forms
// the caller will read.  Needs a barrier before use.
template <bool SGN, bool SGX>
__device__ __forceinline__ void fill_sign_table(SignTable& tab, uint64_t g0, uint32_t key0,
                                                uint32_t key1, uint32_t t, uint32_t turn = 0u) {
    if ((t >> 7) == (turn & 3u)) {
        const uint32_t b = t & 127u;
        const u32x4 s = sign_block((g0 >> 7) + b, key0, key1);
        if (SGN) *reinterpret_cast<uint4*>(&tab.sgn[4 * b]) = make_uint4(s.w[0], s.w[1], s.w[2], s.w[3]);
        if (SGX)
            *reinterpret_cast<uint4*>(&tab.sgx[4 * b]) =
                make_uint4(unshuffle_bits(s.w[0]), unshuffle_bits(s.w[1]), unshuffle_bits(s.w[2]),
                           unshuffle_bits(s.w[3]));
    }
}

// ---------------------------------------------------------------- input -> layout L1
// Raw 16-byte units of a chunk in load order.  Coalesced order: thread t, round j holds
// unit 512 j + t, and the chunk passes through LDS to reach layout L1.  Direct order:
// thread t holds units UNITS t + j, its own 32 consecutive coordinates (layout L1 at
// once; every load instruction of a wave then touches UNITS times as many cache lines,
// each of which the wave's other loads hit again in the vector cache).
template <int UNITS>  // 4 for bf16, 8 for fp32
struct Raw {
    uint4 u[UNITS];
};

// Coalesced loads of one chunk.  `valid` = number of coordinates of this chunk that
// exist (1..16384); the rest read as zero.  ELEM = bytes per coordinate.
template <int UNITS, int ELEM, bool DIRECT = false>
__device__ __forceinline__ void load_raw(Raw<UNITS>& raw, const void* chunk_ptr, uint32_t valid,
                                         uint32_t t) {
    constexpr uint32_t kPerUnit = 16 / ELEM;
    const uint4* src = static_cast<const uint4*>(chunk_ptr);
    if (valid == (uint32_t)kChunk) {
#pragma unroll
        for (int j = 0; j < UNITS; ++j) raw.u[j] = src[DIRECT ? UNITS * t + j : j * kThreads + t];
    } else {
#pragma unroll
        for (int j = 0; j < UNITS; ++j) {
            const uint32_t unit = DIRECT ? UNITS * t + j : j * kThreads + t;
            const uint32_t first = unit * kPerUnit;
            uint4 q = make_uint4(0u, 0u, 0u, 0u);
            if (first + kPerUnit <= valid) {
                q = src[unit];
            } else if (first < valid) {
                uint32_t w[4] = {0u, 0u, 0u, 0u};
                if (ELEM == 2) {
                    const uint16_t* p = static_cast<const uint16_t*>(chunk_ptr) + first;
                    for (uint32_t e = 0; first + e < valid; ++e) w[e >> 1] |= (uint32_t)p[e] << (16 * (e & 1));
                } else {
                    const uint32_t* p = static_cast<const uint32_t*>(chunk_ptr) + first;
                    for (uint32_t e = 0; first + e < valid; ++e) w[e] = p[e];
                }
                q = make_uint4(w[0], w[1], w[2], w[3]);
            }
            raw.u[j] = q;
        }
    }
}

template <int UNITS>
__device__ __forceinline__ void raw_to_lds(Shared& sh, const Raw<UNITS>& raw, uint32_t t) {
    uint4* dst = reinterpret_cast<uint4*>(sh.xb) + lay14::e0_store_unit(t, 0, UNITS);
#pragma unroll
    for (int j = 0; j < UNITS; ++j) dst[j * kThreads] = raw.u[j];
}

// The thread's 32 consecutive coordinates as UNITS 16-byte units -> fp32 registers
// (layout L1): widens bf16 and applies the sign diagonal when SIGNED.
// sx: the thread's sign bits, bf16: even bits in the low half, odd bits in the high half.
template <int UNITS, bool SIGNED>
__device__ __forceinline__ void units_to_l1(uint32_t sx, const uint4 (&unit)[UNITS], float (&v)[kRegs]) {
    if (UNITS == 4) {  // bf16: 8 coordinates per unit, two per dword
#pragma unroll
        for (int k = 0; k < UNITS; ++k) {
            const uint32_t w[4] = {unit[k].x, unit[k].y, unit[k].z, unit[k].w};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int pair = 4 * k + d;  // coordinates 2 pair, 2 pair + 1
                uint32_t x = w[d];
                // sign bits of the pair sit at bits `pair` and 16 + `pair` of sx
                if (SIGNED) x = xor_masked(x, pair == 15 ? sx : (sx << (15 - pair)), 0x80008000u);
                v[2 * pair] = __uint_as_float(x << 16);
                v[2 * pair + 1] = __uint_as_float(x & 0xFFFF0000u);
            }
        }
    } else {  // fp32: 4 coordinates per unit
#pragma unroll
        for (int k = 0; k < UNITS; ++k) {
            const uint32_t w[4] = {unit[k].x, unit[k].y, unit[k].z, unit[k].w};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int r = 4 * k + d;
                uint32_t x = w[d];
                if (SIGNED) x = xor_masked(x, r == 31 ? sx : (sx << (31 - r)), 0x80000000u);
                v[r] = __uint_as_float(x);
            }
        }
    }
}
template <int UNITS, bool SIGNED>
__device__ __forceinline__ void units_to_l1(const SignTable& tab, const uint4 (&unit)[UNITS],
                                            float (&v)[kRegs], uint32_t t) {
    units_to_l1<UNITS, SIGNED>(SIGNED ? (UNITS == 4 ? tab.sgx[t] : tab.sgn[t]) : 0u, unit, v);
}

// Reads this thread's 32 consecutive coordinates back from the buffer (after raw_to_lds
// and a barrier) into layout L1.
template <int UNITS, bool SIGNED>
__device__ __forceinline__ void lds_to_l1(const Shared& sh, const SignTable& tab, float (&v)[kRegs],
                                          uint32_t t) {
    const uint4* src = reinterpret_cast<const uint4*>(sh.xb);
    uint4 unit[UNITS];
#pragma unroll
    for (int k = 0; k < UNITS; ++k) unit[k] = src[lay14::e0_load_unit(t, k, UNITS)];
    units_to_l1<UNITS, SIGNED>(tab, unit, v, t);
}

// ------------------------------------------------------------------ LDS exchanges
__device__ __forceinline__ void x1_store(Shared& sh, const float (&v)[kRegs], uint32_t lane, uint32_t wave) {
    float* reg = sh.xb + wave * 2048;
#pragma unroll
    for (int q = 0; q < 8; ++q)
        *reinterpret_cast<float4*>(reg + lay14::x1_store(lane, q)) =
            make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
}
__device__ __forceinline__ void x1_load(const Shared& sh, float (&v)[kRegs], uint32_t lane, uint32_t wave) {
    const float* reg = sh.xb + wave * 2048;
#pragma unroll
    for (int r = 0; r < kRegs; ++r) v[r] = reg[lay14::x1_load(lane, r)];
}
__device__ __forceinline__ void x2_store(Shared& sh, const float (&v)[kRegs], uint32_t lane, uint32_t wave) {
#pragma unroll
    for (int q = 0; q < 8; ++q)
        *reinterpret_cast<float4*>(sh.xb + lay14::x2_store(wave, lane, q)) =
            make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
}
__device__ __forceinline__ void x2_load(const Shared& sh, float (&v)[kRegs], uint32_t lane, uint32_t wave) {
#pragma unroll
    for (int r = 0; r < kRegs; ++r) v[r] = sh.xb[lay14::x2_load(wave, lane, r)];
}
__device__ __forceinline__ void x3e_store(Shared& sh, const float (&v)[kRegs], uint32_t lane, uint32_t wave) {
#pragma unroll
    for (int r = 0; r < kRegs; ++r) sh.xb[lay14::x3e_store(wave, lane, r)] = v[r];
}
__device__ __forceinline__ void x3e_load(const Shared& sh, float (&v)[kRegs], uint32_t lane, uint32_t wave) {
    const float4* units = reinterpret_cast<const float4*>(sh.xb);   // unit-indexed: provably 16-byte aligned
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float4 f = units[lay14::x3e_load_unit(wave, lane, q)];
        v[4 * q] = f.x;
        v[4 * q + 1] = f.y;
        v[4 * q + 2] = f.z;
        v[4 * q + 3] = f.w;
    }
}
__device__ __forceinline__ void x3d_store(Shared& sh, const float (&v)[kRegs], uint32_t lane, uint32_t wave) {
#pragma unroll
    for (int r = 0; r < kRegs; ++r) sh.xb[lay14::x3d_store(wave, lane, r)] = v[r];
}
__device__ __forceinline__ void x3d_load(const Shared& sh, float (&v)[kRegs], uint32_t lane, uint32_t wave) {
    const float4* units = reinterpret_cast<const float4*>(sh.xb);   // unit-indexed: provably 16-byte aligned
#pragma unroll
    for (int h = 0; h < 8; ++h) {
        const float4 f = units[lay14::x3d_load_unit(wave, lane, h)];
        v[4 * h] = f.x;
        v[4 * h + 1] = f.y;
        v[4 * h + 2] = f.z;
        v[4 * h + 3] = f.w;
    }
}

// Two waves trade half of their registers through LDS: the upper half of the one against the
// lower half of the other, so that register bit 4 and the bit in which the waves' numbers differ
// change places.  `upper`: this wave has the bit set; `mine` / `theirs`: 4 KB per wave, which are still being read on
// return.
__device__ __forceinline__ void trade_halves(float (&v)[kRegs], float4* mine, const float4* theirs, bool upper,
                                             uint32_t lane) {
    // (the empty assembly statements differ, so the two branches are not merged into one that picks
    // its registers by address, which would put v into memory)
    if (upper) {
        asm volatile("; upper wave" ::: "memory");
#pragma unroll
        for (int q = 0; q < 4; ++q) mine[q * 64 + lane] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        asm volatile("; upper wave sent" ::: "memory");
    } else {
        asm volatile("; lower wave" ::: "memory");
#pragma unroll
        for (int q = 0; q < 4; ++q)
            mine[q * 64 + lane] = make_float4(v[16 + 4 * q], v[17 + 4 * q], v[18 + 4 * q], v[19 + 4 * q]);
        asm volatile("; lower wave sent" ::: "memory");
    }
    __syncthreads();
    if (upper) {
        asm volatile("; upper wave" ::: "memory");
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 f = theirs[q * 64 + lane];
            v[4 * q] = f.x;
            v[4 * q + 1] = f.y;
            v[4 * q + 2] = f.z;
            v[4 * q + 3] = f.w;
        }
        asm volatile("; upper wave has" ::: "memory");
    } else {
        asm volatile("; lower wave" ::: "memory");
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 f = theirs[q * 64 + lane];
            v[16 + 4 * q] = f.x;
            v[17 + 4 * q] = f.y;
            v[18 + 4 * q] = f.z;
            v[19 + 4 * q] = f.w;
        }
        asm volatile("; lower wave has" ::: "memory");
    }
}

// Stages 0..13 on a chunk that sits in layout L1 in v; result (unnormalised H_c x) in
// layout L3.  Starts with a barrier (every thread is past its earlier reads of the
// buffer); the buffer is still being read when it returns.
template <bool PRIO>
__device__ __forceinline__ void rotate_l1_to_l3(Shared& sh, float (&v)[kRegs], uint32_t lane,
                                                uint32_t wave) {
    set_prio<PRIO, kPrioRotateEarly>();
    butterflies<0, 5>(v);          // strides 1..16
    __syncthreads();
    // the first exchange stays inside each wave's own 8 KB of the buffer, and a wave's
    // LDS accesses execute in order: no barrier between its stores and loads
    set_prio<PRIO, kPrioExchange>();
    x1_store(sh, v, lane, wave);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    x1_load(sh, v, lane, wave);
    set_prio<PRIO, kPrioRotateEarly>();
    butterflies<0, 5>(v);          // strides 32..512
    __syncthreads();
    set_prio<PRIO, kPrioExchange>();
    x2_store(sh, v, lane, wave);
    __syncthreads();
    x2_load(sh, v, lane, wave);
    set_prio<PRIO, kPrioRotateLate>();
    butterflies<1, 5>(v);          // strides 1024..8192 (register bit 0 is i9, already done)
}

// The same rotation from layout L1 with the lanes of each wave permuted (thread 64 wave + lane owns the
// 32 coordinates of block 64 wave + block_of_lane(lane)): stages 5..8 run between the lanes, so the
// chunk passes LDS once on the way to layout L3.  The exchange uses the map of the last one (X3e) in the
// opposite direction: a wave stores to its own 8 KB, a thread of layout L3 reads 32 words which it alone
// then rewrites in X3e, and X3e's readers take back exactly what they stored here.  So the whole
// item needs two barriers, one behind each set of stores, where the maps X1, X2, X3e needed five.
// On return a value is negated where its coordinate's bits i5..i8 have odd parity (odd_parity4).
__device__ __forceinline__ bool odd_parity4(uint32_t x) { return (0x6996u >> (x & 15u)) & 1u; }
template <bool PRIO>
__device__ __forceinline__ void rotate_lanes_to_l3(Shared& sh, float (&v)[kRegs], uint32_t lane, uint32_t block,
                                                   uint32_t wave) {
    set_prio<PRIO, kPrioRotateEarly>();
    butterflies<0, 5>(v);          // strides 1..16
    lanes::lane_stage<0>(v, (block & 1u) ? -1.0f : 1.0f);   // strides 32..256
    lanes::lane_stage<1>(v, (block & 2u) ? -1.0f : 1.0f);
    lanes::lane_stage<2>(v, (block & 4u) ? -1.0f : 1.0f);
    lanes::lane_stage<3>(v, (block & 8u) ? -1.0f : 1.0f);
    set_prio<PRIO, kPrioExchange>();
    float4* units = reinterpret_cast<float4*>(sh.xb);
#pragma unroll
    for (int q = 0; q < 8; ++q)
        units[lay14::x3e_load_unit(wave, block, q)] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRegs; ++r) v[r] = sh.xb[lay14::x3e_store(wave, lane, r)];
    set_prio<PRIO, kPrioRotateLate>();
    butterflies<0, 5>(v);          // strides 512..8192
}
// L3 -> L4e with permuted lanes, behind rotate_lanes_to_l3 (one barrier); v then holds the 32 coordinates
// of the thread's block.
template <bool PRIO>
__device__ __forceinline__ void l3_to_l4e_lanes(Shared& sh, float (&v)[kRegs], uint32_t lane, uint32_t block, uint32_t wave) {
    set_prio<PRIO, kPrioExchange>();
    x3e_store(sh, v, lane, wave);
    __syncthreads();
    x3e_load(sh, v, block, wave);
    set_prio<PRIO, kPrioTail>();
}

// A rotation without anything hung into it (see below).
struct NoHook {
    template <int K>
    __device__ __forceinline__ void at() {}
};

// The decoders' rotation, from layout L1 with permuted lanes straight to layout L4d: stages 5..8 between
// lanes, 9 and 10 behind register swaps (thc_lanes.h), so that a wave finishes its 2^11 coordinates by
// itself, one exchange of 128-bit accesses (X4d), and the last three stages in the layout of the stores.
// A chunk crosses LDS once, where the maps X1, X2, X3d take it through three times, with 32-bit accesses on
// one side of each: what a single chunk's chain waits for (decoder of 8 workers x 50257 coordinates, 4 chunks:
// 9.0 -> 6.1 us; 7 M coordinates, 433 chunks, u16 sums: 10.4 -> 9.2 us; large decodes are bound by memory).
// The caller's buffer is free (every wave is past a barrier behind its last reads); it is still being read on return.
// On return a value is negated where its coordinate's bits i5..i8 have odd parity: in layout L4d that is the same
// for all values of a thread (l4d_negated).
// hook.at<K>() is called at three points that are some hundred clocks apart (K = 0 in front of the first stage,
// 1 behind the lane stages, 2 behind the barrier): a persistent kernel hangs the next item's global loads there.
template <class Hook>
__device__ __forceinline__ void rotate_lanes_to_l4d(Shared& sh, float (&v)[kRegs], uint32_t lane, uint32_t block,
                                                    uint32_t wave, Hook& hook) {
    hook.template at<0>();
    butterflies<0, 5>(v);          // strides 1..16
    lanes::lane_stage<0>(v, (block & 1u) ? -1.0f : 1.0f);   // strides 32..256
    lanes::lane_stage<1>(v, (block & 2u) ? -1.0f : 1.0f);
    lanes::lane_stage<2>(v, (block & 4u) ? -1.0f : 1.0f);
    lanes::lane_stage<3>(v, (block & 8u) ? -1.0f : 1.0f);
    hook.template at<1>();
    lanes::swap_top_register_bit<16>(v);
    butterflies<4, 5>(v);          // stride 512
    lanes::swap_top_register_bit<32>(v);
    butterflies<4, 5>(v);          // stride 1024
    float4* units = reinterpret_cast<float4*>(sh.xb);
#pragma unroll
    for (int q = 0; q < 8; ++q)
        units[lay14::x4d_store_unit(wave, lane, q)] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    __syncthreads();
    hook.template at<2>();
#pragma unroll
    for (int h = 0; h < 8; ++h) {
        const float4 f = units[lay14::x4d_load_unit(wave, lane, h)];
        v[4 * h] = f.x;
        v[4 * h + 1] = f.y;
        v[4 * h + 2] = f.z;
        v[4 * h + 3] = f.w;
    }
    butterflies<2, 5>(v);          // strides 2048..8192
}
// Whether the values of a thread of layout L4d (lane = i2..i7, wave = i8..i10) come negated.
__device__ __forceinline__ bool l4d_negated(uint32_t lane, uint32_t wave) {
    return odd_parity4((lane >> 3) | ((wave & 1u) << 3));
}

// max |v| over this thread's registers, then over the wave.
__device__ __forceinline__ float wave_absmax(const float (&v)[kRegs]) {
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < kRegs; i += 2)
        asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(m), "v"(v[i]), "v"(v[i + 1]));
    // m >= 0: floats of one sign order like their bit patterns
    return __uint_as_float(wave_umax(__float_as_uint(m)));
}

// max |v| over the whole chunk (every thread returns it).  Two barriers.
__device__ __forceinline__ float chunk_absmax(Shared& sh, const float (&v)[kRegs], uint32_t lane,
                                              uint32_t wave) {
    float m = wave_absmax(v);
    if (lane == 0) sh.red[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(fmaxf(sh.red[0], sh.red[1]), fmaxf(sh.red[2], sh.red[3])),
              fmaxf(fmaxf(sh.red[4], sh.red[5]), fmaxf(sh.red[6], sh.red[7])));
    __syncthreads();
    return m;
}

// (min, max) of v over the whole chunk (every thread returns both).  Two barriers.
struct MinMax {
    float lo, hi;
};
__device__ __forceinline__ MinMax chunk_minmax(Shared& sh, const float (&v)[kRegs], uint32_t lane,
                                               uint32_t wave) {
    float lo = v[0], hi = v[0];
#pragma unroll
    for (int i = 1; i < kRegs; ++i) {
        lo = fminf(lo, v[i]);
        hi = fmaxf(hi, v[i]);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, o, 64));
        hi = fmaxf(hi, __shfl_xor(hi, o, 64));
    }
    float* red_lo = reinterpret_cast<float*>(sh.sign[1].sgn);   // second table: free in one-chunk kernels
    if (lane == 0) {
        sh.red[wave] = hi;
        red_lo[wave] = lo;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        hi = fmaxf(hi, sh.red[k]);
        lo = fminf(lo, red_lo[k]);
    }
    __syncthreads();
    return MinMax{lo, hi};
}

// An end of a rotated chunk's range, from the unnormalised extreme.  An exact zero counts as +0: its
// sign would depend on the order of the partners in the last subtraction that gave it (the lane
// exchanges undo a negation, which turns +0 into -0), and the range is the same bit for bit in all
// forms of the call.
__device__ __forceinline__ float rotated_end(float x) { return (x + 0.0f) * kInvSqrtC; }

// (min, max) over this thread's registers.
__device__ __forceinline__ MinMax thread_minmax(const float (&v)[kRegs]) {
    float lo = v[0], hi = v[0];
#pragma unroll
    for (int i = 1; i < kRegs; ++i) {
        lo = fminf(lo, v[i]);
        hi = fmaxf(hi, v[i]);
    }
    return MinMax{lo, hi};
}

// Order-preserving map of floats onto unsigned words that are never zero for anything
// but a NaN (in the words workgroups exchange, zero means "not published yet"):
// x <= y  <=>  order_key(x) <= order_key(y).
__device__ __forceinline__ uint32_t order_key(float x) {
    const uint32_t b = __float_as_uint(x);
    const uint32_t k = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    return k != 0u ? k : 1u;
}
__device__ __forceinline__ float order_value(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// L3 -> L4d: v[4 h + e] is coordinate 2048 h + 4 t + e.
template <bool PRIO>
__device__ __forceinline__ void l3_to_l4d(Shared& sh, float (&v)[kRegs], uint32_t lane, uint32_t wave) {
    __syncthreads();
    set_prio<PRIO, kPrioExchange>();
    x3d_store(sh, v, lane, wave);
    __syncthreads();
    x3d_load(sh, v, lane, wave);
    set_prio<PRIO, kPrioTail>();
}

// --------------------------------------------------------------------- quantizer
// Stochastic rounding of the L4e-resident chunk onto a grid of L + 1 points, packed.
// v holds the UNNORMALISED rotation; y = v * 2^-7.  For one coordinate
//     c   = fma(float(r), 2^-8, base)          exact; r the coordinate's random byte
//     t   = fma(y - sub, mul, c)               ONE rounding (y - sub is rounded first when RANGED)
//     idx = floor(t)   (clamped to L when CLAMP)
// Symmetric grid on [-s, s]:  sub unused, mul = L / (2 s), base = L/2 + 2^-9, so that
//     t = y * inv + L/2 + (r + 0.5) / 256.
// Min/max grid on [lo, hi] (RANGED):  sub = lo, mul = L / (hi - lo), base = 2^-9.
//   g        global index of the thread's first coordinate
//   CLAMP    false only when the range is the chunk's own: the symmetric grid with s the
//            largest |y| of the chunk (then 0 < t < L + 1 for every coordinate: |y * inv| <=
//            L/2 (1 + 2^-24) and 2^-9 <= c - L/2 <= 255.5 / 256), or the min/max grid with
//            lo and hi the chunk's extremes (fl(y - lo) <= fl(hi - lo) = width, and width *
//            fl(L / width) <= L (1 + 2^-24), so t < L + 255.5/256 + L 2^-24 < L + 1); the
//            minimum with L never binds.  Both bounds need mul finite: the callers set mul = 0
//            for a range below kMinRange, which then gives t = c.  A range handed in by a
//            caller keeps the clamp.
//   FOLD     y = v * 2^-7 is not formed; mul already carries the factor 2^-7 and sub is given
//            in v's units (v - 2^7 lo = 2^7 (y - lo), rounded alike).  Exact as long
//            as the power of two moves nothing into the subnormal range or past the largest
//            float: the callers fold only for 2^-100 <= s <= 2^100.
// Packing: float -> integer conversion writes its result straight into one byte of a
// 32-bit register (sub-dword destination select), so 32 conversions leave 8 registers of 4
// index bytes each and no shift-or per coordinate; register m holds, in byte i, the index
// of coordinate (32 / BITS) * (m / kSub) ... chosen so that the payload word is
//     8 bits:  register d itself                         (bytes = coordinates 4d .. 4d+3)
//     4 bits:  A_d | B_d << 4                            (A: even, B: odd coordinates of 8d .. 8d+7)
//     2 bits:  R_d0 | R_d1 << 2 | R_d2 << 4 | R_d3 << 6  (R_dm byte i = coordinate 16d + 4i + m)
template <int BYTE, bool FIRST>
__device__ __forceinline__ void cvt_into_byte(uint32_t& acc, float tt) {
    static_assert(BYTE >= 0 && BYTE < 4, "byte index");
    if constexpr (FIRST) {   // writes the byte, zeroes the rest of the register
        if constexpr (BYTE == 0) asm("v_cvt_u32_f32_sdwa %0, %1 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD" : "=v"(acc) : "v"(tt));
        if constexpr (BYTE == 1) asm("v_cvt_u32_f32_sdwa %0, %1 dst_sel:BYTE_1 dst_unused:UNUSED_PAD src0_sel:DWORD" : "=v"(acc) : "v"(tt));
        if constexpr (BYTE == 2) asm("v_cvt_u32_f32_sdwa %0, %1 dst_sel:BYTE_2 dst_unused:UNUSED_PAD src0_sel:DWORD" : "=v"(acc) : "v"(tt));
        if constexpr (BYTE == 3) asm("v_cvt_u32_f32_sdwa %0, %1 dst_sel:BYTE_3 dst_unused:UNUSED_PAD src0_sel:DWORD" : "=v"(acc) : "v"(tt));
    } else {                 // writes the byte, keeps the rest
        if constexpr (BYTE == 0) asm("v_cvt_u32_f32_sdwa %0, %1 dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:DWORD" : "+v"(acc) : "v"(tt));
        if constexpr (BYTE == 1) asm("v_cvt_u32_f32_sdwa %0, %1 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD" : "+v"(acc) : "v"(tt));
        if constexpr (BYTE == 2) asm("v_cvt_u32_f32_sdwa %0, %1 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD" : "+v"(acc) : "v"(tt));
        if constexpr (BYTE == 3) asm("v_cvt_u32_f32_sdwa %0, %1 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD" : "+v"(acc) : "v"(tt));
    }
}

// One half of it: the 16 coordinates in registers 16 half .. 16 half + 15, whose block of the rounding
// stream is rb, into index bytes by[4 half .. 4 half + 3].
//   norm     factor from v to y where it is not folded
//   NEG      the lane holds the negated value where sgn = -1 (a lane exchange leaves it so): mul
//            (FOLD) or norm carries the sign already, and sgn itself is used only where v meets sub
template <int BITS, bool CLAMP, bool FOLD, bool RANGED, bool NEG = false>
__device__ __forceinline__ void quantize_drawn(const float (&v)[kRegs], int half, const u32x4& rb, float sub, float mul,
                                               float base, uint32_t L, uint32_t (&by)[8], float norm, float sgn) {
    constexpr int kSub = 8 / BITS;        // coordinates per payload byte: 1, 2, 4
    const float Lf = (float)L;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int r = 16 * half + e;
        float y = FOLD ? v[r] : v[r] * norm;
        if (RANGED) y = FOLD && NEG ? __builtin_fmaf(v[r], sgn, -sub) : y - sub;   // (one rounding either way)
        const uint32_t rnd = (rb.w[e >> 2] >> (8 * (e & 3))) & 0xFFu;
        const float c = __builtin_fmaf((float)rnd, 0x1p-8f, base);
        float tt = __builtin_fmaf(y, mul, c);            // tt >= 0: truncation = floor
        if (CLAMP) tt = fminf(tt, Lf);                   // floor(min(t, L)) = min(floor(t), L)
        // coordinate r sits in payload word d = r / (32 / BITS), at slot j = r % (32 / BITS);
        // its index goes to byte j / kSub of register kSub * d + j % kSub
        constexpr int kPerWord = 32 / BITS;
        const int d = r / kPerWord, j = r % kPerWord;
        const int m = kSub * d + j % kSub, byte = j / kSub;
        switch (byte) {
            case 0: cvt_into_byte<0, true>(by[m], tt); break;
            case 1: cvt_into_byte<1, false>(by[m], tt); break;
            case 2: cvt_into_byte<2, false>(by[m], tt); break;
            default: cvt_into_byte<3, false>(by[m], tt); break;
        }
    }
}
// The same with the block's number: it is drawn here.
template <int BITS, bool CLAMP, bool FOLD, bool RANGED, bool NEG = false>
__device__ __forceinline__ void quantize_half(const float (&v)[kRegs], int half, uint64_t blk, float sub, float mul,
                                              float base, uint32_t L, uint32_t worker, uint32_t key0, uint32_t key1,
                                              uint32_t (&by)[8], float norm = kInvSqrtC, float sgn = 1.0f) {
    quantize_drawn<BITS, CLAMP, FOLD, RANGED, NEG>(v, half, round_block(blk, worker, key0, key1), sub, mul, base, L, by, norm, sgn);
}
// A thread's two blocks of the rounding stream, drawn where the caller puts this: in front of what it waits for.
struct Drawn {
    u32x4 rb[2];
    __device__ __forceinline__ void draw(uint64_t g, uint32_t worker, uint32_t key0, uint32_t key1) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            rb[h] = round_block((g >> 4) + h, worker, key0, key1);
#pragma unroll
            for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(rb[h].w[i]));   // (not moved to where it is used)
        }
    }
};
// Index bytes -> payload words.
template <int BITS>
__device__ __forceinline__ void pack_bytes(const uint32_t (&by)[8], uint32_t (&pk)[BITS]) {
#pragma unroll
    for (int d = 0; d < BITS; ++d) {
        if constexpr (BITS == 8) pk[d] = by[d];
        if constexpr (BITS == 4) pk[d] = by[2 * d] | (by[2 * d + 1] << 4);
        if constexpr (BITS == 2)
            pk[d] = by[4 * d] | (by[4 * d + 1] << 2) | (by[4 * d + 2] << 4) | (by[4 * d + 3] << 6);
    }
}
// drawn: a pointer to a Drawn, or nullptr: the bytes are drawn here.  (A question of the type: asked of the value, it
// changed the registers of the persistent kernels too, and cost the batched one at 8 bits 19 operations.)
template <int BITS, bool CLAMP, bool FOLD, bool RANGED, bool NEG = false, class D = decltype(nullptr)>
__device__ __forceinline__ void quantize_pack(const float (&v)[kRegs], float sub, float mul, float base,
                                              uint32_t L, uint64_t g, uint32_t worker, uint32_t key0,
                                              uint32_t key1, uint32_t (&pk)[BITS], float norm = kInvSqrtC,
                                              float sgn = 1.0f, D drawn = nullptr) {
    uint32_t by[8];                       // index bytes; by[m] serves payload word m / kSub
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        if constexpr (!std::is_same_v<D, decltype(nullptr)>)
            quantize_drawn<BITS, CLAMP, FOLD, RANGED, NEG>(v, half, drawn->rb[half], sub, mul, base, L, by, norm, sgn);
        else
            quantize_half<BITS, CLAMP, FOLD, RANGED, NEG>(v, half, (g >> 4) + half, sub, mul, base, L, worker, key0, key1, by,
                                                          norm, sgn);
    }
    pack_bytes<BITS>(by, pk);
}

template <int BITS>
__device__ __forceinline__ void store_packed(const uint32_t (&pk)[BITS], uint8_t* dst) {
    if constexpr (BITS == 8) {
        reinterpret_cast<uint4*>(dst)[0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        reinterpret_cast<uint4*>(dst)[1] = make_uint4(pk[4], pk[5], pk[6], pk[7]);
    } else if constexpr (BITS == 4) {
        *reinterpret_cast<uint4*>(dst) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
    } else {
        *reinterpret_cast<uint2*>(dst) = make_uint2(pk[0], pk[1]);
    }
}

// Symmetric grid.  An all-zero chunk (s = 0; also one with 2 s < kMinRange) gets index 0 everywhere on the 2^BITS-point
// grid (L odd) and the centre index L/2 on the signed grid (L even).  Evaluation order by
// grid size (kSingleFmaMaxLevels): 2- and 4-bit grids t = fma(y, inv, L/2 + u); 8-bit
// grids t = fma(y + s, inv, u), which is the ranged form with sub = -s.  The clamp stays
// dead there too when s is the chunk's largest magnitude: 0 <= y + s <= 2 s, and
// 2 s * inv <= L (1 + 2^-24), so t < L + 255.5/256 + L 2^-24 < L + 1.
// NEG: the thread's values are negated where sgn = -1 (see rotate_lanes_to_l3); t: its block of 32.
template <int BITS, bool CLAMP, bool NEG = false, class D = decltype(nullptr)>
__device__ __forceinline__ void quantize_store(const float (&v)[kRegs], float s, uint32_t L, uint64_t g0,
                                               uint32_t worker, uint32_t key0, uint32_t key1,
                                               uint8_t* payload, uint32_t t, float sgn = 1.0f,
                                               D drawn = nullptr) {
    constexpr bool kOffset = ((1u << BITS) - 2u) > kSingleFmaMaxLevels;   // both grids of this width
    const float two = s + s;
    const bool ranged = two >= kMinRange;   // false: an all-zero chunk, or one too small for L / two
    const float inv = ranged ? (float)L / two : 0.0f;
    const float centre = (ranged ? !kOffset : (L & 1u) == 0u) ? 0.5f * (float)L : 0.0f;
    const float base = centre + 0x1p-9f;   // exact
    const uint64_t g = g0 + (uint64_t)t * 32u;
    uint32_t pk[BITS];   // 32 coordinates * BITS bits = BITS dwords
    if (s >= 0x1p-100f && s <= 0x1p100f)   // the same for every thread of the workgroup
        quantize_pack<BITS, CLAMP, true, kOffset, NEG>(v, -128.0f * s, inv * (NEG && !kOffset ? kInvSqrtC * sgn : kInvSqrtC),
                                                       base, L, g, worker, key0, key1, pk, kInvSqrtC, sgn, drawn);
    else
        quantize_pack<BITS, CLAMP, false, kOffset, NEG>(v, -s, inv, base, L, g, worker, key0, key1, pk,
                                                        NEG ? kInvSqrtC * sgn : kInvSqrtC, sgn, drawn);
    store_packed<BITS>(pk, payload + (g * BITS) / 8u);
}

// Min/max grid: idx = floor((y - lo) * inv + u), inv = L / (hi - lo) (0 for a constant chunk
// and for one narrower than kMinRange).
// ROTATED false: v holds y itself (the unrotated, zero-padded gradient), not 2^7 y.
template <int BITS, bool ROTATED = true, bool CLAMP = true, class D = decltype(nullptr)>
__device__ __forceinline__ void quantize_store_range(const float (&v)[kRegs], float lo, float hi, uint32_t L,
                                                     uint64_t g0, uint32_t worker, uint32_t key0,
                                                     uint32_t key1, uint8_t* payload, uint32_t t,
                                                     float norm = kInvSqrtC, D drawn = nullptr) {
    const float width = hi - lo;
    const float inv = width >= kMinRange ? (float)L / width : 0.0f;
    const uint64_t g = g0 + (uint64_t)t * 32u;
    uint32_t pk[BITS];
    quantize_pack<BITS, CLAMP, !ROTATED, true>(v, lo, inv, 0x1p-9f, L, g, worker, key0, key1, pk, norm, 1.0f, drawn);
    store_packed<BITS>(pk, payload + (g * BITS) / 8u);
}

// Output side of the inverse rotation: x = D (v * norm), from layout L4d; the first `valid` coordinates
// of the chunk are stored.  norm: 2^-7, negative where the thread's values are negated (a pass of a longer
// rotation takes +-1: its normalisation is one multiplication at the very end).  The product
// is taken with + 0 added in the same rounding: an exact zero, which the lane exchanges leave as +0 in a
// negated thread too, stays the +0 that the stage's subtraction gives.
// The stores go through a buffer descriptor that ends behind the last coordinate (its range check is made
// for each dword): no ragged path, and the compiler knows how many stores are behind a load it waits for.
template <bool SIGNED = true>
__device__ __forceinline__ void store_signed_l4d(const SignTable& tab, const float (&v)[kRegs], float* out,
                                                 uint32_t valid, uint32_t t, float norm) {
    uint64_t addr = reinterpret_cast<uint64_t>(out);   // the same for every lane: in scalar registers
    addr = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(addr >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)addr);
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(addr), 0, (int)(valid * 4u), 0x00020000);
#pragma unroll
    for (int h = 0; h < 8; ++h) {
        const uint32_t i0 = h * 2048u + t * 4u;
        const uint32_t sb = SIGNED ? tab.sgn[i0 >> 5] >> (i0 & 31u) : 0u;   // bits 0..3: signs of the 4 coordinates
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[e] = __builtin_fmaf(v[4 * h + e], norm, 0.0f);
            if (SIGNED) x[e] = __uint_as_float(xor_masked(__float_as_uint(x[e]), sb << (31 - e), 0x80000000u));
        }
        const u32x4_vec q = {__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])};
        __builtin_amdgcn_raw_buffer_store_b128(q, rsrc, i0 * 4u, 0, kStreaming);
    }
}

}  // namespace k14
}  // namespace thc
