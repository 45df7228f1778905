// TopK Chunked (TopKC): per-chunk squared norms in half precision, their sum over workers,
// selection of the J chunks with the largest sums, and the fp16 sum of the selected chunks
// ("Our proposed improvement: Chunks" of the paper's TopK case study).  Everything here is
// a streaming scan; the only part that is not elementwise is the selection, a two-pass
// radix select over the 16-bit keys followed by an ordered compaction.
#include <hip/hip_fp16.h>

#include "thc_device.h"
#include "thc_internal.h"
#include "topkc_search.h"

#pragma clang fp contract(off)

namespace thc {
namespace {

// fp32 -> fp16 bits, round to nearest even (subnormals kept, overflow to inf).
__device__ __forceinline__ uint32_t f32_to_f16_bits(float x) {
    return (uint32_t)__half_as_ushort(__float2half_rn(x));
}
__device__ __forceinline__ float f16_bits_to_f32(uint32_t h) {
    return __half2float(__ushort_as_half((unsigned short)h));
}
// fp16 + fp16 -> fp16: the fp32 sum of two fp16 numbers is exact, so one rounding.
__device__ __forceinline__ uint32_t add_f16_bits(uint32_t a, uint32_t b) {
    return f32_to_f16_bits(f16_bits_to_f32(a) + f16_bits_to_f32(b));
}

// 8 consecutive coordinates starting at g (a multiple of 8), widened to fp32; zeros past n.
template <bool BF16>
__device__ __forceinline__ void load8(const void* grad, uint64_t g, uint64_t n, float (&x)[8]) {
    if (g + 8u <= n) {
        if (BF16) {
            const uint4 q = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(grad) + g);
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                x[2 * d] = __uint_as_float(w[d] << 16);
                x[2 * d + 1] = __uint_as_float(w[d] & 0xFFFF0000u);
            }
        } else {
            const float4 a = *reinterpret_cast<const float4*>(static_cast<const float*>(grad) + g);
            const float4 b = *reinterpret_cast<const float4*>(static_cast<const float*>(grad) + g + 4);
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
            x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v = 0.0f;
            if (g + e < n)
                v = BF16 ? bf16_bits_to_float(static_cast<const uint16_t*>(grad)[g + e])
                         : static_cast<const float*>(grad)[g + e];
            x[e] = v;
        }
    }
}

template <bool BF16>
__device__ __forceinline__ void raw8(const void* grad, uint64_t g, uint64_t n, uint4 (&q)[2]) {
    // whole groups only; BF16: one 16-byte unit, fp32: two
    if (BF16) {
        q[0] = load_last_use(reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(grad) + g));
    } else {
        q[0] = load_last_use(reinterpret_cast<const uint4*>(static_cast<const float*>(grad) + g));
        q[1] = load_last_use(reinterpret_cast<const uint4*>(static_cast<const float*>(grad) + g + 4));
    }
}
template <bool BF16>
__device__ __forceinline__ void widen8(const uint4 (&q)[2], float (&x)[8]) {
    if (BF16) {
        const uint32_t w[4] = {q[0].x, q[0].y, q[0].z, q[0].w};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            x[2 * d] = __uint_as_float(w[d] << 16);
            x[2 * d + 1] = __uint_as_float(w[d] & 0xFFFF0000u);
        }
    } else {
        const uint32_t w[8] = {q[0].x, q[0].y, q[0].z, q[0].w, q[1].x, q[1].y, q[1].z, q[1].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(w[e]);
    }
}
// The value of the lane N above, within a row of 16 lanes (0 past the row's end).
template <int N>
__device__ __forceinline__ float from_lane_above(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x100 + N, 0xF, 0xF, true));
}
// Adds up over the chunk's lanes, adjacent pairs first; the sum is whole in the chunk's lowest
// lane, the only one that stores it.
__device__ __forceinline__ void norm_of_group(const float (&x)[8], uint64_t k, uint64_t groups,
                                              uint32_t lanes_per_chunk, uint32_t lanes_log2, uint16_t* norms) {
    float s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = x[e] * x[e];
    float t = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    if (lanes_per_chunk > 1u) t = t + from_lane_above<1>(t);
    if (lanes_per_chunk > 2u) t = t + from_lane_above<2>(t);
    if (lanes_per_chunk > 4u) t = t + from_lane_above<4>(t);
    if (lanes_per_chunk > 8u) t = t + from_lane_above<8>(t);
    if (lanes_per_chunk > 16u) t = t + __shfl_down(t, 16, 64);
    if (lanes_per_chunk > 32u) t = t + __shfl_down(t, 32, 64);
    if (k < groups && (k & (uint64_t)(lanes_per_chunk - 1u)) == 0)
        norms[k >> lanes_log2] = (uint16_t)f32_to_f16_bits(t);
}

// Squared norm of every chunk of C = 8 * lanes_per_chunk coordinates: squares in fp32,
// summed as a balanced tree over adjacent pairs (inside the thread, then across lanes
// 1, 2, 4, ... apart), rounded to fp16.  Bound by reading the gradient once, so what counts is
// bytes in flight: a workgroup takes a tile of kNormUnroll x 256 groups of 8 coordinates, and a
// thread loads its kNormUnroll groups (256 apart: whole lines per wave) before it uses any.
// Measured (launches of a round, every gradient another): 108 M bf16, C = 64: 44.8 -> 34.4 us (6.3 TB/s)
// against one group per thread and trip of a grid-wide stride, which kept one load in flight up to
// 200 M coordinates; on one buffer again and again: 7 M bf16 8.9 -> 3.5 us, 1 G bf16 345 -> 323 us.  Two groups per
// thread: 331 us at 1 G, eight: 329 us, and 5 % slower than four on fp32.
constexpr int kNormUnroll = 4;
template <bool BF16>
__global__ __launch_bounds__(256) void norms_kernel(const void* grad, uint64_t n, uint32_t lanes_per_chunk,
                                                    uint32_t lanes_log2, uint64_t groups, uint64_t tiles,
                                                    uint16_t* norms) {
    constexpr uint64_t kTile = kNormUnroll * 256u;
    const uint64_t whole = n / 8u;   // groups below this are complete
    for (uint64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint64_t k = tile * kTile + threadIdx.x;
        if ((tile + 1u) * kTile <= whole) {
            uint4 q[kNormUnroll][2];
#pragma unroll
            for (int u = 0; u < kNormUnroll; ++u) raw8<BF16>(grad, (k + u * 256u) * 8u, n, q[u]);
#pragma unroll
            for (int u = 0; u < kNormUnroll; ++u) {
                float x[8];
                widen8<BF16>(q[u], x);
                norm_of_group(x, k + u * 256u, groups, lanes_per_chunk, lanes_log2, norms);
            }
        } else {   // the gradient ends in this tile: the element-wise loader; all lanes stay for the exchanges
#pragma unroll 1
            for (int u = 0; u < kNormUnroll; ++u) {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = 0.0f;
                if (k + u * 256u < groups) load8<BF16>(grad, (k + u * 256u) * 8u, n, x);
                norm_of_group(x, k + u * 256u, groups, lanes_per_chunk, lanes_log2, norms);
            }
        }
    }
}

// s_p = fp16 sum over workers, in worker order, of norms_all[w * P + p].
__global__ __launch_bounds__(256) void sum_norms_kernel(const uint16_t* norms_all, uint32_t W, uint64_t P,
                                                        uint16_t* s) {
    const uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    uint32_t acc = norms_all[p];
    for (uint32_t w = 1; w < W; ++w) acc = add_f16_bits(acc, norms_all[(uint64_t)w * P + p]);
    s[p] = (uint16_t)acc;
}
// The same, four chunks per thread through 8-byte loads (P a multiple of 4, both arrays
// 8-byte aligned: then every worker's row is too).
__global__ __launch_bounds__(256) void sum_norms4_kernel(const uint16_t* norms_all, uint32_t W, uint64_t P,
                                                         uint16_t* s) {
    const uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;   // chunks 4 q .. 4 q + 3
    if (q * 4u >= P) return;
    uint32_t acc[4];
    for (uint32_t w = 0; w < W; ++w) {
        const uint2 x = load_last_use(reinterpret_cast<const uint2*>(norms_all + (uint64_t)w * P) + q);
        const uint32_t h[4] = {x.x & 0xFFFFu, x.x >> 16, x.y & 0xFFFFu, x.y >> 16};
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = w == 0 ? h[e] : add_f16_bits(acc[e], h[e]);
    }
    reinterpret_cast<uint2*>(s)[q] = make_uint2(acc[0] | (acc[1] << 16), acc[2] | (acc[3] << 16));
}

// ---- selection -----------------------------------------------------------------------------
// Workspace words: [0,256) histogram of the keys' high bytes, [256,512) histogram of the
// low bytes inside the threshold bucket, [512] threshold bucket, [513] still to take
// inside it, [514] threshold key T, [515] how many keys equal to T are taken, then per
// segment of kSegment keys the pair (keys above T, keys equal to T).
// The keys are a few MB, so a launch and a chain of dependent loads cost more than the bytes: the
// walk over a histogram is done by every wave of the kernel that needs its result (256 words from
// L2) and block 0 notes the result for the kernels after it.
// Measured, five launches in the place of nine: 2048 keys 28.9 -> 13.7 us, 1.7 M 38.0 -> 30.7, 20.3 M 174 -> 106.
constexpr uint32_t kSegment = 2048;
constexpr uint32_t kHdr = 516;

// One wave walks a 256-bin histogram from the top: the largest bin b whose count together
// with the counts above it reaches `want` (bin 0 if none does), and the count above it.
// Lane i holds bins 4 i .. 4 i + 3.  All 64 lanes call it; all get the result.
struct Found {
    uint32_t bin, above;
};
__device__ __forceinline__ Found find_bin(const uint32_t* hist, uint32_t want) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t* bins = hist + 4u * lane;   // (the workspace is only 4-byte aligned)
    const uint4 c = make_uint4(bins[0], bins[1], bins[2], bins[3]);
    const uint32_t tot = c.x + c.y + c.z + c.w;
    uint32_t suf = tot;   // -> this lane's bins and all above them
#pragma unroll
    for (uint32_t o = 1; o < 64u; o <<= 1) {
        const uint32_t y = __shfl_down(suf, o, 64);
        if (lane + o < 64u) suf += y;
    }
    const uint32_t s4 = suf - tot;   // everything above bin 4 lane + 3
    const uint32_t s3 = s4 + c.w, s2 = s3 + c.z, s1 = s2 + c.y, s0 = s1 + c.x;
    int best = -1;
    uint32_t above = 0;
    if (s3 >= want) { best = 3; above = s4; }
    else if (s2 >= want) { best = 2; above = s3; }
    else if (s1 >= want) { best = 1; above = s2; }
    else if (s0 >= want) { best = 0; above = s1; }
    const unsigned long long found = __ballot(best >= 0);
    Found r = {0u, (uint32_t)__shfl(s1, 0, 64)};   // nothing reaches `want`: bin 0, as the walk from the top would end
    if (found != 0ull) {
        const int winner = 63 - __builtin_clzll(found);
        r.bin = 4u * (uint32_t)winner + (uint32_t)__shfl(best, winner, 64);
        r.above = __shfl(above, winner, 64);
    }
    return r;
}

// PASS 0: histogram of key >> 8.  PASS 1: of key & 255 among keys in the bucket in which the
// J-th largest key lies (block 0 notes the bucket and how many to take inside it).
// VEC (s 16-byte aligned): a thread takes 8 consecutive keys per load and adds runs of equal
// bins with one LDS atomic each (norms that underflow to zero, or lie in one bucket, come in
// runs); the keys past the last whole group of 8 are left to the first block.
// A round's keys lie in a few tens of bins: kCopies histograms, one per lane modulo kCopies and
// an odd number of words apart, keep the lanes of a wave off one LDS word.
constexpr uint32_t kCopies = 16;
template <int PASS, bool VEC>
__global__ __launch_bounds__(256) void hist_kernel(const uint16_t* s, uint64_t P, uint32_t J, uint32_t* ws) {
    __shared__ uint32_t copies[kCopies * 257u];
    for (uint32_t i = threadIdx.x; i < kCopies * 257u; i += 256u) copies[i] = 0u;
    uint32_t bucket = 0u;
    if (PASS == 1) {
        const Found f = find_bin(ws, J);
        bucket = f.bin;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            ws[512] = f.bin;
            ws[513] = J - f.above;   // still to take inside the bucket (>= 1)
        }
    }
    __syncthreads();
    uint32_t* h = copies + (threadIdx.x & (kCopies - 1u)) * 257u;
    auto bin_of = [&](uint32_t key) -> int {
        if (PASS == 0) return (int)(key >> 8);
        return (key >> 8) == bucket ? (int)(key & 255u) : -1;
    };
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    if (VEC) {
        const uint64_t groups = P / 8u;
        for (uint64_t g = tid; g < groups; g += stride) {
            const uint4 q = reinterpret_cast<const uint4*>(s)[g];
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
            int cur = -1;
            uint32_t cnt = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int b = bin_of((w[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
                if (b != cur) {
                    if (cur >= 0) atomicAdd(&h[cur], cnt);
                    cur = b;
                    cnt = 1u;
                } else {
                    ++cnt;
                }
            }
            if (cur >= 0) atomicAdd(&h[cur], cnt);
        }
        if (blockIdx.x == 0 && groups * 8u + threadIdx.x < P) {   // fewer than 8 keys
            const int b = bin_of(s[groups * 8u + threadIdx.x]);
            if (b >= 0) atomicAdd(&h[b], 1u);
        }
    } else {
        for (uint64_t p = tid; p < P; p += stride) {
            const int b = bin_of(s[p]);
            if (b >= 0) atomicAdd(&h[b], 1u);
        }
    }
    __syncthreads();
    uint32_t c = 0u;
#pragma unroll
    for (uint32_t i = 0; i < kCopies; ++i) c += copies[i * 257u + threadIdx.x];
    if (c) atomicAdd(&ws[256 * PASS + threadIdx.x], c);
}

// The 8 keys of segment `base` that belong to this thread, index order = (thread, k) order, two to a word;
// past the end: 0 (and not counted by the callers).
template <bool VEC>
__device__ __forceinline__ void load_keys(const uint16_t* s, uint64_t P, uint64_t base, uint32_t (&w)[4]) {
    const uint64_t p = base + 8u * threadIdx.x;
    if (VEC && p + 8u <= P) {
        const uint4 q = *reinterpret_cast<const uint4*>(s + p);
        w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
    } else {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t lo = p + 2 * d < P ? s[p + 2 * d] : 0u;
            const uint32_t hi = p + 2 * d + 1 < P ? s[p + 2 * d + 1] : 0u;
            w[d] = lo | (hi << 16);
        }
    }
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// Finds the threshold key (block 0 notes it and how many of its equals to take) and counts, per
// segment, the keys above it and equal to it.
template <bool VEC>
__global__ __launch_bounds__(256) void seg_count_kernel(const uint16_t* s, uint64_t P, uint32_t* ws) {
    __shared__ uint32_t wave_cnt[4];
    const uint64_t base = (uint64_t)blockIdx.x * kSegment;
    uint32_t w[4];
    load_keys<VEC>(s, P, base, w);
    const uint32_t want = ws[513];
    const Found f = find_bin(ws + 256, want);
    const uint32_t T = (ws[512] << 8) | f.bin;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ws[514] = T;
        ws[515] = want - f.above;   // keys equal to T that are taken (>= 1)
    }
    uint32_t both = 0;   // above | equal << 16, at most kSegment each
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t key = (w[k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
        if (base + 8u * threadIdx.x + k < P) both += (key > T ? 1u : 0u) + (key == T ? 0x10000u : 0u);
    }
    both = wave_sum(both);
    if ((threadIdx.x & 63u) == 0) wave_cnt[threadIdx.x >> 6] = both;
    __syncthreads();
    if (threadIdx.x == 0) {
        both = wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3];
        ws[kHdr + 2u * blockIdx.x] = both & 0xFFFFu;
        ws[kHdr + 2u * blockIdx.x + 1u] = both >> 16;
    }
}

// Exclusive scan of the per-segment pairs, one workgroup: for more than kOwnPrefix segments.
__global__ __launch_bounds__(1024) void seg_scan_kernel(uint32_t* ws, uint32_t segments) {
    __shared__ uint32_t wave_tot[2][16];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t per = (segments + 1023u) / 1024u;
    const uint32_t lo = t * per, hi = min(lo + per, segments);
    uint32_t a = 0, e = 0;
    for (uint32_t i = lo; i < hi; ++i) {
        a += ws[kHdr + 2u * i];
        e += ws[kHdr + 2u * i + 1u];
    }
    // exclusive scan of the 1024 thread totals: inclusive inside each wave by lane shifts,
    // then the totals of the waves before this one
    uint32_t ia = a, ie = e;
    for (uint32_t o = 1; o < 64u; o <<= 1) {
        const uint32_t ya = __shfl_up(ia, o, 64), ye = __shfl_up(ie, o, 64);
        if (lane >= o) {
            ia += ya;
            ie += ye;
        }
    }
    if (lane == 63u) {
        wave_tot[0][wave] = ia;
        wave_tot[1][wave] = ie;
    }
    __syncthreads();
    uint32_t oa = 0, oe = 0;
    for (uint32_t w = 0; w < wave; ++w) {
        oa += wave_tot[0][w];
        oe += wave_tot[1][w];
    }
    a = oa + ia - a;
    e = oe + ie - e;
    for (uint32_t i = lo; i < hi; ++i) {
        const uint32_t xa = ws[kHdr + 2u * i], xe = ws[kHdr + 2u * i + 1u];
        ws[kHdr + 2u * i] = a;
        ws[kHdr + 2u * i + 1u] = e;
        a += xa;
        e += xe;
    }
}

// Ordered compaction: chunk p is selected if its key is above T, or equal to T with fewer
// than `need` equal keys before it; its place is (#above before) + min(#equal before, need).
// SCANNED: the pairs are scanned already; else a workgroup adds up those before its own.  Up to
// kOwnPrefix segments (4 M keys) that is at most 16 loads per thread, out of L2, in the place of a launch.
constexpr uint32_t kOwnPrefix = 2048;
template <bool VEC, bool SCANNED>
__global__ __launch_bounds__(256) void write_indices_kernel(const uint16_t* s, uint64_t P, const uint32_t* ws,
                                                            uint32_t* indices) {
    __shared__ uint32_t wave_tot[2][4], wave_pre[2][4];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * kSegment;
    uint32_t w[4];
    load_keys<VEC>(s, P, base, w);
    const uint32_t T = ws[514], need = ws[515];
    uint32_t above_before = 0, equal_before = 0;
    if (SCANNED) {
        above_before = ws[kHdr + 2u * blockIdx.x];
        equal_before = ws[kHdr + 2u * blockIdx.x + 1u];
    } else {
        uint32_t pa = 0, pe = 0;
        for (uint32_t i = threadIdx.x; i < blockIdx.x; i += 256u) {
            pa += ws[kHdr + 2u * i];
            pe += ws[kHdr + 2u * i + 1u];
        }
        pa = wave_sum(pa);
        pe = wave_sum(pe);
        if (lane == 0) {
            wave_pre[0][wave] = pa;
            wave_pre[1][wave] = pe;
        }
    }
    // this thread's keys above T and equal to it, a bit each
    uint32_t is_above = 0, is_equal = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t key = (w[k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
        if (base + 8u * threadIdx.x + k < P) {
            is_above |= (key > T ? 1u : 0u) << k;
            is_equal |= (key == T ? 1u : 0u) << k;
        }
    }
    // exclusive scan of (above | equal << 16) over the 256 threads: at most kSegment each
    const uint32_t own = (uint32_t)__popc(is_above) | ((uint32_t)__popc(is_equal) << 16);
    uint32_t inc = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(inc, o, 64);
        if (lane >= (uint32_t)o) inc += u;
    }
    if (lane == 63) {
        wave_tot[0][wave] = inc & 0xFFFFu;
        wave_tot[1][wave] = inc >> 16;
    }
    __syncthreads();
    if (!SCANNED) {
        above_before = wave_pre[0][0] + wave_pre[0][1] + wave_pre[0][2] + wave_pre[0][3];
        equal_before = wave_pre[1][0] + wave_pre[1][1] + wave_pre[1][2] + wave_pre[1][3];
    }
    for (uint32_t v = 0; v < wave; ++v) {
        above_before += wave_tot[0][v];
        equal_before += wave_tot[1][v];
    }
    above_before += (inc - own) & 0xFFFFu;
    equal_before += (inc - own) >> 16;
    for (uint32_t left = is_above | is_equal; left != 0u; left &= left - 1u) {
        const uint32_t bit = left & (0u - left);
        const bool eq = (is_equal & bit) != 0u;
        if (!eq || equal_before < need)
            indices[above_before + min(equal_before, need)] =
                (uint32_t)(base + 8u * threadIdx.x) + (uint32_t)__builtin_ctz(bit);
        if (eq) ++equal_before; else ++above_before;
    }
}

// All of the selection in one workgroup: thread t holds keys 8 G t .. 8 G t + 8 G - 1 in registers, both histograms and
// the scan lie in LDS, and nothing goes through the workspace.  For few keys the selection is five launches' time, 15 us
// and more where the host issues them one by one; for many, one CU's LDS atomics.  A round of 8 workers, C = 64 and 32, five launches |
// this, us: 2048 and 4096 keys 60.8 | 44.4, 63.4 | 42.8, 16384 57.6 | 47.1, 32768 62.5 | 54.9 and 62.8 | 52.6, 65536 63.6 | 71.8,
// which is where the line comes from.
constexpr uint32_t kOneThreads = 1024;
constexpr uint64_t kOneKeys = 32768;
template <int G>
__global__ __launch_bounds__(kOneThreads) void select_one_kernel(const uint16_t* s, uint32_t P, uint32_t J,
                                                                 uint32_t* indices) {
    __shared__ uint32_t copies[kCopies * 257u];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t wave_tot[2][kOneThreads / 64u];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t first = t * (8u * G);
    const bool vec = (reinterpret_cast<uintptr_t>(s) & 15u) == 0;
    uint32_t w[G][4];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t p = first + 8u * g;
        if (vec && p + 8u <= P) {
            const uint4 q = *reinterpret_cast<const uint4*>(s + p);
            w[g][0] = q.x; w[g][1] = q.y; w[g][2] = q.z; w[g][3] = q.w;
        } else {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t lo = p + 2 * d < P ? s[p + 2 * d] : 0u;
                const uint32_t hi = p + 2 * d + 1 < P ? s[p + 2 * d + 1] : 0u;
                w[g][d] = lo | (hi << 16);
            }
        }
    }
    const uint32_t mine = first < P ? (P - first < 8u * G ? P - first : 8u * G) : 0u;   // keys of this thread
    auto key_of = [&](int g, int e) { return (w[g][e >> 1] >> (16 * (e & 1))) & 0xFFFFu; };
    uint32_t want = J, bucket = 0u, T = 0u;
    uint32_t* h = copies + (t & (kCopies - 1u)) * 257u;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        for (uint32_t i = t; i < kCopies * 257u; i += kOneThreads) copies[i] = 0u;
        __syncthreads();
        int cur = -1;
        uint32_t cnt = 0;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t key = key_of(g, e);
                int b = pass == 0 ? (int)(key >> 8) : (key >> 8) == bucket ? (int)(key & 255u) : -1;
                if (8u * g + e >= mine) b = -1;
                if (b != cur) {
                    if (cur >= 0) atomicAdd(&h[cur], cnt);
                    cur = b;
                    cnt = 1u;
                } else {
                    ++cnt;
                }
            }
        if (cur >= 0) atomicAdd(&h[cur], cnt);
        __syncthreads();
        if (t < 256u) {
            uint32_t c = 0u;
#pragma unroll
            for (uint32_t i = 0; i < kCopies; ++i) c += copies[i * 257u + t];
            hist[t] = c;
        }
        __syncthreads();
        const Found f = find_bin(hist, want);
        want -= f.above;   // keys still to take in the bin (>= 1)
        if (pass == 0) bucket = f.bin;
        else T = (bucket << 8) | f.bin;
    }
    uint32_t above = 0, equal = 0;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (8u * g + e < mine) {
                above += key_of(g, e) > T ? 1u : 0u;
                equal += key_of(g, e) == T ? 1u : 0u;
            }
    uint32_t ia = above, ie = equal;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t ya = __shfl_up(ia, o, 64), ye = __shfl_up(ie, o, 64);
        if (lane >= (uint32_t)o) {
            ia += ya;
            ie += ye;
        }
    }
    if (lane == 63u) {
        wave_tot[0][wave] = ia;
        wave_tot[1][wave] = ie;
    }
    __syncthreads();
    uint32_t above_before = ia - above, equal_before = ie - equal;
    for (uint32_t v = 0; v < wave; ++v) {
        above_before += wave_tot[0][v];
        equal_before += wave_tot[1][v];
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (8u * g + e < mine) {
                const uint32_t key = key_of(g, e);
                if (key > T || (key == T && equal_before < want))
                    indices[above_before + min(equal_before, want)] = first + 8u * g + e;
                above_before += key > T ? 1u : 0u;
                equal_before += key == T ? 1u : 0u;
            }
}

// ---- selected chunks --------------------------------------------------------------------------
// values[j * C + e] = fp16 sum over workers, in worker order, of fp16(x_w[indices[j] * C + e]).
template <bool BF16>
__global__ __launch_bounds__(256) void gather_sum_kernel(const FusedWorkerPtrs ptrs, uint32_t W, uint64_t n,
                                                         uint32_t C, const uint32_t* indices, uint64_t threads,
                                                         uint16_t* values) {
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid >= threads) return;
    const uint64_t flat = tid * 8u;                 // position in the J x C value array
    const uint64_t j = flat / C;
    const uint32_t e0 = (uint32_t)(flat - j * C);
    const uint64_t g = (uint64_t)indices[j] * C + e0;
    uint32_t acc[8];
    for (uint32_t w = 0; w < W; ++w) {
        float x[8];
        load8<BF16>(ptrs.grad[w], g, n, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t h = f32_to_f16_bits(x[e]);
            acc[e] = w == 0 ? h : add_f16_bits(acc[e], h);
        }
    }
    *reinterpret_cast<uint4*>(values + flat) =
        make_uint4(acc[0] | (acc[1] << 16), acc[2] | (acc[3] << 16), acc[4] | (acc[5] << 16), acc[6] | (acc[7] << 16));
}

// out[indices[j] * C + e] = float(values[j * C + e]) / W  (out zeroed beforehand).
__global__ __launch_bounds__(256) void scatter_kernel(const uint16_t* values, const uint32_t* indices, uint32_t C,
                                                      uint32_t W, uint64_t n, uint64_t threads, float* out) {
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid >= threads) return;
    const uint64_t flat = tid * 8u;
    const uint64_t j = flat / C;
    const uint32_t e0 = (uint32_t)(flat - j * C);
    const uint64_t g = (uint64_t)indices[j] * C + e0;
    const uint4 q = *reinterpret_cast<const uint4*>(values + flat);
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    const float Wf = (float)W;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float v = f16_bits_to_f32((w[e >> 1] >> (16 * (e & 1))) & 0xFFFFu) / Wf;
        if (g + e < n) out[g + e] = v;
    }
}

// The dense estimate in ONE pass over the output: every coordinate is written exactly once,
// float(value) / W inside the selected chunks and 0 elsewhere.  `indices` is ascending, so a
// workgroup that owns a contiguous range of chunks searches for its first selected chunk
// (topkc_search.h) and then walks the list: per tile of kTileChunks chunks, thread t looks at
// indices[j + t] and, if that chunk lies in the tile, records its rank j + t for the
// chunk; no more than kTileChunks selected chunks can lie in a tile, so one look per thread
// sees them all.  `out` must be 16-byte aligned.
constexpr int kScatterThreads = 256;
constexpr int kTileChunks = kScatterThreads;
// Workgroups wanted, where the output has that many pieces of one 16-byte unit per thread: 2^20 coordinates, C = 64, as 64
// tiles 10.9 us of kernel, as 1024 pieces 4 (512 and 2048 pieces: the round 2 % slower for 2^17 .. 2^19 coordinates, the
// same above).
// The search by one wave, 64 entries at a time: with all 256 threads every workgroup read up to 1024 scattered entries, which
// costs launches of many small workgroups more than one round of reads fewer gains them; 8 coordinates to a chunk, halving by one
// thread | 256 | 64, us: 20 M outputs, a tenth selected 22.2 | 25.1 | 18.7, 7.1 M 11.0 | 12.0 | 9.7; all four waves, 64 each 21.0.
constexpr uint64_t kScatterGroups = 1024;
__global__ __launch_bounds__(kScatterThreads) void scatter_dense_kernel(
    const uint16_t* values, const uint32_t* indices, uint32_t J, uint32_t C, uint32_t W, uint64_t n, uint64_t P,
    uint64_t chunks_per_group, float* out) {
    __shared__ uint32_t rank[kTileChunks];
    __shared__ uint32_t first;
    const uint32_t t = threadIdx.x;
    const uint64_t begin = (uint64_t)blockIdx.x * chunks_per_group;
    if (begin >= P) return;
    const uint64_t end = begin + chunks_per_group < P ? begin + chunks_per_group : P;
    if (t < 64u) {   // the first wave searches for the first j with indices[j] >= begin
        SearchRange r = {0u, J};
        while (r.lo < r.hi) {
            const uint32_t step = r.step(64u);
            const uint64_t at = r.at(t, step);
            const bool below = at < r.hi && (uint64_t)indices[at] < begin;
            r.cut((uint32_t)__popcll(__ballot(below)), step);
        }
        if (t == 0u) first = r.lo;
    }
    __syncthreads();
    uint32_t j = first;
    const float Wf = (float)W;
    const uint32_t units_per_chunk = C / 4u;            // 16-byte units of fp32 output per chunk
    const uint32_t shift = 31u - (uint32_t)__builtin_clz(units_per_chunk);
    for (uint64_t c0 = begin; c0 < end; c0 += kTileChunks) {
        const uint64_t c1 = c0 + kTileChunks < end ? c0 + kTileChunks : end;
        rank[t] = kNotSelected;
        __syncthreads();
        const uint64_t cand = (uint64_t)j + t < (uint64_t)J ? (uint64_t)indices[j + t] : ~0ull;
        const bool inside = cand >= c0 && cand < c1;    // cand >= c0 whenever the list is ascending
        if (inside) rank[cand - c0] = j + t;
        j += (uint32_t)__syncthreads_count(inside);     // also orders the writes of rank before its reads
        const uint64_t unit0 = c0 * units_per_chunk;
        const uint64_t units = (c1 - c0) * units_per_chunk;
        for (uint64_t u = t; u < units; u += kScatterThreads) {
            const uint32_t lc = (uint32_t)(u >> shift);
            const uint32_t e0 = ((uint32_t)u & (units_per_chunk - 1u)) * 4u;
            const uint32_t place = rank[lc];
            float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (is_selected(place)) {
                const uint2 q = *reinterpret_cast<const uint2*>(values + (uint64_t)place * C + e0);
                x[0] = f16_bits_to_f32(q.x & 0xFFFFu) / Wf;
                x[1] = f16_bits_to_f32(q.x >> 16) / Wf;
                x[2] = f16_bits_to_f32(q.y & 0xFFFFu) / Wf;
                x[3] = f16_bits_to_f32(q.y >> 16) / Wf;
            }
            const uint64_t g = (unit0 + u) * 4u;
            if (g + 4u <= n) {
                store_streaming(out + g, x[0], x[1], x[2], x[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (g + e < n) out[g + e] = x[e];
            }
        }
        __syncthreads();                                // rank is rewritten by the next tile
    }
}

// Largest grid of the norm kernel, in blocks of 256 threads.
constexpr uint64_t kNormBlocks = 32768;

uint32_t blocks_for(uint64_t threads, uint32_t per_block) {
    return (uint32_t)((threads + per_block - 1) / per_block);
}

}  // namespace

hipError_t launch_topkc_norms(const void* grad, bool bf16, uint64_t n, uint32_t C, uint16_t* norms,
                              hipStream_t stream) {
    const uint64_t P = (n + C - 1) / C;
    const uint64_t threads = P * (C / 8u);
    if (threads == 0) return hipSuccess;
    const uint64_t tiles = (threads + kNormUnroll * 256u - 1) / (kNormUnroll * 256u);
    const dim3 grid((uint32_t)(tiles < kNormBlocks ? tiles : kNormBlocks)), block(256);
    const uint32_t lanes = C / 8u, lanes_log2 = 31u - (uint32_t)__builtin_clz(lanes);
    if (bf16)
        hipLaunchKernelGGL(norms_kernel<true>, grid, block, 0, stream, grad, n, lanes, lanes_log2, threads, tiles, norms);
    else
        hipLaunchKernelGGL(norms_kernel<false>, grid, block, 0, stream, grad, n, lanes, lanes_log2, threads, tiles, norms);
    return hipGetLastError();
}

hipError_t launch_topkc_sum_norms(const uint16_t* norms_all, uint32_t W, uint64_t P, uint16_t* s,
                                  hipStream_t stream) {
    if (P == 0) return hipSuccess;
    if (P % 4u == 0 && reinterpret_cast<uint64_t>(norms_all) % 8u == 0 && reinterpret_cast<uint64_t>(s) % 8u == 0)
        hipLaunchKernelGGL(sum_norms4_kernel, dim3(blocks_for(P / 4u, 256)), dim3(256), 0, stream, norms_all, W, P, s);
    else
        hipLaunchKernelGGL(sum_norms_kernel, dim3(blocks_for(P, 256)), dim3(256), 0, stream, norms_all, W, P, s);
    return hipGetLastError();
}

uint64_t topkc_select_workspace_words(uint64_t P) {
    return kHdr + 2u * ((P + kSegment - 1) / kSegment);
}

template <bool VEC>
static void select_kernels(const uint16_t* s, uint64_t P, uint32_t J, uint32_t* indices, uint32_t* ws,
                           uint32_t segments, hipStream_t stream) {
    uint32_t hb = blocks_for(P, 256 * 16);
    if (hb > 1024) hb = 1024;
    hipLaunchKernelGGL((hist_kernel<0, VEC>), dim3(hb), dim3(256), 0, stream, s, P, J, ws);
    hipLaunchKernelGGL((hist_kernel<1, VEC>), dim3(hb), dim3(256), 0, stream, s, P, J, ws);
    hipLaunchKernelGGL(seg_count_kernel<VEC>, dim3(segments), dim3(256), 0, stream, s, P, ws);
    if (segments <= kOwnPrefix) {
        hipLaunchKernelGGL((write_indices_kernel<VEC, false>), dim3(segments), dim3(256), 0, stream, s, P, ws, indices);
    } else {
        hipLaunchKernelGGL(seg_scan_kernel, dim3(1), dim3(1024), 0, stream, ws, segments);
        hipLaunchKernelGGL((write_indices_kernel<VEC, true>), dim3(segments), dim3(256), 0, stream, s, P, ws, indices);
    }
}

hipError_t launch_topkc_select(const uint16_t* s, uint64_t P, uint32_t J, uint32_t* indices, uint32_t* ws,
                               hipStream_t stream) {
    if (P <= kOneKeys) {
        const dim3 grid(1), block(kOneThreads);
        if (P <= 8u * kOneThreads) hipLaunchKernelGGL(select_one_kernel<1>, grid, block, 0, stream, s, (uint32_t)P, J, indices);
        else if (P <= 16u * kOneThreads) hipLaunchKernelGGL(select_one_kernel<2>, grid, block, 0, stream, s, (uint32_t)P, J, indices);
        else hipLaunchKernelGGL(select_one_kernel<4>, grid, block, 0, stream, s, (uint32_t)P, J, indices);
        return hipGetLastError();
    }
    const uint32_t segments = (uint32_t)((P + kSegment - 1) / kSegment);
    hipError_t e = launch_zero_words(ws, kHdr, stream);
    if (e != hipSuccess) return e;
    if ((reinterpret_cast<uintptr_t>(s) & 15u) == 0) select_kernels<true>(s, P, J, indices, ws, segments, stream);
    else select_kernels<false>(s, P, J, indices, ws, segments, stream);
    return hipGetLastError();
}

hipError_t launch_topkc_gather_sum(const FusedWorkerPtrs& ptrs, bool bf16, uint32_t W, uint64_t n, uint32_t C,
                                   const uint32_t* indices, uint32_t J, uint16_t* values, hipStream_t stream) {
    const uint64_t threads = (uint64_t)J * (C / 8u);
    if (threads == 0) return hipSuccess;
    const dim3 grid(blocks_for(threads, 256)), block(256);
    if (bf16)
        hipLaunchKernelGGL(gather_sum_kernel<true>, grid, block, 0, stream, ptrs, W, n, C, indices, threads, values);
    else
        hipLaunchKernelGGL(gather_sum_kernel<false>, grid, block, 0, stream, ptrs, W, n, C, indices, threads, values);
    return hipGetLastError();
}

hipError_t launch_topkc_scatter(const uint16_t* values, const uint32_t* indices, uint32_t J, uint32_t C,
                                uint32_t W, uint64_t n, float* out, hipStream_t stream) {
    const uint64_t P = (n + C - 1) / C;
    if (P == 0) return hipSuccess;
    if ((reinterpret_cast<uintptr_t>(out) & 15u) == 0) {
        // one pass: contiguous ranges of whole tiles, or of parts of one where the tiles are few
        const uint64_t tiles = (P + kTileChunks - 1) / kTileChunks;
        uint64_t groups = 16384u;   // (5.2 GB written: 2048 groups 1.37 ms, 4096 1.20, 16384 1.12, 32768 1.11)
        if (groups > tiles) groups = tiles;
        uint64_t chunks_per_group = (tiles + groups - 1) / groups * kTileChunks;
        while (chunks_per_group > 1024u / C && P / chunks_per_group < kScatterGroups) chunks_per_group >>= 1;
        groups = (P + chunks_per_group - 1) / chunks_per_group;
        hipLaunchKernelGGL(scatter_dense_kernel, dim3((uint32_t)groups), dim3(kScatterThreads), 0, stream, values,
                           indices, J, C, W, n, P, chunks_per_group, out);
        return hipGetLastError();
    }
    // an output that is only 4-byte aligned: fill, then scatter
    hipError_t e = launch_zero_words(reinterpret_cast<uint32_t*>(out), n, stream);
    if (e != hipSuccess) return e;
    const uint64_t threads = (uint64_t)J * (C / 8u);
    if (threads == 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_kernel, dim3(blocks_for(threads, 256)), dim3(256), 0, stream, values, indices, C,
                       W, n, threads, out);
    return hipGetLastError();
}

}  // namespace thc
