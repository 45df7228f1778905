// Full rotation (l' = l): the Hadamard transform of a whole gradient padded to 2^l
// coordinates, l > 14, as the paper's baseline for the partial rotation.  Stages run in
// the same order as everywhere else (stride 1, 2, 4, ..., 2^(l-1), every stage one
// separately rounded fp32 add and subtract), so results are bit-identical to the
// stage-by-stage definition:
//   stages 0..13    the chunk-2^14 kernels (thc_fast14.hip), data in registers and LDS
//                   (0..14 for 2^25 coordinates: thc_full15.hip)
//   the rest        "high passes" over the fp32 array in global memory, up to 11 stages per
//                   pass (this file), in place
// plus the steps of the quantizer on rotated data, which the partial-rotation path fuses into
// its rotation kernels: as elementwise kernels on stored values (range, encode, decode), and
// as variants of the last forward pass that keep only the range of its results, or quantize
// them once the shared scale is known, so that the rotated values are never stored.
#include "thc_core14.h"
#include "thc_internal.h"
#include "thc_lanes.h"
#include "thc_resident.h"

#pragma clang fp contract(off)

namespace thc {
namespace {

using k14::butterflies;
using k14::kRegs;

// One pass over stages [s0, s0 + M), 1 <= M <= 11, s0 >= 14.  A tile is 2^max(M, 6) "rows" of 32
// consecutive floats (16 for M = 11); row bit b < M is stage s0 + b, row bits M.. of a short pass
// extend the column index, so that it reads longer runs.  A thread holds 16 rows x 2 consecutive
// floats (a wave reads four whole 128-byte lines per load, eight halves for M = 11); the rows:
//   row bits 0..3   the slot of the thread's registers
//   row bits 4, 5   lane bits 4, 5 (M = 11: row bits 4..6 are lane bits 3..5): they change places
//                   with slot bit 3 by register swaps between lanes (thc_lanes.h), one after the other
//   the rest        the wave: it changes places with slot bits 0.. through LDS, once, the two
//                   floats of a pair in turn so that the buffer takes half the data
// So passes of up to 6 stages need neither LDS nor barriers: every wave streams by itself, and
// the others keep 32 waves per CU (64 registers, 64 KB of LDS per 16 waves, in the inverse's last pass of
// 9 stages 68), except for the inverse's last pass of 10 stages: 128 registers, 68 KB
// (the exchange and a sign word per row), 16 waves.  Bound by memory (8 bytes per coordinate in
// place, 4 for the range alone).  The shape before, 8 rows x 4 floats per thread, exchanged
// twice for every pass through 64 KB of LDS and reached 9 stages, so 2^25 coordinates took
// 14 + 6 + 5 stages, then 14 + 11: round of 8 workers x 25.6 M fp32 1366 -> 1021 us (15 + 10 since: 934 us).
struct HighPassArgs {
    float* data;        // 2^l floats, transformed in place (unless `out`)
    float* out;         // last pass of the inverse: x (n floats); else null
    uint64_t n;         // coordinates to write to `out`
    uint32_t s0;
    float factor;       // of the last pass
    uint32_t key0, key1;
    uint64_t tiles;
    uint32_t xcd_run_log2;   // see xcd_order
    uint64_t valid;     // floats of `data` that hold values, a multiple of 2^s0; what lies beyond
                        // reads as zero and is neither read nor, in a pass that is not the last,
                        // written (the zero padding behind the gradient is implied, pass after
                        // pass, until the last pass mixes it with everything)
    uint32_t* absmax;   // last forward pass: receives max |value written| by an unsigned atomic
                        // maximum (zeroed beforehand); may be null
    // last forward pass evaluated for the quantizer instead of being stored:
    const float* scale; // one float, shared by all workers
    uint32_t levels;    // largest grid index L
    uint32_t worker;
    uint8_t* payload;   // 2^l * bits / 8 bytes
};

// What a pass does with its results.
enum class Kind : int {
    InPlace = 0,       // written back to `data`
    InPlaceLast = 1,   // the same, times `factor`; keeps the largest magnitude if asked
    ToX = 2,           // inverse direction, last pass: sign diagonal, first n values to `out`
    RangeOnly = 3,     // forward direction, last pass: only their largest magnitude is kept
    Encode = 4         // forward direction, last pass: quantized and packed
};

// Shape of a pass of M stages: bits of the wave's number that are rows, and tiles and waves of a workgroup.
// Workgroups have up to 8 (M <= 6) or 16 waves and take neighbouring tiles where one tile needs fewer: the
// rows of a tile lie up to gigabytes apart, so the bytes a workgroup takes from each of them should be many
// (2^29 coordinates, passes of 8 and 7 stages: 6.23 ms with one tile per workgroup, 5.65 ms like this).
// A small array has too few tiles for that (2^20 coordinates: 512): there the launch groups fewer.
constexpr int wave_rows(int M) { return M == 11 ? 4 : M > 6 ? M - 6 : 0; }
constexpr int pass_tiles(int M) { return M <= 6 ? 8 : M <= 9 ? 16 >> wave_rows(M) : 1; }
constexpr int pass_waves(int M) { return pass_tiles(M) << wave_rows(M); }
// Lane bits that are columns (pairs of floats); the others are rows.
constexpr int column_bits(int M) { return M == 11 ? 3 : 4; }

// Row of slot s in a lane, before the stages ...
template <int M>
__device__ __forceinline__ uint32_t row_before(uint32_t s, uint32_t lane, uint32_t wave) {
    return s | ((lane >> column_bits(M)) << 4) | (wave << (4 + 6 - column_bits(M)));
}
// ... and after them: slot bit 3 has changed places with the lane's row bits, one after the other (as far
// as there are stages for them), slot bits 0.. with the wave's bits.  wave: 0 where waves are independent.
template <int M>
__device__ __forceinline__ uint32_t row_after(uint32_t s, uint32_t lane, uint32_t wave) {
    const uint32_t l4 = (lane >> 4) & 1u, l5 = (lane >> 5) & 1u, top = (s >> 3) & 1u;
    if constexpr (M <= 4) return s | (l4 << 4) | (l5 << 5);
    if constexpr (M == 11) return (s << 7) | (wave & 7u) | ((lane >> 3) << 3) | ((wave >> 3) << 6);
    if constexpr (M == 5) return (s & 7u) | (l4 << 3) | (top << 4) | (l5 << 5);
    constexpr uint32_t nw = (uint32_t)wave_rows(M), kTraded = (1u << nw) - 1u;
    const uint32_t mixed = (l4 << 3) | (l5 << 4);
    if constexpr (nw < 4) {
        return ((s & kTraded) << 6) | (s & 7u & ~kTraded) | (wave & kTraded) | mixed | (top << 5);
    } else {
        return (s << 6) | (wave & 7u) | mixed | ((wave >> 3) << 5);
    }
}

// Tile of a workgroup or wave by its place in the launch order: workgroups go to the eight XCDs in turn, and
// neighbouring tiles write neighbouring 16-byte pieces of the same payload lines, which should meet in one L2
// instead of leaving eight of them as partial lines.  This order gives each XCD runs of 2^run_log2 workgroups
// (xcd_run_log2).  (The tiles of a workgroup stay together.)
__device__ __forceinline__ uint64_t xcd_order(uint64_t place, uint32_t run_log2, uint32_t together) {
    const uint32_t log2 = 31u - (uint32_t)__builtin_clz(together);
    const uint64_t group = place >> log2, j = group >> 3;
    return ((((j >> run_log2) << (3u + run_log2)) | ((group & 7u) << run_log2) | (j & ((1ull << run_log2) - 1ull))) << log2) |
           (place & (together - 1u));
}
// Workgroups of such a run, of a launch of `groups` (a power of two).
//   a payload line's worth of tiles  all XCDs together then read one contiguous range of columns: 2^25 coordinates,
//                                    10 stages, 4 bits, 36 us (each XCD one contiguous eighth of the tiles
//                                    38.5, tiles in turn 44); 2^29, 7 stages, 2 bits 467 (eighths 481)
//   a contiguous eighth              where the chip holds the launch at once (512 workgroups; 2^24: a round of 308 us,
//                                    with runs 311); for passes of 11 stages, whose tiles are half lines of the array
//                                    (17 M coordinates, eight workers 752 us, with runs 772 and more); for up to 6
//                                    stages, where a workgroup of eight independent waves is a line's worth or half
//                                    of it already (2^26: 4 bits 43 us, with runs 48; 2 bits 42, with runs 56), and
//                                    for 7 at 2 bits (2^27: 118 and 121 us)
inline uint32_t xcd_run_log2(int M, int bits, uint64_t groups, uint32_t together) {
    if (groups < 16u) return 0u;   // (as launched)
    const uint32_t eighth = 60u - (uint32_t)__builtin_clzll(groups);
    if (M <= 6 || M == 11 || (M == 7 && bits == 2) || groups <= 512u) return eighth;
    const uint32_t line = bits == 8 ? 2u : bits == 4 ? 3u : 4u;   // tiles of a payload line (32 columns each)
    const uint32_t log2 = 31u - (uint32_t)__builtin_clz(together);
    const uint32_t run = line > log2 ? line - log2 : 0u;
    return run < eighth ? run : eighth;
}

// Where a tile lies.
template <int M>
struct Tile {
    static constexpr uint32_t kExt = M < 6 ? 6u - M : 0u;   // row bits that extend the column
    uint64_t block;   // first float of the 2^(s0 + M) block it belongs to
    uint64_t base;    // first float of its row 0
    uint32_t s0;
    __device__ __forceinline__ Tile(uint32_t stage0, uint64_t tile) : s0(stage0) {
        constexpr uint32_t kRowLog2 = (uint32_t)column_bits(M) + 1u + kExt;
        const uint32_t jb_bits = stage0 - kRowLog2;         // column blocks per 2^s0 run
        block = (tile >> jb_bits) << (stage0 + M);
        base = block + ((tile & ((1ull << jb_bits) - 1ull)) << kRowLog2);
    }
    __device__ __forceinline__ uint64_t row_start(uint32_t row) const {
        return base + ((uint64_t)(row & ((1u << M) - 1u)) << s0) + (uint64_t)((row >> M) * 32u);
    }
};

// The thread's 16 rows x 2 floats of a tile.
template <int M>
__device__ __forceinline__ void load_rows(const HighPassArgs& a, const Tile<M>& T, uint32_t lane, uint32_t wave,
                                          float2 (&raw)[16]) {
    const uint32_t jq = lane & ((1u << column_bits(M)) - 1u);
    // rows of the block that hold values (`valid` and the block are multiples of 2^s0)
    const uint64_t rows64 = a.valid > T.block ? (a.valid - T.block) >> T.s0 : 0u;
    const uint32_t rows = rows64 > (1ull << M) ? 1u << M : (uint32_t)rows64;
    const float* src = a.data + T.row_start(row_before<M>(0u, lane, wave)) + 2u * jq;
    if (rows == 1u << M) {
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const uint64_t off = ((uint64_t)(s & ((1 << M) - 1)) << T.s0) + (uint64_t)((s >> M) * 32);
            raw[s] = *reinterpret_cast<const float2*>(src + off);
        }
    } else {
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const uint64_t off = ((uint64_t)(s & ((1 << M) - 1)) << T.s0) + (uint64_t)((s >> M) * 32);
            raw[s] = make_float2(0.0f, 0.0f);
            if ((row_before<M>((uint32_t)s, lane, wave) & ((1u << M) - 1u)) < rows)
                raw[s] = *reinterpret_cast<const float2*>(src + off);
        }
    }
}

// The stages of the pass on one tile.  `xb`: the workgroup's buffer (M > 6), 16 floats per thread; it is
// free again at the end.
template <int M>
__device__ __forceinline__ void rotate_tile(float (&v)[kRegs], float* xb, uint32_t lane, uint32_t wave) {
    butterflies<1, (M < 4 ? M : 4) + 1>(v);   // (register bit 0 is the float of the pair, slot bits follow)
    if constexpr (M == 11) {
        lanes::swap_top_register_bit<8>(v);
        butterflies<4, 5>(v);
    }
    if constexpr (M > 4) {
        lanes::swap_top_register_bit<16>(v);
        butterflies<4, 5>(v);
    }
    if constexpr (M > 5) {
        lanes::swap_top_register_bit<32>(v);
        butterflies<4, 5>(v);
    }
    if constexpr (M > 6) {
        constexpr int nw = wave_rows(M), kW = 1 << nw, kHigh = 16 >> nw;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
#pragma unroll
            for (int s = 0; s < 16; ++s)
                xb[((((uint32_t)(s & (kW - 1)) * kW + wave) * kHigh) + (s >> nw)) * 64u + lane] = v[2 * s + e];
            __syncthreads();
#pragma unroll
            for (int s = 0; s < 16; ++s)
                v[2 * s + e] = xb[(((wave * kW + (uint32_t)(s & (kW - 1))) * kHigh) + (s >> nw)) * 64u + lane];
            __syncthreads();
        }
        butterflies<1, nw + 1>(v);
    }
}

// Waves per SIMD the registers must allow: 8 (64 registers), but 4 for the inverse's last pass of 10 stages,
// whose output addresses and sign words do not fit (44.8 us with the spills, 27.8 us without,
// 2^24 coordinates) and whose workgroup of 16 waves then has a CU to itself.
constexpr int pass_waves_per_simd(int M, Kind kind) { return kind == Kind::ToX && M >= 10 ? 4 : 8; }

template <int M, Kind KIND, int BITS>
__global__ __launch_bounds__(64 * pass_waves(M), pass_waves_per_simd(M, KIND)) void high_pass_kernel(const HighPassArgs a) {
    constexpr int kWaves = pass_waves(M);
    constexpr bool kIndependent = M <= 6;
    constexpr bool kRange = KIND == Kind::RangeOnly || KIND == Kind::InPlaceLast;
    // exchange of the stages (M > 6) and, inside each wave's 4 KB, of the quantizer's runs
    __shared__ float4 buf[(M > 6 || KIND == Kind::Encode) ? 256 * kWaves : 1];
    constexpr uint32_t kTiles = (uint32_t)pass_tiles(M), kTileWaves = (uint32_t)kWaves / kTiles;
    constexpr uint32_t kRows = M > 6 ? 1u << M : 64u;   // of a tile
    __shared__ uint32_t signs[KIND == Kind::ToX ? kRows * kTiles : 1];
    __shared__ uint32_t most[kWaves];
    const uint32_t t = threadIdx.x, lane0 = t & 63u;
    const uint32_t wave_all = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    const uint32_t mine_of = wave_all / kTileWaves, wave = wave_all % kTileWaves;   // tile of the workgroup, wave of the tile
    const uint32_t together = blockDim.x / (64u * kTileWaves);   // tiles of this workgroup, at most kTiles
    const uint64_t stride = (uint64_t)gridDim.x * together;
    uint64_t tile = (uint64_t)blockIdx.x * together + mine_of;
    float largest = 0.0f;
    for (; tile < a.tiles; tile += stride) {
        // (row offsets are recomputed from these on every trip: kept across the loop they would take
        // more registers than the data)
        uint32_t s0 = a.s0;
        uint32_t lane = lane0;
        asm volatile("" : "+s"(s0), "+v"(lane));
        const uint32_t jq = lane & ((1u << column_bits(M)) - 1u), la = lane >> column_bits(M);
        const Tile<M> now(s0, (KIND == Kind::Encode || M == 11) ? xcd_order(tile, a.xcd_run_log2, together) : tile);
        // a tile mixes values of one block of 2^(s0 + M) floats: if that block lies in the implied
        // zero padding its results are zero too, and the next pass is told so instead of reading them
        // (the last pass writes everything: an empty gradient gives zeros).  Tiles are in the order of
        // their blocks, so all later ones lie there as well (and a workgroup's tiles in the same block).
        if (KIND == Kind::InPlace && now.block >= a.valid) break;
        float2 raw[16];
        load_rows<M>(a, now, lane, wave, raw);
        float v[kRegs];
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            v[2 * s] = raw[s].x;
            v[2 * s + 1] = raw[s].y;
        }
        uint32_t* sign_of = signs + mine_of * kRows;   // ToX: of this tile's rows
        if constexpr (KIND == Kind::ToX) {
            // one sign word per row (32 coordinates; with 11 stages it would be half of one): the rows lie far apart, a
            // lane computes a row's block.  Ordered by the barriers of the exchange, or inside the wave.
#pragma unroll
            for (uint32_t r = 0; r < kRows; r += 64u * kTileWaves) {
                const uint32_t row = r + 64u * wave + lane;
                const uint64_t g = now.row_start(row);
                const u32x4 sb = sign_block(g >> 7, a.key0, a.key1);
                const uint32_t which = (uint32_t)(g >> 5) & 3u;
                sign_of[row] = which == 0u ? sb.w[0] : which == 1u ? sb.w[1] : which == 2u ? sb.w[2] : sb.w[3];
            }
            if constexpr (kIndependent) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        rotate_tile<M>(v, reinterpret_cast<float*>(buf + 256u * kTileWaves * mine_of), lane, wave);

        if constexpr (KIND == Kind::RangeOnly || KIND == Kind::InPlaceLast) {
#pragma unroll
            for (int i = 0; i < kRegs; i += 2) {
                if (KIND == Kind::InPlaceLast) {
                    v[i] = v[i] * a.factor;
                    v[i + 1] = v[i + 1] * a.factor;
                }
                asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(largest) : "v"(largest), "v"(v[i]), "v"(v[i + 1]));
            }
        }
        if constexpr (KIND == Kind::InPlace || KIND == Kind::InPlaceLast) {
#pragma unroll
            for (int s = 0; s < 16; ++s)
                *reinterpret_cast<float2*>(a.data + now.row_start(row_after<M>((uint32_t)s, lane, wave)) + 2u * jq) =
                    make_float2(v[2 * s], v[2 * s + 1]);
        } else if constexpr (KIND == Kind::ToX) {
            // what lies below n, by row and column of the block (32-bit compares): rows before `full`, and of
            // row `full` the columns before `rest`
            const uint64_t left = a.n > now.block ? a.n - now.block : 0u;
            const uint64_t full64 = left >> s0;
            const uint32_t full = full64 > (1ull << M) ? 1u << M : (uint32_t)full64;
            const uint32_t rest = full64 > (1ull << M) ? 0u : (uint32_t)(left & ((1ull << s0) - 1ull));
            const uint32_t col0 = (uint32_t)(now.base - now.block) + 2u * jq;
            float* out = a.out + now.base + 2u * jq;
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const uint32_t row = row_after<M>((uint32_t)s, lane, wave);
                const uint32_t k = row & ((1u << M) - 1u), ext = (row >> M) * 32u;
                const uint32_t sw = sign_of[row] >> (2u * jq);
                const float x = __uint_as_float(xor_masked(__float_as_uint(v[2 * s] * a.factor), sw << 31, 0x80000000u));
                const float y = __uint_as_float(xor_masked(__float_as_uint(v[2 * s + 1] * a.factor), sw << 30, 0x80000000u));
                float* dst = out + (((uint64_t)k << s0) + ext);
                if (k < full + (col0 + ext + 2u <= rest ? 1u : 0u)) *reinterpret_cast<float2*>(dst) = make_float2(x, y);
                else if ((a.n & 1u) && k == full && col0 + ext + 1u == rest) *dst = x;
            }
        } else if constexpr (KIND == Kind::Encode) {
            // exchange inside the wave: 2 floats in each of 8 lanes -> 16 consecutive floats in one lane (run
            // L of 64), the coordinates of one block of the rounding stream and 2 * BITS payload
            // bytes; half of the slots at a time.  16-byte unit c of run L at column c ^ (L / 4 mod 4).
            float4* mine = buf + 256u * wave_all;
            uint64_t blk[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const uint32_t L = M == 11 ? 8u * s + la : 8u * s + 2u * la + (jq >> 3);
                    const uint32_t unit = 4u * L + (((jq >> 1) & 3u) ^ ((L >> 2) & 3u));
                    reinterpret_cast<float2*>(mine)[2u * unit + (jq & 1u)] = make_float2(v[2 * (8 * h + s)], v[2 * (8 * h + s) + 1]);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const uint32_t from = (M == 11 ? lane & 7u : (lane >> 1) & 3u) << column_bits(M);   // a lane of the run's row
                blk[h] = (now.row_start(row_after<M>(8u * h + (lane >> 3), from, wave)) >> 4) + (M == 11 ? 0u : lane & 1u);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 f = mine[4u * lane + ((uint32_t)i ^ ((lane >> 2) & 3u))];
                    v[16 * h + 4 * i] = f.x;
                    v[16 * h + 4 * i + 1] = f.y;
                    v[16 * h + 4 * i + 2] = f.z;
                    v[16 * h + 4 * i + 3] = f.w;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
            // same arithmetic and random stream as the fused encoders (quantize_store)
            constexpr bool kOffset = ((1u << BITS) - 2u) > kSingleFmaMaxLevels;
            const float s = a.scale[0], two = s + s;
            const bool ranged = two >= kMinRange;
            const float inv = ranged ? (float)a.levels / two : 0.0f;
            const float base = (ranged && !kOffset ? 0.5f * (float)a.levels : 0.0f) + 0x1p-9f;
            uint32_t by[8], pk[BITS];
#pragma unroll
            for (int h = 0; h < 2; ++h)
                k14::quantize_half<BITS, true, false, kOffset>(v, h, blk[h], -s, inv, base, a.levels, a.worker, a.key0,
                                                               a.key1, by, a.factor);
            k14::pack_bytes<BITS>(by, pk);
            uint8_t* d0 = a.payload + blk[0] * (2u * BITS);
            uint8_t* d1 = a.payload + blk[1] * (2u * BITS);
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
        // the next tile's sign words and exchange overwrite what other waves may still be reading
        if constexpr (M > 6 && (KIND == Kind::ToX || KIND == Kind::Encode)) __syncthreads();
    }
    if constexpr (kRange) {
        if (a.absmax) {   // (uniform over the grid) non-negative floats order like their bit patterns
            if (KIND == Kind::RangeOnly) largest = largest * a.factor;   // (monotone: the largest stays the largest)
            asm volatile("s_nop 1" : "+v"(largest));   // wait states between the assembly's write and a lane exchange
            uint32_t m = wave_umax(__float_as_uint(largest));
            if (lane0 == 0) most[wave_all] = m;
            __syncthreads();
            if (t == 0) {
                for (uint32_t w = 0; w < blockDim.x / 64u; ++w) m = most[w] > m ? most[w] : m;
                // (a stale read only costs an atomic more; most workgroups stay below the running maximum.
                // One look per workgroup: one per wave, 16384 of them on one address, took longer than
                // reading 134 MB.)
                if (m > __hip_atomic_load(a.absmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(a.absmax, m);
            }
        }
    }
}

// ---- quantizer on stored values ------------------------------------------------------------
// Stochastic rounding of rotated values (already normalised) onto the grid of [-s, s]:
// same arithmetic and random stream as the fused encoders.
struct FullQuant {
    float s, inv, half, off, Lf;
};
__device__ __forceinline__ FullQuant full_quant(float s, uint32_t levels) {
    FullQuant q;
    q.s = s;
    const float two = s + s;
    q.Lf = (float)levels;
    const bool ranged = two >= kMinRange;
    q.inv = ranged ? q.Lf / two : 0.0f;
    const bool single = levels <= kSingleFmaMaxLevels;   // evaluation order by grid size
    q.half = (single && ranged) ? 0.5f * q.Lf : 0.0f;   // an all-zero (or vanishingly small) vector gets index 0
    q.off = single ? 0.0f : s;
    return q;
}
// 16 consecutive coordinates (the ones of Philox block `blk` of the rounding stream) -> 2 * BITS payload bytes.
template <int BITS>
__device__ __forceinline__ void quantize_run(const float (&yv)[16], uint64_t blk, const FullQuant& q, uint32_t worker,
                                             uint32_t key0, uint32_t key1, uint8_t* payload) {
    const u32x4 rb = round_block(blk, worker, key0, key1);
    uint32_t pk[4] = {0u, 0u, 0u, 0u};
    // u = (r + 0.5) / 256 and L/2 + u are exact in fp32, so one multiply-add gives the same c = L/2 + u
    // (or u alone on the large grids); t >= 0, so the conversion's truncation is the floor.
    const float c0 = q.half + 0x1p-9f;
    const uint32_t L = (uint32_t)q.Lf;
    auto place = [&](int j, float y) {
        const uint32_t r = (rb.w[j >> 2] >> (8 * (j & 3))) & 0xFFu;
        const float c = __builtin_fmaf((float)r, 0x1p-8f, c0);
        const float tt = __builtin_fmaf(y, q.inv, c);
        const uint32_t idx = min((uint32_t)tt, L);
        const int bit = j * BITS;
        pk[bit >> 5] |= idx << (bit & 31);
    };
    if (q.off != 0.0f) {   // (uniform) large grids: fma(y + s, inv, u)
#pragma unroll
        for (int j = 0; j < 16; ++j) place(j, yv[j] + q.off);
    } else {               // small grids: fma(y, inv, L/2 + u)
#pragma unroll
        for (int j = 0; j < 16; ++j) place(j, yv[j]);
    }
    uint8_t* dst = payload + blk * (2u * BITS);
    if constexpr (BITS == 8) {
        *reinterpret_cast<uint4*>(dst) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
    } else if constexpr (BITS == 4) {
        *reinterpret_cast<uint2*>(dst) = make_uint2(pk[0], pk[1]);
    } else {
        *reinterpret_cast<uint32_t*>(dst) = pk[0];
    }
}

// ---- elementwise steps on rotated data ---------------------------------------------------
// Largest |y| of the whole array into *absmax (zeroed beforehand): non-negative floats
// order like their bit patterns, so an unsigned atomic max does it.
__global__ __launch_bounds__(256) void full_absmax_kernel(const float* y, uint64_t count, uint32_t* absmax) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x * 4u;
    float m = 0.0f;
    for (uint64_t i = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4u; i < count; i += stride) {
        const float4 q = *reinterpret_cast<const float4*>(y + i);
        m = fmaxf(fmaxf(m, fmaxf(fabsf(q.x), fabsf(q.y))), fmaxf(fabsf(q.z), fabsf(q.w)));
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63u) == 0) atomicMax(absmax, __float_as_uint(m));
}

// The quantizer on stored rotated values.  One thread: 16 coordinates, one Philox block,
// 2 * BITS payload bytes.
template <int BITS>
__global__ __launch_bounds__(256) void full_encode_kernel(const float* y, uint64_t count, const float* scale,
                                                          uint32_t levels, uint32_t worker, uint32_t key0,
                                                          uint32_t key1, uint8_t* payload) {
    const uint64_t blk = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t g0 = blk * 16u;
    if (g0 >= count) return;
    const FullQuant fq = full_quant(scale[0], levels);
    float yv[16];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float4 q = *reinterpret_cast<const float4*>(y + g0 + 4 * k);
        yv[4 * k] = q.x;
        yv[4 * k + 1] = q.y;
        yv[4 * k + 2] = q.z;
        yv[4 * k + 3] = q.w;
    }
    quantize_run<BITS>(yv, blk, fq, worker, key0, key1, payload);
}

// sums -> rotated-domain estimate of the mean: yhat = S * (step / W) - s.
template <typename SumT>
__global__ __launch_bounds__(256) void full_decode_kernel(const SumT* sums, uint64_t count, const float* scale,
                                                          uint32_t levels, uint32_t W, float* yhat) {
    const uint64_t g0 = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4u;
    if (g0 >= count) return;
    const float s = scale[0];
    const float step = (s + s) / (float)levels;
    const float q = step / (float)W;
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (float)(uint32_t)sums[g0 + e] * q - s;
    *reinterpret_cast<float4*>(yhat + g0) = make_float4(o[0], o[1], o[2], o[3]);
}

// ---- launch ------------------------------------------------------------------------------------
// One tile per workgroup (or independent wave), except for the range, whose workgroups stay so that few of
// them report.
template <int M, Kind KIND, int BITS = 4>
void launch_pass_t(uint32_t log2_size, hipStream_t stream, HighPassArgs& a) {
    constexpr int kFloatsLog2 = (M > 6 ? M : 6) + column_bits(M) + 1;   // of a tile
    constexpr auto kernel = high_pass_kernel<M, KIND, BITS>;
    a.tiles = 1ull << (log2_size - kFloatsLog2);
    uint32_t together = (uint32_t)pass_tiles(M);
    constexpr bool kReports = KIND == Kind::RangeOnly || KIND == Kind::InPlaceLast;
    // (two workgroups per CU; half a one where each reports to the same word)
    while (together > 1u && a.tiles / together < (kReports ? 128u : 512u)) together >>= 1;
    const uint32_t threads = 64u * together << wave_rows(M);
    uint64_t grid = a.tiles / together;
    a.xcd_run_log2 = xcd_run_log2(M, BITS, grid, together);
    if (kReports) {
        const uint32_t resident = resident_grid<kernel>((uint32_t)(64 * pass_waves(M)));   // (of full workgroups)
        if (resident != 0 && grid > resident) grid = resident;
    }
    hipLaunchKernelGGL(kernel, dim3((uint32_t)grid), dim3(threads), 0, stream, a);
}
// Stages of a high pass at most.  11 stages move 64-byte pieces, at about 0.7 of the rate of whole lines,
// and still beat a pass more (2^25 coordinates behind chunks of 2^14, 102 MB of them data: range 31.7 us, payload
// 42 us, inverse 64 us; as 6 + 5 stages 32 + 22, 33 and 44 + 51 us).
constexpr int kMaxStages = 11;

// Whether a plan has a pass of M stages of this kind: the first of two takes half of 12 .. 19 stages, a pass
// that is the last (or the only) one may have any number (11 only forward: 2^25 coordinates, a short gradient).
constexpr bool pass_exists(Kind kind, int M) {
    return kind == Kind::InPlace ? M >= 6 && M <= 10 : kind != Kind::ToX || M <= 10;
}

template <Kind KIND, int BITS = 4, int M = 1>
hipError_t launch_pass(uint32_t m, uint32_t log2_size, hipStream_t stream, HighPassArgs& a) {
    if constexpr (M <= kMaxStages) {
        if (m != (uint32_t)M) return launch_pass<KIND, BITS, M + 1>(m, log2_size, stream, a);
        if constexpr (pass_exists(KIND, M)) {
            launch_pass_t<M, KIND, BITS>(log2_size, stream, a);
            return hipGetLastError();
        }
    }
    return hipErrorInvalidValue;   // (no plan asks for it)
}

}  // namespace

// Stages first_log2 .. l-1 on data (2^l floats, the stages before them already done), in place; the last pass
// multiplies by `factor`, and for the inverse direction (`x` non-null) applies the sign
// diagonal and writes the first n coordinates to x instead.  Forward direction: only the
// first `valid` floats of data have been written (the rest is the zero padding, which the
// first pass supplies by itself), and `absmax`, if not null, receives the largest
// magnitude of the result (the word was zeroed by an earlier launch).  `deferred`, forward direction:
// RangeOnly = the last pass only reports the range and leaves data as the pass before it wrote
// it; EncodeOnly = only the last pass runs, on such data, and its results go through the
// quantizer into deferred->payload.
hipError_t launch_high_passes(float* data, uint32_t log2_size, float factor, float* x, uint64_t n,
                              uint32_t key0, uint32_t key1, hipStream_t stream, uint64_t valid,
                              float* absmax, uint32_t first_log2, const FullDeferred* deferred) {
    const bool range_only = deferred && deferred->kind == FullLast::RangeOnly;
    const bool encode_only = deferred && deferred->kind == FullLast::EncodeOnly;
    if ((deferred && (x || range_only == encode_only)) || (range_only && !absmax)) return hipErrorInvalidValue;
    uint32_t s0 = first_log2;
    const uint32_t passes = (log2_size - s0 + kMaxStages - 1u) / (uint32_t)kMaxStages;
    for (uint32_t p = 0; p < passes; ++p) {
        const uint32_t left = log2_size - s0;
        // spread the stages evenly so that no pass is needlessly short
        // (13 = 6 + 7, not 7 + 6: the pass that moves most goes without LDS.  2^27 coordinates, of them 70 M fp32
        // data: range 255 us and payload 90 us against 270 and 98 us, inverse 540 against 531; 108 M bf16: the
        // same either way)
        const uint32_t m = passes - p == 2u && left == 13u ? 6u : (left + (passes - p) - 1u) / (passes - p);
        const bool last = p + 1u == passes;
        HighPassArgs a{};
        a.data = data;
        a.s0 = s0;
        a.factor = factor;
        a.key0 = key0;
        a.key1 = key1;
        a.n = n;
        a.valid = valid;
        a.absmax = (last && !x) ? reinterpret_cast<uint32_t*>(absmax) : nullptr;
        hipError_t e = hipSuccess;
        if (last && x) {
            a.out = x;
            e = launch_pass<Kind::ToX>(m, log2_size, stream, a);
        } else if (last && range_only) {
            e = launch_pass<Kind::RangeOnly>(m, log2_size, stream, a);
        } else if (last && encode_only) {
            a.scale = deferred->scale;
            a.levels = deferred->levels;
            a.worker = deferred->worker;
            a.payload = deferred->payload;
            if (deferred->bits == 2) e = launch_pass<Kind::Encode, 2>(m, log2_size, stream, a);
            else if (deferred->bits == 4) e = launch_pass<Kind::Encode, 4>(m, log2_size, stream, a);
            else e = launch_pass<Kind::Encode, 8>(m, log2_size, stream, a);
        } else if (!encode_only) {
            e = last ? launch_pass<Kind::InPlaceLast>(m, log2_size, stream, a)
                     : launch_pass<Kind::InPlace>(m, log2_size, stream, a);
        }
        if (e != hipSuccess) return e;
        // what is not zero afterwards: the blocks of 2^(s0 + m) floats that held a value
        const uint64_t block = 1ull << (s0 + m);
        valid = (valid + block - 1) / block * block;
        s0 += m;
    }
    return hipSuccess;
}

hipError_t launch_full_absmax(const float* y, uint32_t log2_size, float* absmax, hipStream_t stream) {
    const hipError_t e = launch_zero_words(reinterpret_cast<uint32_t*>(absmax), 1, stream);
    if (e != hipSuccess) return e;
    const uint64_t count = 1ull << log2_size;
    uint64_t blocks = count / (256u * 4u * 8u);   // 8 vectors per thread
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(full_absmax_kernel, dim3((uint32_t)blocks), dim3(256), 0, stream, y, count,
                       reinterpret_cast<uint32_t*>(absmax));
    return hipGetLastError();
}

hipError_t launch_full_encode(const float* y, uint32_t log2_size, const float* scale, uint32_t levels,
                              uint32_t bits, uint32_t worker, uint32_t key0, uint32_t key1,
                              uint8_t* payload, hipStream_t stream) {
    const uint64_t count = 1ull << log2_size;
    const uint64_t blocks = (count / 16u + 255u) / 256u;
    const dim3 grid((uint32_t)blocks), block(256);
    if (bits == 2)
        hipLaunchKernelGGL(full_encode_kernel<2>, grid, block, 0, stream, y, count, scale, levels, worker, key0, key1, payload);
    else if (bits == 4)
        hipLaunchKernelGGL(full_encode_kernel<4>, grid, block, 0, stream, y, count, scale, levels, worker, key0, key1, payload);
    else
        hipLaunchKernelGGL(full_encode_kernel<8>, grid, block, 0, stream, y, count, scale, levels, worker, key0, key1, payload);
    return hipGetLastError();
}

hipError_t launch_full_decode(const void* sums, uint32_t sum_bytes, uint32_t log2_size, const float* scale,
                              uint32_t levels, uint32_t W, float* yhat, hipStream_t stream) {
    const uint64_t count = 1ull << log2_size;
    const uint64_t blocks = (count / 4u + 255u) / 256u;
    const dim3 grid((uint32_t)blocks), block(256);
    if (sum_bytes == 1)
        hipLaunchKernelGGL(full_decode_kernel<uint8_t>, grid, block, 0, stream, static_cast<const uint8_t*>(sums), count, scale, levels, W, yhat);
    else
        hipLaunchKernelGGL(full_decode_kernel<uint16_t>, grid, block, 0, stream, static_cast<const uint16_t*>(sums), count, scale, levels, W, yhat);
    return hipGetLastError();
}

}  // namespace thc
