// Tuned bf16 MFMA GEMM for gfx950 (MI355X):
//   C[Mo x No] = sum_r A(i, r) * B(j, r),  any Mo, No and R > 0 (operand spans below 4 GiB).
// Tile counts that do not fill the last round of CUs are balanced by covering part of the output
// with half-width tiles (TileSched).  A tile that would reach over the output's edge is moved back inside
// where the sizes allow (inside_row, inside_col); otherwise it is clipped: rows beyond an operand read as
// zeros through the buffer bound, columns beyond it are not stored, and the tile takes an epilogue of its
// own (tile_epilogue_clipped, SmallEpilogue).  Clipping tiles that could have been moved costs time (measured on
// 4000 x 2000 x 6000 with bias and GELU: 138 us forward clipped, 132 moved).
//
// One 512-thread workgroup (8 waves, two per SIMD) owns a BM x BN output tile and walks the
// reduction in steps of 64 through two LDS stages.  Operand tiles are copied global -> LDS by
// direct-to-LDS buffer loads (16 bytes per lane, no register staging).  MFMA 16x16x32 fragments
// are read from LDS with ds_read_b128 when the reduction index is contiguous in memory (KC) and
// with the transposing ds_read_b64_tr_b16 when the output index is contiguous (MC), so no operand
// is ever transposed in global memory.  16-byte chunks are permuted on their way into LDS (the
// lane chooses which global chunk it fetches) so that fragment reads are spread over the banks.
//
// The steady-state loop contains no vector ALU work at all: measurements showed that every VALU
// instruction (64-bit address arithmetic above all) takes issue slots from the MFMAs of the same
// SIMD.  Global addresses are a buffer descriptor per operand tile, a per-lane byte offset computed
// once, and a scalar offset that advances with the reduction step; LDS fragment addresses are
// per-lane registers computed once per stage, with the tile / sub-step part in the instruction's
// immediate offset; the loop is unrolled over the two stages so that nothing depends on the
// stage index at run time.
//
// The 16x16x32 MFMA is used rather than the 32x32x16 one: at the chip's power limit a loop of
// nothing but MFMAs on random operands sustains 2.0 PFLOP/s with the former and 1.75 with the
// latter (two waves per SIMD).  The accumulators hold the transposed 16x16 tile (B fragment
// first), which gives each lane 4 consecutive output columns; the epilogue rounds to bf16 once,
// stages the wave's sub-tile through LDS and writes full 128-byte row segments.
//
// Sustained, the kernel runs at the chip's power limit rather than at a cycle limit: the loop
// takes about 2260 cycles per step where its MFMAs need 2048, at a clock (1.8 GHz) that the power
// controller sets; a probe without the per-step barrier needed 6 % fewer cycles and ran at a 5 %
// lower clock, for the same time.  What is worth changing here is therefore what saves energy per
// flop (operand traffic) or removes idle time of whole CUs, not what hides stalls.
//
// The tile bodies serve gemm_mixed_kernel and gemm_mid_kernel (one product per launch) and gemm_group_kernel
// (gemm_group.hpp: the tiles of up to twelve independent products in one grid).
#pragma once
#include <type_traits>

#include "axo_common.hpp"

namespace axo {

constexpr int TILE_THREADS = 512;
constexpr int TILE_BK = 64;
constexpr int NUM_XCD = 8;

typedef __attribute__((address_space(3))) void* lds_void_ptr;

#ifndef AXO_PRIO
#define AXO_PRIO 1
#endif
#if AXO_PRIO
#define AXO_SETPRIO(n) __builtin_amdgcn_s_setprio(n)
#else
#define AXO_SETPRIO(n)
#endif
#ifndef AXO_SCHED
#define AXO_SCHED 1
#endif

// KC tile in LDS: row r is 128 bytes = 8 chunks of 16 bytes, chunk c stored at c ^ ((r / 2) % 8):
// 16 consecutive rows read at the same c then hit 16 different 16-byte bank groups.
__device__ __forceinline__ int swz_kc(int r) { return (r >> 1) & 7; }
// MC tile in LDS: reduction row k is ROWS*2 bytes, chunk c stored at c ^ f(k) with
// f(k) = 4*(k % 4) + 2*((k / 8) % 2): half a wave's transposing read touches 8 reduction rows
// (k % 4 and (k / 8) % 2 vary) times two 16-byte chunks, which then land in 16 different bank
// groups (without the second term the 16-lane groups collide: measured 50 % conflict cycles).
// Rows of 64 or 128 bytes (32 or 64 output indices): 4 or 2 of them share a 256-byte sweep of the banks, and the
// remaining bits of that choice pick the chunk.
template <int ROWS>
__device__ __forceinline__ int swz_mc(int k) {
    static_assert(ROWS == 32 || ROWS == 64 || ROWS == 128 || ROWS == 256, "row pitch");
    return ROWS == 32   ? ((k >> 3) & 1) << 1
           : ROWS == 64 ? (((k >> 1) & 1) << 1) | (((k >> 3) & 1) << 2)
                        : ((k & 3) << 2) | (((k >> 3) & 1) << 1);
}

// How one launch is cut into workgroups.  The output is covered by two column regions: columns
// [0, big_cols * 256) with 256x256 tiles and the rest with 256x128 tiles.  Workgroups
// [0, n_big) take the big tiles, the following n_small the small ones, so that CUs that run out
// of big tiles pick up small ones: a tile count that does not fill the last round of CUs is
// balanced by choosing how many columns each region gets (see the host-side planner).
struct TileSched {
    int tiles_m;     // tile rows (both regions use 256-row tiles)
    int big_cols;    // tile columns of the 256-wide region
    int small_cols;  // tile columns of the 128-wide region
    int n_big;       // = tiles_m * big_cols
    int group_m;     // band height of the tile order
    int shift;       // start_shift() units, 0 = none
};

// Start-up phase shift.  Tiles of equal length that start together end together, and then all CUs write their
// outputs in one burst, which the memory side takes microseconds to absorb while nothing computes.  The first workgroup on
// every CU (ids below 256) therefore sleeps phase * units * 640 cycles before it starts, phase = 0..7 dealt round-robin over
// the CUs of each XCD; later workgroups start whenever their CU falls free, so the shift persists through the launch.
// What it costs is a late start of up to 7 units, so it pays only where a tile is short and the launch has several
// rounds of them; the host decides (shift_units).
constexpr int SHIFT_PHASES = 8;
__device__ __forceinline__ void start_shift(int bid, int units) {
    if (units > 0 && bid < 256) {
        const int n = ((bid >> 3) % SHIFT_PHASES) * units;
        for (int i = 0; i < n; ++i) __builtin_amdgcn_s_sleep(10);
    }
}

// Workgroup -> output tile.  Consecutive workgroup ids go round-robin to the 8 XCDs, each with
// its own L2, so the ids that land on one XCD are given one contiguous run of tiles, and tiles
// are ordered in bands of group_m tile-rows so that the tiles in flight on an XCD share operand
// panels.  Any count: the first nblk % 8 XCDs get one tile more.
__device__ __forceinline__ int xcd_run(int bid, int nblk) {
    const int x = bid % NUM_XCD, q = nblk / NUM_XCD, r = nblk % NUM_XCD;
    return x * q + min(x, r) + bid / NUM_XCD;
}

__device__ __forceinline__ void tile_of_index(int t, int tiles_m, int tiles_n, int group_m, int& tm, int& tn) {
    const int band = group_m * tiles_n;
    const int b = t / band;
    const int first_m = b * group_m;
    const int gm = min(group_m, tiles_m - first_m);
    const int in_band = t - b * band;
    tm = first_m + in_band % gm;
    tn = in_band / gm;
}

template <int BM, int BN, int WGM, int WGN>
struct TileCfg {
    static constexpr int WTM = BM / WGM, WTN = BN / WGN;  // wave tile
    static constexpr int TM = WTM / 16, TN = WTN / 16;    // 16x16 MFMA tiles per wave
    static constexpr int AH = TM / 2;                     // A tiles per MFMA group (half the wave tile's rows)
    static constexpr int A_BYTES = BM * TILE_BK * 2, B_BYTES = BN * TILE_BK * 2;
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int WAVES = WGM * WGN, THREADS = WAVES * 64;
    static constexpr int A_ROUNDS = BM * (TILE_BK / 8) / THREADS, B_ROUNDS = BN * (TILE_BK / 8) / THREADS;
    static constexpr int LOADS_PER_STAGE = A_ROUNDS + B_ROUNDS;
    static constexpr int EPI_STRIDE = WTN * 2 + 16;  // bytes per staged row (padded)
    static constexpr int EPI_BYTES = WAVES * WTM * EPI_STRIDE;
    static constexpr int RING_BYTES = 2 * STAGE_BYTES;
    static constexpr int LDS_BYTES = (RING_BYTES > EPI_BYTES) ? RING_BYTES : EPI_BYTES;
    static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile is made of pairs of 16x16 MFMA tiles");
    static_assert((BM * (TILE_BK / 8)) % THREADS == 0 && (BN * (TILE_BK / 8)) % THREADS == 0, "whole load rounds");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of one CU");
};

// A tile whose operands are staged in a ring of D stages (gemm_ring_body).
template <int BM, int BN, int WGM, int WGN, int D>
struct RingCfg : TileCfg<BM, BN, WGM, WGN> {
    using T = TileCfg<BM, BN, WGM, WGN>;
    static constexpr int LDS_BYTES = D * T::STAGE_BYTES > T::EPI_BYTES ? D * T::STAGE_BYTES : T::EPI_BYTES;
};

// Per-lane byte offset (from the operand tile's origin at reduction step 0) of the 16-byte chunk
// this lane fetches in each load round.  Must stay below 2^32 (checked on the host).
template <int ROWS, int LAYOUT, int ROUNDS, int THREADS>
__device__ __forceinline__ void load_offsets(int tid, int64_t ld, uint32_t* off) {
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int q = j * THREADS + tid;
        if (LAYOUT == KC) {
            constexpr int CPR = TILE_BK / 8;  // chunks per row
            const int r = q / CPR, cs = q % CPR;
            off[j] = (uint32_t)(((int64_t)r * ld + ((cs ^ swz_kc(r)) << 3)) * 2);
        } else {
            constexpr int CPR = ROWS / 8;  // chunks per reduction row
            const int k = q / CPR, cs = q % CPR;
            off[j] = (uint32_t)(((int64_t)k * ld + ((cs ^ swz_mc<ROWS>(k)) << 3)) * 2);
        }
    }
}

// LDS byte addresses from which this lane reads its MFMA fragments of one operand in one stage.
// A 16x16x32 fragment is 8 consecutive reduction elements (lane/16 selects which 8 of the 32) of
// row/column lane%16 of the tile.  KC: one address per 32-wide reduction sub-step (the tile
// index adds 16 rows = 2048 bytes, folded into the instruction offset).  MC: one address per
// MFMA tile (the sub-step adds 32 reduction rows, folded into the instruction offset).  The two
// stages of an operand are adjacent in LDS, so the stage is an instruction offset as well and one
// set of addresses serves both.
template <int ROWS, int LAYOUT, int NT>
struct FragAddr {
    static constexpr int N = (LAYOUT == KC) ? 2 : NT;
    static constexpr int STAGE_STRIDE = ROWS * TILE_BK * 2;  // bytes between the operand's two stages
    uint32_t a[N];
    __device__ __forceinline__ void init(int row0, int lane, uint32_t tile_base) {
        if (LAYOUT == KC) {
            const int r = row0 + (lane & 15);
#pragma unroll
            for (int kq = 0; kq < 2; ++kq) {
                const int c = kq * 4 + (lane >> 4);
                a[kq] = tile_base + r * (TILE_BK * 2) + ((c ^ swz_kc(r)) << 4);
            }
        } else {
            const int i = lane & 15;
            const int krow = ((lane >> 4) << 3) + (i >> 2);
            const int sw = swz_mc<ROWS>(krow);  // unchanged by the +4 and +32 row offsets added in read()
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int n = row0 + t * 16 + ((i & 3) << 2);
                const int c = n >> 3, h = (n >> 2) & 1;
                a[t] = tile_base + krow * (ROWS * 2) + ((c ^ sw) << 4) + (h << 3);
            }
        }
    }
    // fragment of MFMA tile t at 32-wide sub-step kq of stage s (all compile-time after unrolling)
    __device__ __forceinline__ bf16x8 read(const char* lds0, int s, int t, int kq) const {
        if (LAYOUT == KC) {
            return *reinterpret_cast<const bf16x8*>(lds0 + a[kq] + s * STAGE_STRIDE + t * (16 * TILE_BK * 2));
        } else {
            // two transposing reads: each hands this lane 4 consecutive reduction elements of its column;
            // lane i of a 16-lane group addresses reduction row i/4, columns 4*(i%4)..+3
            typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
            const char* p = lds0 + a[t] + s * STAGE_STRIDE + kq * (32 * ROWS * 2);
            s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
            s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * (ROWS * 2)));
            union { struct { s16x4 a, b; } s; bf16x8 v; } u;
            u.s.a = lo;
            u.s.b = hi;
            return u.v;
        }
    }
};

// Whole cache lines of a KC operand whose rows do not start on them.  A 128-byte segment of such a row lies in two lines, and
// the loads of a step, which the texture path takes a line at a time, then touch each line twice, once for either step.
// Here stage j receives the row's lines instead: its chunks 8 j - phase .. 8 j + 7 - phase, where `phase` is the position
// of the row's start in its line.  Reduction chunk c of step j is then chunk (c + phase) % 8 of stage j, or of stage j + 1
// where c + phase passes 7: a step needs two stages, and a product one more stage than steps.
__device__ __forceinline__ int line_phase(const bf16_t* origin, int64_t ld, int r) {
    return (int)((uint32_t)(reinterpret_cast<uint64_t>(origin) >> 4) + (uint32_t)r * (uint32_t)(ld >> 3)) & 7;
}
// Chunk c of a step lies in its stage where it lies without phases, c ^ swz_kc, so that fragment reads stay free of bank conflicts
// (at its place in the line, 30-50 % of the LDS cycles were conflicts).  Stage j thus holds there chunk 8 j + line_chunk(c, phase).
__device__ __forceinline__ int line_chunk(int c, int phase) { return c + phase < 8 ? c : c - 8; }
// load_offsets for that: `first` for stage 0, where chunks in front of the row are replaced by its first one; `later`
// counts from the line behind stage 0's, so that it is never negative.
template <int ROUNDS, int THREADS>
__device__ __forceinline__ void line_load_offsets(int tid, const bf16_t* origin, int64_t ld, uint32_t* first, uint32_t* later) {
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int q = j * THREADS + tid, r = q >> 3, cs = q & 7;
        const int chunk = line_chunk(cs ^ swz_kc(r), line_phase(origin, ld, r));
        const uint32_t row = (uint32_t)r * (uint32_t)(ld * 2);  // the caller sees to it that offsets stay below 2^32
        first[j] = row + (uint32_t)(max(chunk, 0) * 16);
        later[j] = row + (uint32_t)((chunk + 8) * 16);
    }
}
// FragAddr for that, on a ring of D stages.  The rows of an operand's MFMA tiles lie 16 rows apart, which is a whole number
// of lines, so a lane has the same phase in all of them.
template <int ROWS, int D>
struct LineFragAddr {
    static constexpr int STAGE_STRIDE = ROWS * TILE_BK * 2;
    uint32_t a[2], last[2];  // per sub-step, from stage 0 and from the last stage, whose next one is stage 0
    __device__ __forceinline__ void init(int row0, int lane, uint32_t tile_base, const bf16_t* origin, int64_t ld) {
        const int r = row0 + (lane & 15), phase = line_phase(origin, ld, r);
#pragma unroll
        for (int kq = 0; kq < 2; ++kq) {
            const int c = kq * 4 + (lane >> 4) + phase;
            a[kq] = tile_base + r * (TILE_BK * 2) + (((c - phase) ^ swz_kc(r)) << 4) + (c >> 3) * STAGE_STRIDE;
            last[kq] = a[kq] + (D - 1) * STAGE_STRIDE - (c >> 3) * (D * STAGE_STRIDE);
        }
    }
    __device__ __forceinline__ bf16x8 read(const char* lds0, int s, int t, int kq) const {
        return *reinterpret_cast<const bf16x8*>(lds0 + (s == D - 1 ? last[kq] : a[kq] + s * STAGE_STRIDE) + t * (16 * TILE_BK * 2));
    }
};

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;  // a buffer resource descriptor in four SGPRs

// The first `n` (none if n <= 0, all if n >= 8) of the 8 bf16 elements of a 16-byte chunk, the others zero.
__device__ __forceinline__ u32x4 first_elements(u32x4 w, int n) {
#pragma unroll
    for (int d = 0; d < 4; ++d) w[d] &= n >= 2 * d + 2 ? 0xFFFFFFFFu : (n == 2 * d + 1 ? 0xFFFFu : 0u);
    return w;
}
__device__ __forceinline__ bf16x8 first_elements(bf16x8 f, int n) {
    union { bf16x8 v; u32x4 u; } x;
    x.v = f;
    x.u = first_elements(x.u, n);
    return x.v;
}

// Bound of the buffer descriptor of an operand tile: bytes from the tile's origin to the end of the last
// valid element of its `rows` valid rows (KC) or columns (MC) of a reduction of R.
template <int LAYOUT>
__device__ __forceinline__ uint32_t operand_bound(int64_t ld, int rows, int R) {
    const int64_t elems = LAYOUT == KC ? (int64_t)(rows - 1) * ld + R : ((int64_t)R - 1) * ld + rows;
    return R > 0 ? (uint32_t)((elems * 2 + 3) & ~(int64_t)3) : 0u;
}

// Raw buffer descriptor: base, stride 0, dword format, bound in bytes.
__device__ __forceinline__ u32x4_t tile_rsrc(const bf16_t* p, uint32_t bound) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    u32x4_t r;
    r[0] = __builtin_amdgcn_readfirstlane((uint32_t)v);
    r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32) & 0xFFFFu);
    r[2] = __builtin_amdgcn_readfirstlane(bound);
    r[3] = 0x00020000u;
    return r;
}

// Four bf16 values in two dwords, the first in the low half.
__device__ __forceinline__ f32x4 bf16x4_of(uint32_t lo, uint32_t hi) {
    return f32x4{__uint_as_float(lo << 16), __uint_as_float(lo & 0xFFFF0000u), __uint_as_float(hi << 16), __uint_as_float(hi & 0xFFFF0000u)};
}
// Four consecutive bf16 values of memory (8-byte aligned), the first `valid` of them inside the matrix, the others zero.
// The loads of a part are independent of each other (indices clamped, not a loop of `valid` rounds, each of which waits for
// its load).
__device__ __forceinline__ f32x4 load_bf16x4(const bf16_t* p, int valid) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (valid >= 4) {
        const uint2 raw = *reinterpret_cast<const uint2*>(p);
        x = bf16x4_of(raw.x, raw.y);
    } else if (valid > 0) {
        const bf16_t v0 = p[0], v1 = p[min(1, valid - 1)], v2 = p[min(2, valid - 1)];
        x[0] = bf16_bits_to_f32(v0);
        x[1] = valid > 1 ? bf16_bits_to_f32(v1) : 0.f;
        x[2] = valid > 2 ? bf16_bits_to_f32(v2) : 0.f;
    }
    return x;
}
__device__ __forceinline__ f32x4 load_f32x4(const float* p, int valid) {
    if (valid >= 4) return *reinterpret_cast<const f32x4*>(p);
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (valid > 0) {
        const float v0 = p[0], v1 = p[min(1, valid - 1)], v2 = p[min(2, valid - 1)];
        x[0] = v0;
        x[1] = valid > 1 ? v1 : 0.f;
        x[2] = valid > 2 ? v2 : 0.f;
    }
    return x;
}

// Stores four consecutive outputs of one row, `valid` (1..4) of them inside the matrix, rounded to bf16.
__device__ __forceinline__ void store_bf16_quad(const GemmArgs& g, f32x4 v, const int row, const int col, const int valid) {
    bf16_t* out = g.C + (int64_t)row * g.ldc + col;
    uint2 packed;
    packed.x = pack_bf16x2(v[0], v[1]);
    packed.y = pack_bf16x2(v[2], v[3]);
    if (valid >= 4) *reinterpret_cast<uint2*>(out) = packed;
    else {
        out[0] = (bf16_t)packed.x;
        if (valid > 1) out[1] = (bf16_t)(packed.x >> 16);
        if (valid > 2) out[2] = (bf16_t)packed.y;
    }
}
// The same in fp32.
__device__ __forceinline__ void store_f32_quad(const GemmArgs& g, f32x4 v, const int row, const int col, const int valid) {
    float* out = reinterpret_cast<float*>(g.C) + (int64_t)row * g.ldc + col;
    if (valid >= 4) *reinterpret_cast<f32x4*>(out) = v;
    else
        for (int e = 0; e < valid; ++e) out[e] = v[e];
}
template <int V>
using IC = std::integral_constant<int, V>;

// Tells the scheduler to deal the memory instructions of a group out between its MFMAs: one MFMA
// occupies the matrix pipe for 16 cycles, the wave can issue LDS reads in that shadow, and the
// other wave of the SIMD fills the pipe meanwhile.  (The direct-to-LDS loads are inline assembly
// and stay where the source puts them: at the head of their group.)
template <int N_MFMA, int N_VMEM, int N_DS, int I>
struct Interleave {
    static __device__ __forceinline__ void run() {
#if AXO_SCHED
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // 1 MFMA
        constexpr int V = (I + 1) * N_VMEM / N_MFMA - I * N_VMEM / N_MFMA;
        if constexpr (V > 0) __builtin_amdgcn_sched_group_barrier(0x020, V, 0);  // VMEM reads
        constexpr int D = (I + 1) * N_DS / N_MFMA - I * N_DS / N_MFMA;
        if constexpr (D > 0) __builtin_amdgcn_sched_group_barrier(0x100, D, 0);  // LDS reads
        if constexpr (I + 1 < N_MFMA) Interleave<N_MFMA, N_VMEM, N_DS, I + 1>::run();
#endif
    }
};

// s_waitcnt with only vmcnt set (gfx9 encoding: vmcnt in bits 3:0 and 15:14).
#define AXO_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

// Whether rows of the output straddle cache lines: by their pitch, or all alike by where the first one starts.
__host__ __device__ __forceinline__ bool rows_straddle(const GemmArgs& g) {
    return ((reinterpret_cast<uintptr_t>(g.C) | (uintptr_t)(g.ldc * 2)) & 127) != 0;
}

// A lane's 16 bytes of a whole tile's row.  Non-temporal where rows lie in whole cache lines: the
// output is not read again by this launch, and plain stores let it evict operand panels from L2 (0.5-5 % in grouped launches; plain / non-temporal in
// us on 128 x 128 tiles forward 2048 x 2048 x 256 6.65 / 6.24, x 1024 11.9 / 11.2, wgrad 4096 x 1024 of 512 tokens 8.0 / 7.55, on 64 x 64 ones two to a CU
// wgrad 2048 x 1024 of 512 6.3 / 6.15, level in one round, on 64 x 128 ones dgrad 512 x 4096 x 4096 27.4 / 20.0, 2048 x 1024 x 1024 level).  Plain where rows
// straddle lines: a non-temporal store of a part of a line does not wait in L2 for the rest of it, which the tile or wave beside this one
// writes.  Non-temporal / plain in us: dgrad 10600 x 7736 x 48 69.0 / 49.4, wgrad 5640 x 6152 of 72 tokens 35.9 / 27.3, forward 8200 x 4104 x 200
// 40.0 / 34.8, 3000 x 3000 x 200 14.9 / 13.1, 5000 x 10000 x 1000 114 / 105, on smaller tiles 264 x 328 x 136 4.17 / 3.43, 1000 x 1000 x 200 4.47 / 4.09,
// dgrad 1000^3 7.0 / 6.5, wgrad 3000 x 1000 of 2000 tokens 19.1 / 18.6, and 8 elements off lines on a pitch of whole ones forward 2048 x 2048 x 256
// 8.3 / 7.7, 1024 x 1024 x 128 4.1 / 3.7.  With two exceptions, which are always non-temporal:
// * tiles of 256 rows beyond 16 steps, where the panels may count for more (wgrad 2000 x 6000 of 4000 tokens 80 us, plain 90; 4104 x 4104 x 4104 152
//   either way; but forward 5000 x 10000 x 1200 130 and 121, x 2000 181 and 173), and in grouped launches: with the choice made in the
//   kernel, those and single launches with long reductions took 0.5-1 % longer, so it is a kernel of its own, of single launches only, and there
//   by the pitch alone;
// * whole 128 x 128 data gradient tiles, whose epilogue is that of the 256-row ones: plain 0.5-2.5 % quicker without an activation
//   (2000 x 2000 x 500 8.9 and 8.8 us), 1.6 % slower through the erf form (2001 x 2037 x 725 14.8 and 15.05).
template <bool PLAIN>
__device__ __forceinline__ void store_row(const u32x4 v, u32x4* to) {
    if constexpr (PLAIN) *to = v;
    else __builtin_nontemporal_store(v, to);
}

// Epilogue of a workgroup tile of 256 rows: acc[a][b][e] is C[i0 + wm*WTM + a*16 + lane%16][j0 + wn*WTN + b*16 + 4*(lane/16) + e].
template <typename C, int LA, int LB, bool PLAIN>
__device__ __forceinline__ void tile_epilogue(const GemmArgs& g, f32x4 (&acc)[C::TM][C::TN], const int i0, const int j0,
                                              const int wave, const int wm, const int wn, const int lane, char* smem) {
    __syncthreads();  // all waves are done reading the operand buffers
    char* stage = smem + wave * (C::WTM * C::EPI_STRIDE);
    // The epilogue kind is decided once, outside the element loops: the plain path is then
    // straight-line code (the activation code is large; branching around it per element made the
    // epilogue several times slower than the stores it feeds).  Every branch of that decision is
    // a complete epilogue, stores included; whatever the branches share (the wave tile's origin,
    // the output pointer) is formed here, ahead of the decision, with the origin pinned in scalar
    // registers, so no branch has a version of its own to merge afterwards.  (An earlier form
    // computed the origin behind a three-way switch; the generated code of one dgrad branch then
    // lacked the upper half of the 64-bit column offset and the stores went astray.  Positional,
    // bit-exact tests of the dgrad epilogues on every tile kernel, which they ask for by name, guard this.)
    int wrow0 = i0 + wm * C::WTM, wcol0 = j0 + wn * C::WTN;
    asm volatile("" : "+s"(wrow0), "+s"(wcol0));
    bf16_t* const Cw = g.C + (int64_t)wrow0 * g.ldc + wcol0;
    // The bias of a lane's four columns in the wave tile's block b of 16.
    auto bias_of = [&](const int b) __attribute__((always_inline)) {
        return g.add_bias ? load_bf16x4(g.bias + wcol0 + b * 16 + 4 * (lane >> 4), 4) : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto convert_and_stage = [&](auto epi_tag, auto far_tag) __attribute__((always_inline)) {
        constexpr int EPI = decltype(epi_tag)::value;
        constexpr bool FAR = decltype(far_tag)::value != 0;
        constexpr bool FWD_EPI = EPI >= EPI_BIAS && EPI <= EPI_BIAS_GELU_ERF;
        constexpr bool DACT = EPI == EPI_MUL_DGELU_TANH || EPI == EPI_MUL_DGELU_ERF;
#pragma unroll
        for (int b = 0; b < C::TN; ++b) {
            const int ncol = b * 16 + 4 * (lane >> 4);  // within the wave tile
            f32x4 bv = {0.f, 0.f, 0.f, 0.f};
            if (FWD_EPI) bv = bias_of(b);
#pragma unroll
            for (int a = 0; a < C::TM; ++a) {
                const int mrow = a * 16 + (lane & 15);
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[a][b][e];
                if (EPI == EPI_BIAS_GELU_ERF) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        // FAR: or the arithmetic that both forms share moves ahead of the choice between them, and the kernel spills
                        if (FAR) asm volatile("" : "+v"(v[e]));
                        v[e] = gelu_erf<FAR>(v[e] + bv[e]);
                    }
                } else if (FWD_EPI) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = apply_epilogue(v[e], bv[e], EPI);
                }
                if (DACT) {  // the four pre-activations that belong to this lane's four outputs
                    const uint2 raw = *reinterpret_cast<const uint2*>(
                        g.aux + (int64_t)(wrow0 + mrow) * g.ldaux + wcol0 + ncol);
                    v[0] = apply_dact(v[0], __uint_as_float(raw.x << 16), EPI);
                    v[1] = apply_dact(v[1], __uint_as_float(raw.x & 0xFFFF0000u), EPI);
                    v[2] = apply_dact(v[2], __uint_as_float(raw.y << 16), EPI);
                    v[3] = apply_dact(v[3], __uint_as_float(raw.y & 0xFFFF0000u), EPI);
                }
                uint2 packed;
                packed.x = pack_bf16x2(v[0], v[1]);
                packed.y = pack_bf16x2(v[2], v[3]);
                *reinterpret_cast<uint2*>(stage + mrow * C::EPI_STRIDE + ncol * 2) = packed;
            }
        }
    };
    // The staged sub-tile out to memory as full row segments of 16 bytes per lane.
    auto store_staged = [&]() __attribute__((always_inline)) {
        // the staging region is private to the wave: only wave-level ordering is needed
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_wave_barrier();
        constexpr int LANES_PER_ROW = C::WTN * 2 / 16;
        constexpr int ROWS_PER_PASS = 64 / LANES_PER_ROW;
        // All reads are issued before the first store: interleaved one by one (as the compiler
        // orders them when left alone) every store waits for its own LDS read, and the 16 round
        // trips cost more than the stores themselves (measured 5000 cycles for the slower wave of
        // each SIMD).  The accumulators are dead by now, so the registers are free.
        constexpr int PASSES = C::WTM / ROWS_PER_PASS;
        u32x4 vdat[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int row = p * ROWS_PER_PASS + lane / LANES_PER_ROW, ch = lane % LANES_PER_ROW;
            vdat[p] = *reinterpret_cast<const u32x4*>(stage + row * C::EPI_STRIDE + ch * 16);
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int row = p * ROWS_PER_PASS + lane / LANES_PER_ROW, ch = lane % LANES_PER_ROW;
            store_row<PLAIN>(vdat[p], reinterpret_cast<u32x4*>(Cw + (int64_t)row * g.ldc + ch * 8));
        }
    };
    auto finish = [&](auto epi_tag, auto far_tag) __attribute__((always_inline)) {
        convert_and_stage(epi_tag, far_tag);
        store_staged();
    };
    // Each product has its own epilogue kinds, so each layout pair compiles only those.
    if (LA == KC && LB == MC) {  // forward
        switch (g.epilogue) {
            case EPI_NONE: finish(IC<EPI_NONE>{}, IC<0>{}); return;
            case EPI_BIAS: finish(IC<EPI_BIAS>{}, IC<0>{}); return;
            case EPI_BIAS_GELU_TANH: finish(IC<EPI_BIAS_GELU_TANH>{}, IC<0>{}); return;
            default: break;
        }
        // A wave asks first if the erf form meets values that want the longer arithmetic (FAR of gelu_erf).  With 64 or 128 values
        // per lane that pays: forward 8192 x 512 x 8192 takes 101 us where there are none, 112 where there are, and 109 with that
        // arithmetic throughout (32768 x 2048 x 4096: 452, 469 and 462).
        float least = 0.f;  // the least sum of a column plus its bias is its least value
#pragma unroll
        for (int b = 0; b < C::TN; ++b) {
            const f32x4 bv = bias_of(b);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float sum = acc[0][b][e];
#pragma unroll
                for (int a = 1; a < C::TM; ++a) sum = fminf(sum, acc[a][b][e]);
                least = fminf(least, sum + bv[e]);
            }
        }
        if (__any(least < GELU_ERF_FAR)) finish(IC<EPI_BIAS_GELU_ERF>{}, IC<1>{});
        else finish(IC<EPI_BIAS_GELU_ERF>{}, IC<0>{});
    } else if (LA == KC && LB == KC) {  // dgrad
        switch (g.epilogue) {
            case EPI_NONE: finish(IC<EPI_NONE>{}, IC<0>{}); return;
            case EPI_MUL_DGELU_TANH: finish(IC<EPI_MUL_DGELU_TANH>{}, IC<0>{}); return;
            default: finish(IC<EPI_MUL_DGELU_ERF>{}, IC<0>{}); return;
        }
    } else {  // wgrad
        if (g.epilogue == EPI_ACC_F32) {
            // fp32 accumulation dW32 += acc, no rounding.  The wave's 64 fp32 columns are 256 bytes
            // per row: the sums are staged through the wave's LDS region (half the wave tile's rows
            // at a time, rows padded to 272 bytes) so that 16 lanes read, add and write back one
            // whole row segment with 16 bytes each; the old values are requested before the staging so
            // that their latency hides behind it.  (Straight from the MFMA register layout a row is
            // four separate 64-byte runs: measured 14-28 % over the bf16-output product.)
            float* Cf = reinterpret_cast<float*>(g.C) + (int64_t)wrow0 * g.ldc + wcol0;
            constexpr int F_STRIDE = C::WTN * 4 + 16;  // bytes per staged fp32 row
            constexpr int RP = C::WTM / 2;             // rows per pass
            constexpr int NI = RP / 4;                 // a wave instruction covers 4 rows
            static_assert(C::WTN == 64, "16 lanes x 16 bytes per fp32 row");
            static_assert(RP * F_STRIDE <= C::WTM * C::EPI_STRIDE, "fits the wave's staging region");
            const int frow = lane >> 4, fcol = (lane & 15) << 2;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x4 old[NI];
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    old[i] = *reinterpret_cast<const f32x4*>(Cf + (int64_t)(h * RP + i * 4 + frow) * g.ldc + fcol);
#pragma unroll
                for (int a = 0; a < C::TM / 2; ++a)
#pragma unroll
                    for (int b = 0; b < C::TN; ++b)
                        *reinterpret_cast<f32x4*>(stage + (a * 16 + (lane & 15)) * F_STRIDE + (b * 16 + 4 * (lane >> 4)) * 4) =
                            acc[h * (C::TM / 2) + a][b];
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the region is private to the wave
                __builtin_amdgcn_wave_barrier();
                f32x4 sum[NI];
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    sum[i] = *reinterpret_cast<const f32x4*>(stage + (i * 4 + frow) * F_STRIDE + fcol * 4);
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    *reinterpret_cast<f32x4*>(Cf + (int64_t)(h * RP + i * 4 + frow) * g.ldc + fcol) = old[i] + sum[i];
                __builtin_amdgcn_wave_barrier();  // LDS operations of a wave complete in order: the next pass may overwrite
            }
            return;
        }
        finish(IC<EPI_NONE>{}, IC<0>{});
    }
}

// f(0) .. f(N - 1), four to a pass of a loop.
template <int N, typename F>
__device__ __forceinline__ void by_four(F f) {
    static_assert(N % 4 == 0, "whole passes");
#pragma nounroll
    for (int i0 = 0; i0 < N; i0 += 4)
#pragma unroll
        for (int i = 0; i < 4; ++i) f(i0 + i);
}

// The epilogue of a tile of 256 rows that reaches over the output's edge, any kind, one compact path: the wave stages its
// sums in fp32 and stores the quads of columns that lie inside.  Same operations per element as the whole-tile epilogue, so an element's
// bits do not depend on the tile that it falls in.  (wrow0, wcol0): the wave tile's origin.
// Plain sums and forward kinds go half the wave tile's rows at a time.  What reads pre-activations or old fp32 values goes 32 rows at a
// time and requests them a pass ahead: one trip to memory is left of each tile's.  (Requested four rows at a time when they were wanted there
// were eight, every quad of columns chose its kind anew, and in launches of one round the tiles at the edge ended long after the others.)
// Before and now in us: wgrad into fp32 3001 x 3003 of 77 tokens 32.8 / 20.4, 4001 x 4003 of 1000 71 / 56, 3000 x 3000 of 100 19.1 / 17.6; dgrad 3001 x 3003
// x 77 through tanh GELU 35.3 / 21.2, x 1000 through the erf form 52.4 / 38.6; forward 3001 x 3003 x 1000 with a bias 31.0 / 26.1, with erf GELU
// 39.3 / 35.5, without either 25.3 / 25.2.
template <typename C, int LA, int LB>
__device__ __forceinline__ void tile_epilogue_clipped(const GemmArgs& g, f32x4 (&acc)[C::TM][C::TN], const int wrow0,
                                                      const int wcol0, const int wave, const int lane, char* smem) {
    constexpr bool FWD = LA == KC && LB == MC, DGRAD = LA == KC && LB == KC;
    constexpr int F_STRIDE = C::WTN * 4 + 16, QPR = C::WTN / 4, RPI = 64 / QPR;
    // a lane keeps its four columns
    const int lc = (lane % QPR) * 4, col = wcol0 + lc, valid = min(4, g.No - col);
    // sums of `tiles` rows of MFMA tiles from `first` on to the wave's region
    auto put_sums = [&](char* stage, auto first, auto tiles) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < decltype(tiles)::value; ++a)
#pragma unroll
            for (int b = 0; b < C::TN; ++b)
                *reinterpret_cast<f32x4*>(stage + (a * 16 + (lane & 15)) * F_STRIDE + (b * 16 + 4 * (lane >> 4)) * 4) =
                    acc[decltype(first)::value + a][b];
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the region is private to the wave
        __builtin_amdgcn_wave_barrier();
    };
    if (FWD || g.epilogue == EPI_NONE) {
        constexpr int RP = C::WTM / 2, ITERS = RP / RPI;
        static_assert(RP * F_STRIDE <= C::WTM * C::EPI_STRIDE, "fits the wave's staging region");
        char* const stage = smem + wave * (C::WTM * C::EPI_STRIDE);
        f32x4 bias = {0.f, 0.f, 0.f, 0.f};
        if (FWD && g.epilogue != EPI_NONE && g.add_bias && valid > 0) bias = load_bf16x4(g.bias + col, valid);
        __syncthreads();  // all waves are done reading the operand buffers
        auto half = [&](auto h) __attribute__((always_inline)) {
            put_sums(stage, IC<decltype(h)::value * (C::TM / 2)>{}, IC<C::TM / 2>{});
            const int row0 = wrow0 + decltype(h)::value * RP;
            if (g.epilogue == EPI_NONE) {
#pragma unroll 4
                for (int i = 0; i < ITERS; ++i) {
                    const int lr = i * RPI + lane / QPR, row = row0 + lr;
                    if (row < g.Mo && valid > 0)
                        store_bf16_quad(g, *reinterpret_cast<const f32x4*>(stage + lr * F_STRIDE + lc * 4), row, col, valid);
                }
            } else if constexpr (FWD) {
                auto rows = [&](auto f) __attribute__((always_inline)) {
                    by_four<ITERS>([&](int i) __attribute__((always_inline)) {
                        const int lr = i * RPI + lane / QPR, row = row0 + lr;
                        f32x4 v = *reinterpret_cast<const f32x4*>(stage + lr * F_STRIDE + lc * 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = f(v[e], bias[e]);
                        if (row < g.Mo && valid > 0) store_bf16_quad(g, v, row, col, valid);
                    });
                };
                switch (g.epilogue) {
                    case EPI_BIAS: rows([](float s, float x) { return apply_epilogue(s, x, EPI_BIAS); }); break;
                    case EPI_BIAS_GELU_TANH: rows([](float s, float x) { return apply_epilogue(s, x, EPI_BIAS_GELU_TANH); }); break;
                    default: rows([](float s, float x) { return apply_epilogue(s, x, EPI_BIAS_GELU_ERF); }); break;
                }
            }
            __builtin_amdgcn_wave_barrier();  // LDS operations of a wave complete in order: the next pass may overwrite
        };
        half(IC<0>{});
        half(IC<1>{});
        return;
    }
    if constexpr (!FWD) {
        constexpr int ROWS = 32, ITERS = ROWS / RPI;
        constexpr int WAVE_BYTES = ROWS * (F_STRIDE + C::WTN * 2);  // the sums, and behind them the pre-activations
        static_assert(C::WAVES * WAVE_BYTES <= C::LDS_BYTES, "fits the operand buffers");
        char* const stage = smem + wave * WAVE_BYTES;
        char* const pre = stage + ROWS * F_STRIDE;
        const bool inside = wcol0 + C::WTN <= g.No;
        // A pass's old fp32 values or pre-activations: in four dwords or in two, or, in a wave tile that reaches over the last column, in
        // one each.  What lies beyond the matrix stands for the last row's or column's, and is not stored.
        u32x4 in[ITERS];
        auto request = [&](auto inside_tag, const int row0, const int i) __attribute__((always_inline)) {
            const int row = min(row0 + i * RPI + lane / QPR, g.Mo - 1);
            auto load = [&](auto* at) __attribute__((always_inline)) {
                if constexpr (!decltype(inside_tag)::value) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) in[i][e] = at[min(col + e, g.No - 1)];
                } else if constexpr (!DGRAD) in[i] = *reinterpret_cast<const u32x4*>(at + col);
                else {
                    const uint2 raw = *reinterpret_cast<const uint2*>(at + col);
                    in[i][0] = raw.x;
                    in[i][1] = raw.y;
                }
            };
            if constexpr (DGRAD) load(g.aux + (int64_t)row * g.ldaux);
            else load(reinterpret_cast<const uint32_t*>(g.C) + (int64_t)row * g.ldc);
        };
        auto first = [&](auto inside_tag) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < ITERS; ++i) request(inside_tag, wrow0, i);
        };
        auto tile = [&](auto inside_tag) __attribute__((always_inline)) {
            auto pass = [&](auto p_tag) __attribute__((always_inline)) {
                constexpr int p = decltype(p_tag)::value;
                constexpr bool more = p + 1 < C::WTM / ROWS;
                const int row0 = wrow0 + p * ROWS;
                if constexpr (DGRAD) {
#pragma unroll
                    for (int i = 0; i < ITERS; ++i) {
                        *reinterpret_cast<uint2*>(pre + (i * RPI + lane / QPR) * (C::WTN * 2) + lc * 2) =
                            decltype(inside_tag)::value ? uint2{in[i][0], in[i][1]} : uint2{in[i][0] | in[i][1] << 16, in[i][2] | in[i][3] << 16};
                        if constexpr (more) request(inside_tag, row0 + ROWS, i);
                    }
                }
                put_sums(stage, IC<p * (ROWS / 16)>{}, IC<ROWS / 16>{});
                auto sums = [&](int lr) __attribute__((always_inline)) { return *reinterpret_cast<const f32x4*>(stage + lr * F_STRIDE + lc * 4); };
                if constexpr (!DGRAD) {
#pragma unroll
                    for (int i = 0; i < ITERS; ++i) {
                        const int lr = i * RPI + lane / QPR, row = row0 + lr;
                        const f32x4 sum = __builtin_bit_cast(f32x4, in[i]) + sums(lr);
                        if (row < g.Mo && valid > 0) store_f32_quad(g, sum, row, col, decltype(inside_tag)::value ? 4 : valid);
                        if constexpr (more) request(inside_tag, row0 + ROWS, i);
                    }
                } else {
                    auto rows = [&](auto f) __attribute__((always_inline)) {
                        by_four<ITERS>([&](int i) __attribute__((always_inline)) {
                            const int lr = i * RPI + lane / QPR, row = row0 + lr;
                            const uint2 raw = *reinterpret_cast<const uint2*>(pre + lr * (C::WTN * 2) + lc * 2);
                            const f32x4 x = bf16x4_of(raw.x, raw.y);
                            f32x4 v = sums(lr);
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = f(v[e], x[e]);
                            if (row < g.Mo && valid > 0) store_bf16_quad(g, v, row, col, valid);
                        });
                    };
                    if (g.epilogue == EPI_MUL_DGELU_TANH) rows([](float s, float x) { return apply_dact(s, x, EPI_MUL_DGELU_TANH); });
                    else rows([](float s, float x) { return apply_dact(s, x, EPI_MUL_DGELU_ERF); });
                }
                __builtin_amdgcn_wave_barrier();  // LDS operations of a wave complete in order: the next pass may overwrite
            };
            pass(IC<0>{});
            pass(IC<1>{});
            if constexpr (C::WTM > 64) {
                pass(IC<2>{});
                pass(IC<3>{});
            }
        };
        if (inside) first(std::true_type{});
        else first(std::false_type{});
        __syncthreads();  // all waves are done reading the operand buffers; outside the branches, which the waves of a tile take differently
        if (inside) tile(std::true_type{});
        else tile(std::false_type{});
    }
}

// Epilogue of a tile of at most 128 x 128, whole or reaching over the output's edge.  What it reads from memory beside the sums is
// requested on its own and kept as it comes, so that 64 x 64 tiles can do that ahead of the reduction: a short kernel has nothing else to
// hide a trip to memory behind.  The arithmetic is done in the accumulators' layout for both kinds of tiles, only the stores differ.
// With the epilogues of the 256-row tiles, which load when they need it, and where clipped in two batches one behind the other, dgrad
// 1001 x 1027 x 515 through the erf form spent 1.4 us between the last MFMA of a whole tile and its last store, and 3.3 us in the
// tiles of the last three columns; the kernel took 10.6 us and takes 9.8 now.  Likewise, before and now: forward 1001 x 515 x 1027 with a bias
// 8.0 and 7.25, 512 x 1024 x 1024 with tanh GELU 6.6 and 6.3, wgrad into fp32 1000^3 9.6 and 9.1, 1001 x 1003 x 1000 9.95 and 8.8; on
// 128 x 128 tiles dgrad 2001 x 2037 x 725 through the erf form 18.7 and 16.1, forward 2048 x 2048 x 512 with tanh GELU 9.5 and 9.0.
template <typename C, int LA, int LB>
struct SmallEpilogue {
    static constexpr bool FWD = LA == KC && LB == MC, DGRAD = LA == KC && LB == KC;
    static constexpr int ROWS = C::TM, COLS = C::TN;
    // fp32 sums are added in another layout, in which the lanes of a row follow each other: QPR quads per row, half the rows at a time
    static constexpr int F_STRIDE = C::WTN * 4 + 16, RP = C::WTM / 2, QPR = C::WTN / 4, RPI = 64 / QPR, ITERS = RP / RPI;
    static_assert(RP * F_STRIDE <= C::WTM * C::EPI_STRIDE, "fits the wave's staging region");
    u32x4 in[FWD ? COLS : DGRAD ? ROWS * COLS : 2 * ITERS];
    int wrow0, wcol0, lane;
    bool inside;

    __device__ __forceinline__ int sum_row(int i) const { return wrow0 + i / ITERS * RP + i % ITERS * RPI + lane / QPR; }
    __device__ __forceinline__ int sum_col() const { return wcol0 + lane % QPR * 4; }
    // (wrow0_, wcol0_): the wave tile's origin
    __device__ __forceinline__ void request(const GemmArgs& g, int wrow0_, int wcol0_, int lane_) {
        wrow0 = wrow0_;
        wcol0 = wcol0_;
        lane = lane_;
        if (g.epilogue == EPI_NONE) return;
        if (FWD && !g.add_bias) {
#pragma unroll
            for (u32x4& x : in) x = u32x4{0u, 0u, 0u, 0u};
            inside = true;
            return;
        }
        // A wave tile inside the columns takes whole quads, one that reaches over the last column single values; what lies beyond the
        // matrix stands for the last row's or column's, and is not stored.  One choice per wave, no lane's own: registers that different
        // loads of a lane may write make the compiler wait for one before the other.
        inside = wcol0 + C::WTN <= g.No;
        if (inside) load(g, std::true_type{});
        else load(g, std::false_type{});
    }
    template <typename Inside>
    __device__ __forceinline__ void load(const GemmArgs& g, Inside) {
        if constexpr (FWD || DGRAD) {
#pragma unroll
            for (int b = 0; b < COLS; ++b)
#pragma unroll
                for (int a = 0; a < (FWD ? 1 : ROWS); ++a) {
                    const int row = min(wrow0 + a * 16 + (lane & 15), g.Mo - 1), col = wcol0 + b * 16 + 4 * (lane >> 4);
                    const bf16_t* const p = FWD ? g.bias : g.aux + (int64_t)row * g.ldaux;
                    u32x4& x = in[FWD ? b : a * COLS + b];  // four values in two dwords, or in one each
                    if constexpr (Inside::value) {
                        const uint2 raw = *reinterpret_cast<const uint2*>(p + col);
                        x[0] = raw.x;
                        x[1] = raw.y;
                    } else
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = p[min(col + e, g.No - 1)];
                }
        } else {
#pragma unroll
            for (int i = 0; i < 2 * ITERS; ++i) {
                const uint32_t* const p = reinterpret_cast<const uint32_t*>(g.C) + (int64_t)min(sum_row(i), g.Mo - 1) * g.ldc;
                if constexpr (Inside::value) in[i] = *reinterpret_cast<const u32x4*>(p + sum_col());
                else
#pragma unroll
                    for (int e = 0; e < 4; ++e) in[i][e] = p[min(sum_col() + e, g.No - 1)];
            }
        }
    }
    __device__ __forceinline__ f32x4 extra(int a, int b) const {
        const u32x4 x = in[FWD ? b : a * COLS + b];
        return bf16x4_of(x[0], x[1]);
    }
    // behind the barrier after which the operand buffers may be overwritten
    __device__ __forceinline__ void finish(const GemmArgs& g, f32x4 (&acc)[C::TM][C::TN], int wave, char* smem, bool whole) {
        char* const stage = smem + wave * (C::WTM * C::EPI_STRIDE);
        if constexpr (!FWD && !DGRAD) if (g.epilogue == EPI_ACC_F32) {
            float* const out = reinterpret_cast<float*>(g.C);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int a = 0; a < ROWS / 2; ++a)
#pragma unroll
                    for (int b = 0; b < COLS; ++b)
                        *reinterpret_cast<f32x4*>(stage + (a * 16 + (lane & 15)) * F_STRIDE + (b * 16 + 4 * (lane >> 4)) * 4) =
                            acc[h * (ROWS / 2) + a][b];
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the region is private to the wave
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < ITERS; ++i) {
                    const int row = sum_row(h * ITERS + i), col = sum_col();
                    const f32x4 v = *reinterpret_cast<const f32x4*>(stage + (i * RPI + lane / QPR) * F_STRIDE + lane % QPR * 16);
                    const f32x4 sum = __builtin_bit_cast(f32x4, in[h * ITERS + i]) + v;
                    if (whole) *reinterpret_cast<f32x4*>(out + (int64_t)row * g.ldc + col) = sum;
                    else if (row < g.Mo && col < g.No) store_f32_quad(g, sum, row, col, min(4, g.No - col));
                }
                __builtin_amdgcn_wave_barrier();  // LDS operations of a wave complete in order: the next pass may overwrite
            }
            return;
        }
        auto convert = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < COLS; ++b)
#pragma unroll
                for (int a = 0; a < ROWS; ++a) {
                    const f32x4 v = f(acc[a][b], a, b);
                    uint2 packed;
                    packed.x = pack_bf16x2(v[0], v[1]);
                    packed.y = pack_bf16x2(v[2], v[3]);
                    *reinterpret_cast<uint2*>(stage + (a * 16 + (lane & 15)) * C::EPI_STRIDE + (b * 16 + 4 * (lane >> 4)) * 2) = packed;
                }
        };
        auto each = [&](auto f) __attribute__((always_inline)) {  // f(sum, what is read for it)
            if (!inside)
#pragma unroll
                for (u32x4& x : in) x = u32x4{x[0] | x[1] << 16, x[2] | x[3] << 16, 0u, 0u};
            convert([&](f32x4 v, int a, int b) __attribute__((always_inline)) {
                const f32x4 x = extra(a, b);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = f(v[e], x[e]);
                return v;
            });
        };
        auto plain = [&]() __attribute__((always_inline)) { convert([](f32x4 v, int, int) { return v; }); };
        if constexpr (FWD) switch (g.epilogue) {
            case EPI_NONE: plain(); break;
            case EPI_BIAS: each([](float s, float x) { return apply_epilogue(s, x, EPI_BIAS); }); break;
            case EPI_BIAS_GELU_TANH: each([](float s, float x) { return apply_epilogue(s, x, EPI_BIAS_GELU_TANH); }); break;
            // the longer arithmetic on every value: 1024^3 6.2 us, 6.4 where a wave asks first if it needs it
            default: each([](float s, float x) { return apply_epilogue(s, x, EPI_BIAS_GELU_ERF); }); break;
        } else if constexpr (DGRAD) switch (g.epilogue) {
            case EPI_NONE: plain(); break;
            case EPI_MUL_DGELU_TANH: each([](float s, float x) { return apply_dact(s, x, EPI_MUL_DGELU_TANH); }); break;
            default: each([](float s, float x) { return apply_dact(s, x, EPI_MUL_DGELU_ERF); }); break;
        } else plain();
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the region is private to the wave
        __builtin_amdgcn_wave_barrier();
        constexpr int LANES_PER_ROW = C::WTN * 2 / 16, ROWS_PER_PASS = 64 / LANES_PER_ROW, PASSES = C::WTM / ROWS_PER_PASS;
        u32x4 out[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p)  // all reads ahead of the first store, as in tile_epilogue
            out[p] = *reinterpret_cast<const u32x4*>(stage + (p * ROWS_PER_PASS + lane / LANES_PER_ROW) * C::EPI_STRIDE + lane % LANES_PER_ROW * 16);
        const int row0 = wrow0 + lane / LANES_PER_ROW, col = wcol0 + lane % LANES_PER_ROW * 8, valid = g.No - col;
        bf16_t* const to = g.C + (int64_t)row0 * g.ldc + col;
        if (whole) {
            auto rows = [&](auto plain_tag) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < PASSES; ++p)
                    store_row<decltype(plain_tag)::value>(out[p], reinterpret_cast<u32x4*>(to + (int64_t)(p * ROWS_PER_PASS) * g.ldc));
            };
            if (rows_straddle(g)) rows(std::true_type{});
            else {  // between two statements that it does not move: or the compiler makes one of both kinds of stores, a plain one
                asm volatile("; non-temporal");
                rows(std::false_type{});
                asm volatile("; non-temporal");
            }
            return;
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            bf16_t* const at = to + (int64_t)(p * ROWS_PER_PASS) * g.ldc;
            if (row0 + p * ROWS_PER_PASS >= g.Mo) continue;
            if (valid >= 8) *reinterpret_cast<u32x4*>(at) = out[p];
            else
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (e < valid) at[e] = (bf16_t)(out[p][e / 2] >> (e % 2 * 16));
        }
    }
};

// One BM x BN output tile with its top-left corner at (i0, j0), whole reduction.  LINES: the rows of A, which is KC, are
// fetched by whole cache lines (line_phase), on three stages; with them and two of B the LDS is full, so rows of B that
// do not start on lines still put every segment into two.  The loads of a step then touch 768 lines (dgrad) or 576 (forward) instead
// of 1024 or 832.
template <int BM, int BN, int WGM, int WGN, int LA, int LB, bool LINES = false, bool PLAIN = false>
__device__ __forceinline__ void gemm_tile_body(const GemmArgs& g, const int i0, const int j0, char* smem) {
    using C = TileCfg<BM, BN, WGM, WGN>;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    // The loop is unrolled over the two LDS stages, so it walks the reduction rounded up to the
    // next multiple of 128; what lies beyond the true length must contribute nothing, whatever
    // the memory there holds (zeros would do for finite data, but a stray infinity times a zero
    // of the other operand would put a NaN into a row that has none: BOTH operands are made zero).
    //  * MC operand (reduction index = row index): rows at or beyond R lie behind the buffer
    //    descriptor's bound, the byte count from the tile origin to the end of the tile's columns
    //    in row R - 1, and read as zeros.
    //  * KC operand (reduction inside the rows): the overrun of a row lands in the next row,
    //    which no linear bound can mask; the surplus 16-byte chunks of the last two steps are
    //    overwritten with zeros in LDS instead, and a chunk that is part inside is masked.  The bound
    //    (end of the tile's last valid row) keeps the last row's overrun from touching memory behind
    //    the matrix and makes rows beyond the matrix read as zeros.
    // On this chip the range check covers the sum of the per-lane offset and the scalar offset
    // that carries the reduction step (measured: lowering the bound by the scalar offset at every
    // step zeroed the second half of the reduction), so one constant bound serves the whole walk.
    const int KT = (g.R + 2 * TILE_BK - 1) / (2 * TILE_BK) * 2;
    const bool tail = (g.R % (2 * TILE_BK)) != 0;

    // global side: descriptor at the tile origin, per-lane offsets, scalar step
    const bf16_t* Ab = (LA == KC) ? g.A + (int64_t)i0 * g.lda : g.A + i0;
    const bf16_t* Bb = (LB == KC) ? g.B + (int64_t)j0 * g.ldb : g.B + j0;
    const uint32_t a_valid = operand_bound<LA>(g.lda, min(BM, g.Mo - i0), g.R);
    const uint32_t b_valid = operand_bound<LB>(g.ldb, min(BN, g.No - j0), g.R);
    const u32x4_t a_rsrc = tile_rsrc(Ab, a_valid);
    const u32x4_t b_rsrc = tile_rsrc(Bb, b_valid);
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void_ptr)smem;
    const uint32_t a_step = (uint32_t)((LA == KC) ? TILE_BK * 2 : (int64_t)TILE_BK * g.lda * 2);
    const uint32_t b_step = (uint32_t)((LB == KC) ? TILE_BK * 2 : (int64_t)TILE_BK * g.ldb * 2);
    uint32_t a_off[C::A_ROUNDS], b_off[C::B_ROUNDS];
    uint32_t a_later[C::A_ROUNDS];
    if constexpr (LINES) line_load_offsets<C::A_ROUNDS, C::THREADS>(tid, Ab, g.lda, a_off, a_later);
    else load_offsets<BM, LA, C::A_ROUNDS, C::THREADS>(tid, g.lda, a_off);
    load_offsets<BN, LB, C::B_ROUNDS, C::THREADS>(tid, g.ldb, b_off);

    // LDS side: [A stage 0][A stage 1][B stage 0][B stage 1] (LINES: three stages of A); fragment addresses of stage 0
    static_assert(!LINES || LA == KC, "lines of rows");
    constexpr int A_STAGES = LINES ? 3 : 2;
    std::conditional_t<LINES, LineFragAddr<BM, A_STAGES>, FragAddr<BM, LA, C::TM>> fra;
    FragAddr<BN, LB, C::TN> frb;
    if constexpr (LINES) fra.init(wm * C::WTM, lane, 0, Ab, g.lda);
    else fra.init(wm * C::WTM, lane, 0);
    frb.init(wn * C::WTN, lane, A_STAGES * C::A_BYTES);

    f32x4 acc[C::TM][C::TN];
#pragma unroll
    for (int a = 0; a < C::TM; ++a)
#pragma unroll
        for (int b = 0; b < C::TN; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[a][b][e] = 0.0f;

    // A reduction step of 64 is four MFMA groups: (sub-step kq, row half ah) for kq, ah in {0, 1};
    // a group multiplies AH A fragments with all TN B fragments of its sub-step.  A fragments are
    // double buffered per group, B fragments per sub-step.
    bf16x8 fa[2][C::AH], fb[2][C::TN];
    auto read_a = [&](int set, int s, int kq, int ah) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < C::AH; ++a) fa[set][a] = fra.read(smem, s, ah * C::AH + a, kq);
    };
    auto read_b = [&](int set, int s, int kq) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < C::TN; ++b) fb[set][b] = frb.read(smem, s, b, kq);
    };
    auto mfma_group = [&](int aset, int bset, int ah) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < C::AH; ++a)
#pragma unroll
            for (int b = 0; b < C::TN; ++b)
                acc[ah * C::AH + a][b] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[bset][b], fa[aset][a], acc[ah * C::AH + a][b], 0, 0, 0);
    };
    constexpr int N_MFMA = C::AH * C::TN;
    constexpr int RD_A = (LA == KC ? 1 : 2) * C::AH, RD_B = (LB == KC ? 1 : 2) * C::TN;
    uint32_t a_soff = 0, b_soff = 0;  // scalar byte offsets of the reduction step being loaded
    constexpr int NL = C::LOADS_PER_STAGE;
    // One direct-to-LDS load: 16 bytes per lane from descriptor base + off + soff to LDS address
    // M0 + 16 * lane.  Issued through inline assembly on purpose: for a load the compiler knows
    // to write LDS it puts a full vmcnt(0) wait in front of every later transposing LDS read,
    // which stalls the wave for a whole memory latency in every step.  The kernel keeps the
    // ordering itself: the vmcnt(0) wait and the barrier before the last MFMA group of each step.
    // M0 (the LDS destination of the load) is an input operand bound to the physical register, so
    // the compiler writes it itself and knows what the statement reads.
    auto load_lds = [](uint32_t lds_dst, uint32_t off, u32x4_t rsrc, uint32_t soff) __attribute__((always_inline)) {
        asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds"
                     :
                     : "v"(off), "s"(rsrc), "s"(soff), "{m0}"(lds_dst)
                     : "memory");
    };
    // Loads LO..HI-1 of the NL loads that fill stage sa of A and stage s of B with the step at (a_soff, b_soff): the A
    // rounds first, then the B rounds; round j of wave w lands at tile + (j * 512 + w * 64 + lane) * 16.  (LINES: what
    // is loaded of A with a step of B is the stage behind that step's.)
    auto issue_range = [&](auto lo_tag, auto hi_tag, int sa, int s) __attribute__((always_inline)) {
        constexpr int LO = decltype(lo_tag)::value, HI = decltype(hi_tag)::value;
#pragma unroll
        for (int j = LO; j < HI; ++j) {
            if (j < C::A_ROUNDS) {
                load_lds(smem_base + sa * C::A_BYTES + (j * C::THREADS + wave * 64) * 16, a_off[j], a_rsrc, a_soff);
            } else {
                const int jb = j - C::A_ROUNDS;
                load_lds(smem_base + A_STAGES * C::A_BYTES + s * C::B_BYTES + (jb * C::THREADS + wave * 64) * 16,
                         b_off[jb], b_rsrc, b_soff);
            }
        }
    };
    auto advance = [&]() __attribute__((always_inline)) {
        a_soff += a_step;
        b_soff += b_step;
    };
    // A stage's loads are dealt out over three MFMA groups instead of one burst: half right after
    // the barrier that frees the stage, a quarter in each of the first two groups of the next
    // step.  The texture addresser takes one 1 KB wave-load per ~20 cycles, so eight waves that
    // all issue their loads after the barrier block each other (and their MFMAs) for most of a
    // group; the third group of the next step stays free of loads to cover their latency.
    constexpr int E4 = (NL + 1) / 2, E1 = E4 + (NL - E4 + 1) / 2, E2 = NL;

    // One reduction step held in stage s (compile-time).  On entry the fragments of sub-step 0
    // are in register set 0.  The workgroup barrier sits before the last MFMA group: at that
    // point this wave has read all its fragments of stage s and has seen its own copies of stage
    // s^1 land, so after the barrier stage s can be refilled (step j+2) and stage s^1 read.
    // `head`: the previous step began a refill of stage s^1 that this step has to finish;
    // `load`: begin the refill of stage s; `next`: read the first fragments of the next step.
    // Wave priorities fall through the step and are highest right after the barrier: of the two
    // waves of a SIMD the one that lags is then preferred by the MFMA arbiter, which keeps them
    // from serialising (measured: without this one wave of each SIMD waits at the barrier for
    // about 40 % of the step while the other one is starved of MFMA issue slots).
    // A reduction that ends inside the last two steps: what a KC operand's 16-byte chunks hold beyond
    // its end is overwritten with zeros in LDS once the stage has landed, by the lane
    // that fetched them (round j of thread tid filled slot q = j * THREADS + tid of the tile: row
    // q / 8, LDS chunk q % 8, which holds global chunk (q % 8) ^ swz_kc(row), i.e. reduction
    // elements 8 * that onwards).  `step`: 0 for step KT - 2, in stage 0, 1 for step KT - 1, in stage 1.
    auto zero_tail = [&](const int step) __attribute__((always_inline)) {
        auto clear = [&](auto part_tag, auto lines_tag, char* base, const int rounds, const int rem) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < rounds; ++j) {
                const int q = j * C::THREADS + tid, r = q >> 3, cs = q & 7;
                const int phase = decltype(lines_tag)::value ? line_phase(Ab, g.lda, r) : 0;
                const int left = rem - (line_chunk(cs ^ swz_kc(r), phase) << 3);
                u32x4* const p = reinterpret_cast<u32x4*>(base + q * 16);
                if (!decltype(part_tag)::value) {
                    if (left <= 0) *p = u32x4{0u, 0u, 0u, 0u};
                } else if (left < 8) *p = first_elements(left > 0 ? *p : u32x4{0u, 0u, 0u, 0u}, left);
            }
        };
        auto clear_both = [&](auto part_tag) __attribute__((always_inline)) {
            const int rem = g.R - (KT - 2 + step) * TILE_BK;
            if (LINES) {  // stages KT - 2 and KT - 1 of A with step KT - 2 of B, stage KT with step KT - 1
                if (step == 0) clear(part_tag, IC<1>{}, smem, C::A_ROUNDS, rem);
                clear(part_tag, IC<1>{}, smem + (step + 1) * C::A_BYTES, C::A_ROUNDS, rem - TILE_BK);
            } else if (LA == KC) clear(part_tag, IC<0>{}, smem + step * C::A_BYTES, C::A_ROUNDS, rem);
            if (LB == KC) clear(part_tag, IC<0>{}, smem + A_STAGES * C::A_BYTES + step * C::B_BYTES, C::B_ROUNDS, rem);
        };
        // Only a length that is no multiple of 8 ends inside a chunk.  The others do without the code that may read
        // one back: dgrad 8272 x 6328, reduction 712, 125 us with it, 119 without; 9864 x 2568 x 336 45.7 and 42.8; forward
        // 4000 x 6000, reduction 2000, 93.7 and 90.6.
        if (g.R % 8 == 0) clear_both(IC<0>{});
        else clear_both(IC<1>{});
    };
    // `fix` (first of the two tail steps only): stage s^1 holds the last step, which has just
    // landed; its chunks beyond the end of the reduction are zeroed before the barrier publishes it.
    auto step = [&](const int sa, auto s_tag, const bool head, const bool load, const bool next, const bool fix) __attribute__((always_inline)) {
        constexpr int s = decltype(s_tag)::value;
        const int sa_next = sa + 1 < A_STAGES ? sa + 1 : 0, sa_head = sa > 0 ? sa - 1 : A_STAGES - 1;  // of the next step; being filled
        AXO_SETPRIO(2);
        if (head) issue_range(IC<E4>{}, IC<E1>{}, sa_head, s ^ 1);
        read_a(1, sa, 0, 1);
        mfma_group(0, 0, 0);  // (kq 0, ah 0)
        Interleave<N_MFMA, 0, RD_A, 0>::run();
        AXO_SETPRIO(1);
        if (head) {
            issue_range(IC<E1>{}, IC<E2>{}, sa_head, s ^ 1);
            advance();
        }
        read_a(0, sa, 1, 0);
        read_b(1, s, 1);
        mfma_group(1, 0, 1);  // (kq 0, ah 1)
        Interleave<N_MFMA, 0, RD_A + RD_B, 0>::run();
        AXO_SETPRIO(0);
        read_a(1, sa, 1, 1);
        mfma_group(0, 1, 0);  // (kq 1, ah 0)
        Interleave<N_MFMA, 0, RD_A, 0>::run();
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
        if (fix) zero_tail(1);
        __syncthreads();
        AXO_SETPRIO(3);
        if (load) issue_range(IC<0>{}, IC<E4>{}, sa, s);
        if (next) {
            read_a(0, sa_next, 0, 0);
            read_b(0, s ^ 1, 0);
        }
        mfma_group(1, 1, 1);  // (kq 1, ah 1)
        Interleave<N_MFMA, 0, RD_A + RD_B, 0>::run();
    };
    using T0 = std::integral_constant<int, 0>;
    using T1 = std::integral_constant<int, 1>;

    // KT is even and at least 2.  LINES: the walk ends in stages 0 and 1 of A and starts in the one that takes.
    const int first = LINES ? (KT - 2) % 6 / 2 : 0;
    auto a_stage = [&](int n) __attribute__((always_inline)) { return first + n < A_STAGES ? first + n : first + n - A_STAGES; };
    if constexpr (LINES) {
        issue_range(IC<0>{}, IC<C::A_ROUNDS>{}, first, 0);
#pragma unroll
        for (int j = 0; j < C::A_ROUNDS; ++j) a_off[j] = a_later[j];
    }
    issue_range(IC<0>{}, IC<NL>{}, LINES ? a_stage(1) : 0, 0);
    advance();
    issue_range(IC<0>{}, IC<E4>{}, LINES ? a_stage(2) : 1, 1);  // step 0 issues the rest of stage 1
    AXO_WAIT_VMCNT(E4);                                         // what step 0 needs has landed
    __syncthreads();
    read_a(0, first, 0, 0);
    read_b(0, 0, 0);
    if constexpr (LINES) {
        int sa = first;
#pragma nounroll
        for (int n = first; n > 0; --n) {  // (KT - 2) % 6 steps
            step(sa, T0{}, true, true, true, false);
            step(sa + 1 < 3 ? sa + 1 : 0, T1{}, true, true, true, false);
            sa = sa > 0 ? sa - 1 : 2;
        }
        for (int n = (KT - 2) / 6; n > 0; --n) {
            step(0, T0{}, true, true, true, false);
            step(1, T1{}, true, true, true, false);
            step(2, T0{}, true, true, true, false);
            step(0, T1{}, true, true, true, false);
            step(1, T0{}, true, true, true, false);
            step(2, T1{}, true, true, true, false);
        }
    } else {
        for (int j = 0; j + 2 < KT; j += 2) {  // steady state, branch free: steps j, j+1; refills j+2, j+3
            step(0, T0{}, true, true, true, false);
            step(1, T1{}, true, true, true, false);
        }
    }
    // The last two steps: nothing left to load.  Step KT-2 sits in stage 0, landed and published
    // (by the barrier of the step before, or the one above); where the reduction ends inside it
    // its surplus chunks are zeroed now, behind a barrier of their own, and the fragments that
    // were read ahead are read again.
    const bool fix = (LA == KC || LB == KC) && tail;
    if (fix) {
        zero_tail(0);
        __syncthreads();
        read_a(0, 0, 0, 0);
        read_b(0, 0, 0);
    }
    step(0, T0{}, true, false, true, fix);
    step(1, T1{}, false, false, false, false);
    AXO_SETPRIO(0);

    if (i0 + BM <= g.Mo && j0 + BN <= g.No) tile_epilogue<C, LA, LB, PLAIN>(g, acc, i0, j0, wave, wm, wn, lane, smem);
    else tile_epilogue_clipped<C, LA, LB>(g, acc, i0 + wm * C::WTM, j0 + wn * C::WTN, wave, lane, smem);
}

// The same tile on a ring of D stages, for tiles whose step is too short to cover a load's way from HBM: in
// gemm_tile_body the last loads of a stage have little more than half a step to arrive, which a 1.3 us step of
// a 256 x 256 tile covers and the 0.8 us step of a 256 x 128 tile does not once the operands come from HBM.  Here a
// stage is requested D - 1 steps ahead (three stages of a 256 x 128 tile are the LDS of two of a 256 x 256 one).  By whole lines
// (LINES) a step needs the next stage too and a stage is requested D - 2 steps ahead, on a 256 x 128 tile one: as with two
// stages, which is what takes_lines weighs against the lines saved there.
// A step is two MFMA groups (sub-steps of 32); its barrier sits before the second, half of the refill's loads
// right behind it and the other half at the head of the next step, and wave priorities fall through the step, as
// in gemm_tile_body.  (All loads behind the barrier and no priorities: 238 us instead of 216 in the case below.)
// Measured, dgrad 4096 x 2048 with reduction 16384 and cold operands: 280 us with two stages, 216-223 with three;
// dgrad of 4000 x 2000 x 6000 (rows that straddle cache lines) 116 -> 97; with reduction 1536 unchanged (23 us).
// The steps that differ (the last D) are peeled behind a loop without branches.  With their conditions inside one loop the
// masking of the reduction's end, which only the last step needs, joined the path of every step, and behind such a join
// the compiler waits for all LDS reads in flight, those of the other sub-step too.  Peeled: forward 1024 x 1024 with
// reduction 4096 on 64 x 64 tiles 18.7 -> 14.6 us, dgrad 2048^3 on 128 x 128 ones 18.6 -> 16.5, dgrad 4096 x 2048 with
// reduction 6144 on half-width ones 80.3 -> 76.2, 10600 x 7736 with reduction 48 73.4 -> 66.4.
// `tid`: among the threads that work on the tile; `store`: false for a tile whose results are not wanted, as the second of a
// pair of workgroup halves that has none (both halves meet at the same barriers; for tiles below 128 x 128).
template <int BM, int BN, int WGM, int WGN, int D, int LA, int LB, bool LINES = false, bool PLAIN = false>
__device__ __forceinline__ void gemm_ring_body(const GemmArgs& g, const int i0, const int j0, char* smem, const int tid,
                                               const bool store = true) {
    using C = RingCfg<BM, BN, WGM, WGN, D>;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int KT = (g.R + TILE_BK - 1) / TILE_BK;
    // Nothing is under way here, but the compiler does not know that: in gemm_group_kernel it lets the kinds of tiles follow each other and takes
    // what an epilogue of another kind reads for its last outputs to be pending, where those outputs are not stored.  It then waited for that
    // in the loop, s_waitcnt vmcnt(0) in every turn, which empties the ring (half-width forward tiles and pairs; the three
    // products of 4096 x 2048 x 6144 in one chain call 221.1 us, 219.8 without).
    AXO_WAIT_VMCNT(0);

    constexpr bool A_LINES = LINES && LA == KC, B_LINES = LINES && LB == KC;
    constexpr int AHEAD = LINES ? 1 : 0;  // stages that a step needs beyond its own
    const int stages = KT + AHEAD;

    const bf16_t* const Ab = (LA == KC) ? g.A + (int64_t)i0 * g.lda : g.A + i0;
    const bf16_t* const Bb = (LB == KC) ? g.B + (int64_t)j0 * g.ldb : g.B + j0;
    const u32x4_t a_rsrc = tile_rsrc(Ab, operand_bound<LA>(g.lda, min(BM, g.Mo - i0), g.R));
    const u32x4_t b_rsrc = tile_rsrc(Bb, operand_bound<LB>(g.ldb, min(BN, g.No - j0), g.R));
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void_ptr)smem;
    const uint32_t a_step = (uint32_t)((LA == KC) ? TILE_BK * 2 : (int64_t)TILE_BK * g.lda * 2);
    const uint32_t b_step = (uint32_t)((LB == KC) ? TILE_BK * 2 : (int64_t)TILE_BK * g.ldb * 2);
    uint32_t a_off[C::A_ROUNDS], b_off[C::B_ROUNDS];
    uint32_t a_later[C::A_ROUNDS], b_later[C::B_ROUNDS];
    if constexpr (A_LINES) line_load_offsets<C::A_ROUNDS, C::THREADS>(tid, Ab, g.lda, a_off, a_later);
    else load_offsets<BM, LA, C::A_ROUNDS, C::THREADS>(tid, g.lda, a_off);
    if constexpr (B_LINES) line_load_offsets<C::B_ROUNDS, C::THREADS>(tid, Bb, g.ldb, b_off, b_later);
    else load_offsets<BN, LB, C::B_ROUNDS, C::THREADS>(tid, g.ldb, b_off);
    std::conditional_t<A_LINES, LineFragAddr<BM, D>, FragAddr<BM, LA, C::TM>> fra;
    std::conditional_t<B_LINES, LineFragAddr<BN, D>, FragAddr<BN, LB, C::TN>> frb;
    if constexpr (A_LINES) fra.init(wm * C::WTM, lane, 0, Ab, g.lda);
    else fra.init(wm * C::WTM, lane, 0);
    if constexpr (B_LINES) frb.init(wn * C::WTN, lane, D * C::A_BYTES, Bb, g.ldb);
    else frb.init(wn * C::WTN, lane, D * C::A_BYTES);

    f32x4 acc[C::TM][C::TN];
#pragma unroll
    for (int a = 0; a < C::TM; ++a)
#pragma unroll
        for (int b = 0; b < C::TN; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[a][b][e] = 0.0f;
    bf16x8 fa[2][C::TM], fb[2][C::TN];
    auto read = [&](int s, int kq) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < C::TN; ++b) fb[kq][b] = frb.read(smem, s, b, kq);
#pragma unroll
        for (int a = 0; a < C::TM; ++a) fa[kq][a] = fra.read(smem, s, a, kq);
    };
    auto mfma = [&](int kq) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < C::TM; ++a)
#pragma unroll
            for (int b = 0; b < C::TN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[kq][b], fa[kq][a], acc[a][b], 0, 0, 0);
    };
    constexpr int N_MFMA = C::TM * C::TN, RD = (LA == KC ? 1 : 2) * C::TM + (LB == KC ? 1 : 2) * C::TN;
    constexpr int NL = C::A_ROUNDS + C::B_ROUNDS;
    uint32_t a_soff = 0, b_soff = 0;
    auto load_lds = [](uint32_t lds_dst, uint32_t off, u32x4_t rsrc, uint32_t soff) __attribute__((always_inline)) {
        asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds"
                     :
                     : "v"(off), "s"(rsrc), "s"(soff), "{m0}"(lds_dst)
                     : "memory");
    };
    auto issue = [&](auto lo_tag, auto hi_tag, int s) __attribute__((always_inline)) {
        constexpr int LO = decltype(lo_tag)::value, HI = decltype(hi_tag)::value;
#pragma unroll
        for (int j = LO; j < HI; ++j) {
            if (j < C::A_ROUNDS) load_lds(smem_base + s * C::A_BYTES + (j * C::THREADS + wave * 64) * 16, a_off[j], a_rsrc, a_soff);
            else load_lds(smem_base + D * C::A_BYTES + s * C::B_BYTES + ((j - C::A_ROUNDS) * C::THREADS + wave * 64) * 16,
                          b_off[j - C::A_ROUNDS], b_rsrc, b_soff);
        }
        if (HI == NL) {
            a_soff += a_step;
            b_soff += b_step;
        }
    };
    constexpr int NH = (NL + 1) / 2;
    auto mask = [&](int kq, int rem) __attribute__((always_inline)) {
        const int left = rem - kq * 32 - 8 * (lane >> 4);
        if (LA == KC) {
#pragma unroll
            for (int a = 0; a < C::TM; ++a) fa[kq][a] = first_elements(fa[kq][a], left);
        }
        if (LB == KC) {
#pragma unroll
            for (int b = 0; b < C::TN; ++b) fb[kq][b] = first_elements(fb[kq][b], left);
        }
    };
    // One step, held in stage s; `left`: steps left with it, D + 1 for any number above D.  On entry its first fragments are
    // in registers or on their way, and everything is requested but the second half of the last stage.
    auto step = [&](auto s_tag, auto left_tag) __attribute__((always_inline)) {
        constexpr int s = decltype(s_tag)::value, left = decltype(left_tag)::value;
        AXO_SETPRIO(2);
        if (left >= D - AHEAD) issue(IC<NH>{}, IC<NL>{}, (s + D - 1) % D);
        read(s, 1);
        if (left == 1 && (LA == KC || LB == KC) && g.R % TILE_BK != 0) {
            mask(0, g.R % TILE_BK);
            mask(1, g.R % TILE_BK);
        }
        mfma(0);
        Interleave<N_MFMA, 0, RD, 0>::run();
        AXO_SETPRIO(0);
        if (left > 1) {  // what the next step needs has landed, stage s is in registers
            constexpr int in_flight = left >= D - AHEAD ? D - 2 - AHEAD : left > 2 ? left - 2 : 0;
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(in_flight * NL) : "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            AXO_SETPRIO(3);
            if (left > D - AHEAD) issue(IC<0>{}, IC<NH>{}, s);
            read((s + 1) % D, 0);
        }
        mfma(1);
        Interleave<N_MFMA, 0, RD, 0>::run();
    };
    // The walk ends in stage D - 1 and starts in whichever stage that takes, so that the last steps, which differ from the
    // others, exist once, behind a loop without branches.
    static_assert(D >= 3 && D <= 5, "stages of the ring");
    // What SmallEpilogue reads beside the sums is requested ahead of everything else (EARLY) where it is little beside a stage of the
    // operands.  On 128 x 128 tiles pre-activations and old fp32 values are as much as a stage or two, and the reduction would start that
    // much later (dgrad 2048 x 2048 x 1024 through the erf form 14.7 us, 15.4 with them first): those are requested behind it (LATE), and
    // pre-activations of whole tiles a block at a time, by tile_epilogue, where requesting all at once is 2 % slower still (MIXED).
    enum { EARLY, LATE, MIXED };
    constexpr bool SMALL = BM <= 128;
    constexpr int EPILOGUE = BM * BN < 128 * 128 || (LA == KC && LB == MC) ? EARLY : LB == KC ? MIXED : LATE;
    [[maybe_unused]] std::conditional_t<SMALL, SmallEpilogue<C, LA, LB>, char> epilogue;
    if constexpr (SMALL && EPILOGUE == EARLY) epilogue.request(g, i0 + wm * C::WTM, j0 + wn * C::WTN, lane);
    const int lead = KT % D, first = lead > 0 ? D - lead : 0;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        const int s = first + i < D ? first + i : first + i - D;
        if (i < D - 1) {
            if (i < stages) issue(IC<0>{}, IC<NL>{}, s);
        } else if (stages >= D) issue(IC<0>{}, IC<NH>{}, s);  // its first step issues the rest
        if (i > 0) continue;
        if constexpr (A_LINES) {
            a_soff = 0;
#pragma unroll
            for (int j = 0; j < C::A_ROUNDS; ++j) a_off[j] = a_later[j];
        }
        if constexpr (B_LINES) {
            b_soff = 0;
#pragma unroll
            for (int j = 0; j < C::B_ROUNDS; ++j) b_off[j] = b_later[j];
        }
    }
    // The first step waits for what it needs only, also where the whole reduction is requested at once (waiting for
    // all of it made two-step products of up to 256 half-width tiles 2 % slower).
    if (stages >= D) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 2 - AHEAD) * NL + NH) : "memory");
    else if (KT == 4) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NL) : "memory");
    else if (KT == 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NL) : "memory");
    else if (KT == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read(first, 0);
    using More = IC<D + 1>;
    if (KT > D) {
        if constexpr (D > 4) if (lead >= 4) step(IC<D - 4>{}, More{});
        if constexpr (D > 3) if (lead >= 3) step(IC<D - 3>{}, More{});
        if (lead >= 2) step(IC<D - 2>{}, More{});
        if (lead >= 1) step(IC<D - 1>{}, More{});
    }
    for (int n = KT / D; n > 1; --n) {
        step(IC<0>{}, More{});
        step(IC<1>{}, More{});
        step(IC<2>{}, More{});
        if constexpr (D > 3) step(IC<3>{}, More{});
        if constexpr (D > 4) step(IC<4>{}, More{});
    }
    if constexpr (D > 4) if (KT >= 5) step(IC<D - 5>{}, IC<5>{});
    if constexpr (D > 3) if (KT >= 4) step(IC<D - 4>{}, IC<4>{});
    if (KT >= 3) step(IC<D - 3>{}, IC<3>{});
    if (KT >= 2) step(IC<D - 2>{}, IC<2>{});
    step(IC<D - 1>{}, IC<1>{});
    const bool whole = i0 + BM <= g.Mo && j0 + BN <= g.No;
    if constexpr (!SMALL || EPILOGUE == MIXED)
        if (whole) return tile_epilogue<C, LA, LB, PLAIN>(g, acc, i0, j0, wave, wm, wn, lane, smem);
    if constexpr (SMALL) {
        if constexpr (EPILOGUE != EARLY) epilogue.request(g, i0 + wm * C::WTM, j0 + wn * C::WTN, lane);
        __syncthreads();  // all waves are done reading the operand buffers; outside the branch, which the halves of a pair take differently
        if (store) epilogue.finish(g, acc, wave, smem, whole);
    } else tile_epilogue_clipped<C, LA, LB>(g, acc, i0 + wm * C::WTM, j0 + wn * C::WTN, wave, lane, smem);
}

using MixBigCfg = TileCfg<256, 256, 2, 4>;
using MixSmallCfg = RingCfg<256, 128, 4, 2, 3>;
constexpr int MIX_LDS_BYTES = MixBigCfg::LDS_BYTES > MixSmallCfg::LDS_BYTES ? MixBigCfg::LDS_BYTES : MixSmallCfg::LDS_BYTES;
constexpr int LINES_LDS_BYTES = 3 * MixBigCfg::A_BYTES + 2 * MixBigCfg::B_BYTES;
static_assert(LINES_LDS_BYTES >= MIX_LDS_BYTES && LINES_LDS_BYTES <= 160 * 1024, "LDS of one CU");

// Origin of a tile that would reach over the output's edge, moved back inside where that is possible, so that it
// is a whole tile: the elements it then shares with its neighbour are computed twice, by the same instructions
// in the same order, and stored twice with the same bits.  Not for sums that are added to memory, and not where
// the moved origin would break the 16-byte alignment of loads and stores.
template <int BM, int LAYOUT>
__device__ __forceinline__ int inside_row(const GemmArgs& g, const int i0) {
    const bool ok = g.Mo >= BM && g.epilogue != EPI_ACC_F32 && (LAYOUT == KC || g.Mo % 8 == 0);
    return ok ? min(i0, g.Mo - BM) : i0;
}
template <int BN>
__device__ __forceinline__ int inside_col(const GemmArgs& g, const int j0) {
    return g.No >= BN && g.epilogue != EPI_ACC_F32 && g.No % 8 == 0 ? min(j0, g.No - BN) : j0;
}

// One launch over both regions of a TileSched.  LINES: rows by whole lines on no tiles (0), on the large ones (1), on both (2).  PLAIN: stores of whole
// tiles (store_row).
template <int LA, int LB, int LINES, bool PLAIN>
__global__ void __launch_bounds__(TILE_THREADS, 1) gemm_mixed_kernel(GemmArgs g, TileSched sc) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int bid = blockIdx.x;
    start_shift(bid, sc.shift);
    int tm, tn;
    if (bid < sc.n_big) {
        tile_of_index(xcd_run(bid, sc.n_big), sc.tiles_m, sc.big_cols, sc.group_m, tm, tn);
        gemm_tile_body<256, 256, 2, 4, LA, LB, LINES != 0, PLAIN>(g, inside_row<256, LA>(g, tm * 256), inside_col<256>(g, tn * 256), smem);
    } else {
        const int n_small = (int)gridDim.x - sc.n_big;
        tile_of_index(xcd_run(bid - sc.n_big, n_small), sc.tiles_m, sc.small_cols, sc.group_m, tm, tn);
        gemm_ring_body<256, 128, 4, 2, 3, LA, LB, LINES == 2, PLAIN>(g, inside_row<256, LA>(g, tm * 256), inside_col<128>(g, sc.big_cols * 256 + tn * 128), smem, threadIdx.x);
    }
}

// One product on 128 x 128 tiles, eight waves of 32 x 64 each on a four-stage ring, for outputs of at most one
// such tile per CU (4096 x 1024, 2048 x 2048): 256-row tiles leave most CUs without work there.  A step is bound by
// the rate at which a CU takes in operands (32 KB per 515 cycles of MFMA; see gemm_rect_kernel), so this is no tile for
// larger outputs.  Eight waves rather than four of 64 x 64 (a quarter less LDS traffic, but one wave per SIMD: 2048^3 21 us), four stages rather than two
// and two workgroups per CU (24 us).  Measured against the 256-row tiles, forward / dgrad / wgrad: 2048^3
// 25.6 / 24.9 / 24.2 -> 18.2 / 17.4 / 18.2 us, 1536^3 19.6 / 19.0 / 18.4 -> 12.1 / 12.4 / 12.1, wgrad 1536 x 1536 of 4096
// tokens 44 -> 30.  Sums run in the same order as on the other tiles: same bits.
using MidCfg = RingCfg<128, 128, 4, 2, 4>;
template <int LA, int LB, bool LINES>
__global__ void __launch_bounds__(TILE_THREADS, 1) gemm_mid_kernel(GemmArgs g, int tiles_m, int tiles_n, int group_m) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int tm, tn;
    tile_of_index(xcd_run(blockIdx.x, gridDim.x), tiles_m, tiles_n, group_m, tm, tn);
    gemm_ring_body<128, 128, 4, 2, 4, LA, LB, LINES>(g, inside_row<128, LA>(g, tm * 128), inside_col<128>(g, tn * 128), smem, threadIdx.x);
}

// Between those and 64 x 64 ones: 64 x 128 and 128 x 64 tiles, eight waves of 32 x 32 on a four-stage ring, for outputs of at most one
// such tile per CU that are more than one round of 64 x 64 tiles.  A CU takes in operands at 100-115 KB per us, whatever the depth of
// the ring, and that is what these launches are bound by (the loads of a 128 x 128 tile's step alone take 0.31 us, its MFMAs 0.22): half
// as many CUs on 128 x 128 tiles take in two thirds of the bytes, two rounds of 64 x 64 tiles a third more.  64 x 64 / 128 x 128 / these in us:
// forward 1000 x 2000 x 3000 23.9 / 22.7 / 19.9, dgrad 512 x 4096 x 4096 23.8 / 24.0 / 19.9, 256 x 8192 x 8192 71 / 73 / 58, wgrad 1400^3 15.0 / 13.5 / 11.8,
// 900 x 1300 of 6000 tokens 56 / 44 / 38, forward 2000 x 1000 x 1000 10.7 / 10.8 / 9.6.  Three stages and two workgroups per CU: the same.
template <bool WIDE>
using RectCfg = RingCfg<WIDE ? 64 : 128, WIDE ? 128 : 64, WIDE ? 2 : 4, WIDE ? 4 : 2, 4>;
template <int LA, int LB, bool WIDE, bool LINES>
__global__ void __launch_bounds__(TILE_THREADS, 1) gemm_rect_kernel(GemmArgs g, int tiles_m, int tiles_n, int group_m) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    constexpr int BM = WIDE ? 64 : 128, BN = WIDE ? 128 : 64;
    int tm, tn;
    tile_of_index(xcd_run(blockIdx.x, gridDim.x), tiles_m, tiles_n, group_m, tm, tn);
    gemm_ring_body<BM, BN, WIDE ? 2 : 4, WIDE ? 4 : 2, 4, LA, LB, LINES>(g, inside_row<BM, LA>(g, tm * BM), inside_col<BN>(g, tn * BN), smem, threadIdx.x);
}

// The same for smaller outputs: 64 x 64, four waves of 32 x 32 on a four-stage ring, two workgroups per CU.  (Five stages are
// what two workgroups leave room for; they pay where a step needs two of them: 12.0 -> 9.3 us instead of 10.8 for dgrad 1024 x 1024
// with 32 steps and rows 16 bytes off.)  Measured
// against the small tiles whose waves split the reduction (gemm_slim.hpp), forward / dgrad / wgrad: 2048 x 1024 x 1024
// 11.9 / 12.1 / 11.5 -> 8.7 / 8.2 / 9.0 us, 1000^3 10.0 / 9.6 / 10.2 -> 7.3 / 6.6 / 7.9, wgrad 1024 x 1024 of 8192 tokens 29
// both (128 x 128 tiles: 51).  Those stay quicker below some 100 tiles (300^3 3.7 against 5.4).
template <bool LINES>
using SmallCfg = RingCfg<64, 64, 2, 2, LINES ? 5 : 4>;
template <int LA, int LB, bool LINES>
__global__ void __launch_bounds__(256, 2) gemm_small_kernel(GemmArgs g, int tiles_m, int tiles_n, int group_m) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int tm, tn;
    tile_of_index(xcd_run(blockIdx.x, gridDim.x), tiles_m, tiles_n, group_m, tm, tn);
    gemm_ring_body<64, 64, 2, 2, LINES ? 5 : 4, LA, LB, LINES>(g, inside_row<64, LA>(g, tm * 64), inside_col<64>(g, tn * 64), smem, threadIdx.x);
}

}  // namespace axo
