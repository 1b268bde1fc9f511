// Small-tile bf16 MFMA GEMM for gfx950: any Mo, No, R, every edge handled in the kernel.
//   C[Mo x No] = sum_r A(i, r) * B(j, r)
//
// For products whose output is so small, or whose batch is so short, that the tiles of gemm_tile.hpp come to a
// few workgroups with a long serial reduction each.  Such a product is bound by latency and by how fast one CU pulls operands in (a 1 KB wave-load per
// about 20 cycles), so the waves of a workgroup split the REDUCTION of one BM x BN tile between them:
// wave w takes the 64-wide reduction chunks w, w + NW, w + 2 NW, ...  A wave copies its chunks into LDS
// that nobody else touches, so the main loop has no workgroup barrier: it waits for its own loads
// only, and the waves of a CU drift apart and cover each other's latency.  Splitting the reduction also
// means that every LDS byte is read once (a tile shared by a 2 x 2 arrangement of waves reads each
// operand twice).  The partial tiles are added through LDS in ascending wave order: no atomics, the
// result is a fixed function of the input.
//
// A chunk's fragments go to registers before the next one is requested into the same bytes.  On a busy CU one
// LDS stage per wave is best: what hides the latency is the other waves, and a second stage halves the
// workgroups that fit beside each other and with them what overlaps a workgroup's start and end (64 x 64 tiles,
// 2048^3: 38 us with two stages and one workgroup per CU, 28 with one stage and two; 4096 x 1536 x 1536: 48 and
// 32).  A long reduction on at most two 32 x 32 tiles per CU has nothing beside it and takes two stages (dgrad of
// 16 x 2048 x 6144: 13.3 us with one, 9.8 with two; forward of 128 x 9088 x 640: 22.7 and 19.7).
//
// Edges cost nothing in the loop.  Loads go through a buffer descriptor whose bound is the last
// valid element of the operand's tile (rounded up to the dword the range check works in), so rows beyond
// the matrix read as zeros; columns beyond it read whatever the row pitch holds and only reach outputs
// that are not stored.  The one thing a linear bound cannot mask, the end of a reduction that runs inside
// the rows (KC), is masked in registers in the last chunk, on both operands (a zero times a stray infinity
// would be a NaN).
//
// Measured, kernel time of forward / dgrad / wgrad: 96 x 2048 x 6144 11.7 / 11.6 / - us (the general kernel
// took 130 / 238), 77 x 1000 x 48 4.2 / 3.1 / 3.0 (56 / 15 / 19), 256^3 3.3 / 3.3 / 3.2 (256 x 128 tiles: 5.3 each).
#pragma once
#include "gemm_tile.hpp"

namespace axo {

// One operand of a tile as one wave sees it: ROWS output rows (or columns) by 64 reduction elements.
template <int ROWS, int LAYOUT>
struct SlimOperand {
    static constexpr int BYTES = ROWS * TILE_BK * 2;
    static constexpr int LOADS = BYTES / 1024;  // wave-loads of 16 bytes per lane
    static constexpr int NT = ROWS / 16;        // MFMA tiles
    static constexpr int NA = LAYOUT == KC ? 2 : NT;
    uint32_t off[LOADS];  // per-lane byte offset of the chunk fetched by load j, from the tile origin
    uint32_t addr[NA];    // per-lane LDS byte offset of a fragment, from the operand's stage

    __device__ __forceinline__ void init(int lane, int64_t ld) {
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int q = j * 64 + lane;
            if (LAYOUT == KC) {
                const int r = q >> 3, cs = q & 7;
                off[j] = (uint32_t)(((int64_t)r * ld + ((cs ^ swz_kc(r)) << 3)) * 2);
            } else {
                constexpr int CPR = ROWS / 8;
                const int k = q / CPR, cs = q % CPR;
                off[j] = (uint32_t)(((int64_t)k * ld + ((cs ^ swz_mc<ROWS>(k)) << 3)) * 2);
            }
        }
        if (LAYOUT == KC) {
            const int r = lane & 15;
#pragma unroll
            for (int kq = 0; kq < 2; ++kq) addr[kq] = r * (TILE_BK * 2) + (((kq * 4 + (lane >> 4)) ^ swz_kc(r)) << 4);
        } else {
            const int i = lane & 15, krow = ((lane >> 4) << 3) + (i >> 2);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int n = t * 16 + ((i & 3) << 2);
                addr[t % NA] = krow * (ROWS * 2) + (((n >> 3) ^ swz_mc<ROWS>(krow)) << 4) + (((n >> 2) & 1) << 3);
            }
        }
    }
    // fragment of MFMA tile t, 32-wide sub-step kq, of the stage at `stage`
    __device__ __forceinline__ bf16x8 read(const char* stage, int t, int kq) const {
        if (LAYOUT == KC) {
            return *reinterpret_cast<const bf16x8*>(stage + addr[kq] + t * (16 * TILE_BK * 2));
        } else {
            typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
            const char* p = stage + addr[t % NA] + kq * (32 * ROWS * 2);
            union { struct { s16x4 a, b; } s; bf16x8 v; } u;
            u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
            u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * (ROWS * 2)));
            return u.v;
        }
    }
    static __device__ __forceinline__ const bf16_t* origin(const bf16_t* p, int64_t ld, int i0) {
        return LAYOUT == KC ? p + (int64_t)i0 * ld : p + i0;
    }
    static __device__ __forceinline__ uint32_t chunk_step(int64_t ld) {
        return (uint32_t)(LAYOUT == KC ? TILE_BK * 2 : (int64_t)TILE_BK * ld * 2);
    }
};

constexpr int SLIM_WAVES = 4;

template <int BM, int BN, int NW, int ST>
struct SlimCfg {
    static constexpr int THREADS = NW * 64;
    static constexpr int STAGE_BYTES = (BM + BN) * TILE_BK * 2;
    static constexpr int PART_STRIDE = BN + 4;  // floats per row of a partial tile (padded)
    static constexpr int PART_BYTES = BM * PART_STRIDE * 4;
    static constexpr int WAVE_BYTES = ST * STAGE_BYTES > PART_BYTES ? ST * STAGE_BYTES : PART_BYTES;
    static constexpr int LDS_BYTES = NW * WAVE_BYTES;
    static_assert(BM % 32 == 0 && BN % 32 == 0 && LDS_BYTES <= 160 * 1024, "LDS of one CU");
};

// One tile; tid: 0 .. NW * 64 - 1 among the threads that work on it.  Holds exactly one workgroup barrier.
template <int BM, int BN, int NW, int ST, int LA, int LB>
__device__ __forceinline__ void slim_tile_body(const GemmArgs& g, const int i0, const int j0, const int tid, char* smem) {
    using C = SlimCfg<BM, BN, NW, ST>;
    using OA = SlimOperand<BM, LA>;
    using OB = SlimOperand<BN, LB>;
    constexpr int TM = BM / 16, TN = BN / 16;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KT = (g.R + TILE_BK - 1) / TILE_BK;

    OA oa;
    OB ob;
    oa.init(lane, g.lda);
    ob.init(lane, g.ldb);
    const u32x4_t a_rsrc = tile_rsrc(OA::origin(g.A, g.lda, i0), operand_bound<LA>(g.lda, min(BM, g.Mo - i0), g.R));
    const u32x4_t b_rsrc = tile_rsrc(OB::origin(g.B, g.ldb, j0), operand_bound<LB>(g.ldb, min(BN, g.No - j0), g.R));
    const uint32_t a_step = OA::chunk_step(g.lda), b_step = OB::chunk_step(g.ldb);
    char* const mine = smem + wave * C::WAVE_BYTES;
    const uint32_t mine_lds = (uint32_t)(uintptr_t)(lds_void_ptr)smem + wave * C::WAVE_BYTES;

    // one direct-to-LDS load: 16 bytes per lane to LDS address M0 + 16 * lane (see gemm_tile_body)
    auto load_lds = [](uint32_t lds_dst, uint32_t off, u32x4_t rsrc, uint32_t soff) __attribute__((always_inline)) {
        asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds"
                     :
                     : "v"(off), "s"(rsrc), "s"(soff), "{m0}"(lds_dst)
                     : "memory");
    };
    auto issue = [&](const int s, const int chunk) __attribute__((always_inline)) {
        const uint32_t a_soff = (uint32_t)chunk * a_step, b_soff = (uint32_t)chunk * b_step;
        const uint32_t dst = mine_lds + s * C::STAGE_BYTES;
#pragma unroll
        for (int j = 0; j < OA::LOADS; ++j) load_lds(dst + j * 1024, oa.off[j], a_rsrc, a_soff);
#pragma unroll
        for (int j = 0; j < OB::LOADS; ++j) load_lds(dst + OA::BYTES + j * 1024, ob.off[j], b_rsrc, b_soff);
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[a][b][e] = 0.0f;

    // One chunk, held in stage s (compile-time); the stages of a wave are filled in turn.
    auto chunk_step = [&](auto s_tag, const int chunk) __attribute__((always_inline)) {
        constexpr int s = decltype(s_tag)::value;
        if (ST == 2 && chunk + NW < KT) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(OA::LOADS + OB::LOADS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const char* const stage = mine + s * C::STAGE_BYTES;
        bf16x8 fa[2][TM], fb[2][TN];
#pragma unroll
        for (int kq = 0; kq < 2; ++kq) {
#pragma unroll
            for (int a = 0; a < TM; ++a) fa[kq][a] = oa.read(stage, a, kq);
#pragma unroll
            for (int b = 0; b < TN; ++b) fb[kq][b] = ob.read(stage + OA::BYTES, b, kq);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the stage is in registers: refill it
        if (chunk + ST * NW < KT) issue(s, chunk + ST * NW);
        if ((LA == KC || LB == KC) && (g.R % TILE_BK) != 0 && chunk == KT - 1) {
            const int left = g.R - chunk * TILE_BK - 8 * (lane >> 4);  // from this lane's 8 elements of sub-step 0
#pragma unroll
            for (int kq = 0; kq < 2; ++kq) {
                if (LA == KC) {
#pragma unroll
                    for (int a = 0; a < TM; ++a) fa[kq][a] = first_elements(fa[kq][a], left - kq * 32);
                }
                if (LB == KC) {
#pragma unroll
                    for (int b = 0; b < TN; ++b) fb[kq][b] = first_elements(fb[kq][b], left - kq * 32);
                }
            }
        }
#pragma unroll
        for (int kq = 0; kq < 2; ++kq)
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[kq][b], fa[kq][a], acc[a][b], 0, 0, 0);
    };
    if (wave < KT) issue(0, wave);
    if (ST == 2 && wave + NW < KT) issue(1, wave + NW);

    // The outputs of a thread, four consecutive columns of a row at a time.  What its epilogue reads from memory beside the sums is
    // requested here, whole quads of it, and kept as it comes, so that it arrives during the reduction.  (Read when it was wanted, every
    // quad waited for its own load, behind the store of the one before: 2.5 us of forward 96 x 2048 x 6144 with bias and GELU lay between
    // the addition and the last store.  With this and one decision per tile, below, it takes 10.9 us instead of 12.2, its data gradient
    // through the activation 11.4 instead of 11.8.)  The waits of the loop count these loads, too, which makes them no weaker.
    constexpr int QPR = BN / 4, ROUNDS = BM * QPR / C::THREADS;  // quads of columns per row, per thread
    static_assert(BM * QPR % C::THREADS == 0, "whole rounds of quads");
    auto quad_row = [&](int i) __attribute__((always_inline)) { return (i * C::THREADS + tid) / QPR; };
    auto quad_col = [&](int i) __attribute__((always_inline)) { return (i * C::THREADS + tid) % QPR * 4; };
    constexpr bool FWD = LA == KC && LB == MC, DGRAD = LA == KC && LB == KC;
    const bool has_extra = FWD ? g.epilogue != EPI_NONE && g.add_bias : g.epilogue != EPI_NONE;
    u32x4 early[ROUNDS];  // four bf16 values in the first two dwords, or four fp32 ones
    if (has_extra) {
#pragma unroll
        for (int i = 0; i < ROUNDS; ++i) {
            const int row = i0 + quad_row(i), col = j0 + quad_col(i);
            early[i] = u32x4{0u, 0u, 0u, 0u};
            if (row >= g.Mo || col + 4 > g.No) continue;
            if (FWD || DGRAD) {
                const uint2 raw = *reinterpret_cast<const uint2*>(FWD ? g.bias + col : g.aux + (int64_t)row * g.ldaux + col);
                early[i][0] = raw.x;
                early[i][1] = raw.y;
            } else early[i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const float*>(g.C) + (int64_t)row * g.ldc + col);
        }
    }
    for (int chunk = wave; chunk < KT; chunk += ST * NW) {
        chunk_step(IC<0>{}, chunk);
        if (ST == 2 && chunk + NW < KT) chunk_step(IC<ST - 1>{}, chunk + NW);
    }

    // Partial tiles to LDS (each wave inside its own region, whose loads have all landed and been read),
    // then every thread adds the partials of its outputs, four consecutive columns at a time.
    // acc[a][b][e] is element (a * 16 + lane % 16, b * 16 + 4 * (lane / 16) + e) of the tile.
    const int n_part = min(NW, KT);
    if (wave < n_part) {
        float* part = reinterpret_cast<float*>(mine);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
                *reinterpret_cast<f32x4*>(part + (a * 16 + (lane & 15)) * C::PART_STRIDE + b * 16 + 4 * (lane >> 4)) = acc[a][b];
    }
    __syncthreads();
    auto each_quad = [&](auto store) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ROUNDS; ++i) {
            const int row = i0 + quad_row(i), col = j0 + quad_col(i);
            f32x4 sum = {0.f, 0.f, 0.f, 0.f};
            const char* const parts = smem + (quad_row(i) * C::PART_STRIDE + quad_col(i)) * 4;
            if (n_part == NW) {  // reads that do not wait for each other
#pragma unroll
                for (int w = 0; w < NW; ++w) sum += *reinterpret_cast<const f32x4*>(parts + w * C::WAVE_BYTES);
            } else
                for (int w = 0; w < n_part; ++w) sum += *reinterpret_cast<const f32x4*>(parts + w * C::WAVE_BYTES);
            if (row < g.Mo && col < g.No) store(i, row, col, min(4, g.No - col), sum);
        }
    };
    // The kind is decided once, ahead of the quads, and a product compiles only its own kinds: little code, which a short kernel fetches
    // while it runs it.
    auto plain = [&]() __attribute__((always_inline)) {
        each_quad([&](int, int row, int col, int valid, f32x4 sum) __attribute__((always_inline)) { store_bf16_quad(g, sum, row, col, valid); });
    };
    auto with = [&](auto f) __attribute__((always_inline)) {  // f(sum, what is read for it) of every value
        each_quad([&](int i, int row, int col, int valid, f32x4 sum) __attribute__((always_inline)) {
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
            if (has_extra) {
                x = bf16x4_of(early[i][0], early[i][1]);
                if (valid < 4) x = load_bf16x4(FWD ? g.bias + col : g.aux + (int64_t)row * g.ldaux + col, valid);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = f(sum[e], x[e]);
            store_bf16_quad(g, sum, row, col, valid);
        });
    };
    if constexpr (FWD) switch (g.epilogue) {
        case EPI_NONE: return plain();
        case EPI_BIAS: return with([](float s, float x) { return apply_epilogue(s, x, EPI_BIAS); });
        case EPI_BIAS_GELU_TANH: return with([](float s, float x) { return apply_epilogue(s, x, EPI_BIAS_GELU_TANH); });
        default: return with([](float s, float x) { return apply_epilogue(s, x, EPI_BIAS_GELU_ERF); });
    } else if constexpr (DGRAD) switch (g.epilogue) {
        case EPI_NONE: return plain();
        case EPI_MUL_DGELU_TANH: return with([](float s, float x) { return apply_dact(s, x, EPI_MUL_DGELU_TANH); });
        default: return with([](float s, float x) { return apply_dact(s, x, EPI_MUL_DGELU_ERF); });
    } else {
        if (g.epilogue == EPI_NONE) return plain();
        each_quad([&](int i, int row, int col, int valid, f32x4 sum) __attribute__((always_inline)) {
            f32x4 x = __builtin_bit_cast(f32x4, early[i]);
            if (valid < 4) x = load_f32x4(reinterpret_cast<const float*>(g.C) + (int64_t)row * g.ldc + col, valid);
            store_f32_quad(g, x + sum, row, col, valid);
        });
    }
}

// How a product is cut: tiles_m x tiles_n workgroups, tiles ordered in bands of group_m tile rows.
struct SlimSched {
    int tiles_m, tiles_n, group_m;
};

template <int BM, int BN, int NW, int ST, int LA, int LB>
__global__ void __launch_bounds__(NW * 64) gemm_slim_kernel(GemmArgs g, SlimSched sc) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int tm, tn;
    tile_of_index(xcd_run(blockIdx.x, gridDim.x), sc.tiles_m, sc.tiles_n, sc.group_m, tm, tn);
    slim_tile_body<BM, BN, NW, ST, LA, LB>(g, tm * BM, tn * BN, threadIdx.x, smem);
}

}  // namespace axo
