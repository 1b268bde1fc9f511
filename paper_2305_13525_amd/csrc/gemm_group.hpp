// Grouped launches for gfx950: the tiles of several independent products of a chain in one grid, larger tiles
// (gemm_tile.hpp) and small ones (gemm_slim.hpp), and the strips of a bias gradient (bias_grad.hpp).
#pragma once
#include "bias_grad.hpp"
#include "gemm_slim.hpp"
#include "gemm_tile.hpp"

namespace axo {

// ---- grouped launch: the tiles of several independent products in one grid ----------------
// A product on its own often cannot fill the 256 CUs (a 1536x1536 output is 36 big tiles), and a
// chain of such launches pays a ramp-up and a tail each.  A group launch strings the tile lists of
// up to GROUP_MAX_PRODUCTS products together: the grid is cut into segments, a segment is all the
// tiles of one size of one product, and segments are ordered by decreasing tile cost so that the
// in-order workgroup dispatch approximates longest-processing-time-first scheduling.  One of the
// slots may instead hold a bias gradient, whose 64-column strips form one more (cheap, hence
// late) segment of memory-bound workgroups.
constexpr int GROUP_MAX_PRODUCTS = 12;
constexpr int GROUP_MAX_SEGMENTS = 2 * GROUP_MAX_PRODUCTS;

struct GroupSeg {
    int first_block;  // first workgroup id of the segment
    int n_blocks;
    int product;      // index into GroupArgs::g
    int kind;         // 2 * layout pair (0: KC/MC, 1: KC/KC, 2: MC/MC) + (1 if 256x128 tiles);
                      // GROUP_KIND_BIAS_GRAD: 64-column strips of a bias gradient; GROUP_KIND_SLIM + layout
                      // pair: pairs of small tiles; GROUP_KIND_LINES + a kind of tiles: rows fetched by whole cache lines
    int tiles_m;      // tile rows
    int cols;         // tile columns of this segment
    int col0;         // first output column of this segment
    int group_m;      // band height of the tile order
};

constexpr int GROUP_KIND_BIAS_GRAD = 6;
constexpr int GROUP_KIND_SLIM = 7;  // + layout pair: 64 x 64 tiles of gemm_slim.hpp, two per workgroup
constexpr int GROUP_KIND_PAIR = 10;  // + layout pair: 64 x 64 tiles of a ring, two per workgroup
constexpr int GROUP_KIND_LINES = 16;
constexpr int GROUP_BIAS_COLS = 64;

struct GroupArgs {
    int n_seg;
    GroupSeg seg[GROUP_MAX_SEGMENTS];
    GemmArgs g[GROUP_MAX_PRODUCTS];
};

// LINES: some segments are of a GROUP_KIND_LINES.  (A kernel of its own, so that the others keep their LDS size and registers.)
template <bool LINES>
__global__ void __launch_bounds__(TILE_THREADS, 1) gemm_group_kernel(GroupArgs ga) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int bid = blockIdx.x;
    int si = 0;
    for (int i = 1; i < ga.n_seg; ++i)
        if (bid >= ga.seg[i].first_block) si = i;
    const GroupSeg sg = ga.seg[si];
    const GemmArgs g = ga.g[sg.product];
    if (sg.kind == GROUP_KIND_BIAS_GRAD) {
        // A bias gradient rides along: memory-bound strips that fill CUs the products leave idle
        // towards the end of the launch.  Its arguments travel in a GemmArgs: A = dY, C = db (fp32),
        // Mo = rows, No = columns, epilogue = accumulate flag.
        BiasGradArgs bg;
        bg.dY = g.A;
        bg.lddy = g.lda;
        bg.db = reinterpret_cast<float*>(g.C);
        bg.M = g.Mo;
        bg.Nl = g.No;
        bg.accumulate = g.epilogue;
        bias_grad_strip<GROUP_BIAS_COLS, TILE_THREADS>(bg, bid - sg.first_block, reinterpret_cast<float*>(smem));
        return;
    }
    if (sg.kind >= GROUP_KIND_SLIM && sg.kind < GROUP_KIND_PAIR) {
        // A product on small tiles rides along: four waves per tile, two tiles per workgroup, each in its half of
        // the LDS.  (tiles_m x cols tiles; the second half of the last workgroup of an odd count runs on an empty
        // matrix, barrier included.)
        using C = SlimCfg<64, 64, SLIM_WAVES, 1>;
        static_assert(2 * C::THREADS == TILE_THREADS && 2 * C::LDS_BYTES <= MIX_LDS_BYTES, "two tiles per workgroup");
        const int half = __builtin_amdgcn_readfirstlane(threadIdx.x / C::THREADS), tiles = sg.tiles_m * sg.cols;
        const int t = 2 * xcd_run(bid - sg.first_block, sg.n_blocks) + half;
        int tm, tn;
        tile_of_index(min(t, tiles - 1), sg.tiles_m, sg.cols, sg.group_m, tm, tn);
        GemmArgs h = g;
        if (t >= tiles) h.Mo = h.No = h.R = 0;
        char* const lds = smem + half * C::LDS_BYTES;
        const int tid = threadIdx.x % C::THREADS;
        switch (sg.kind - GROUP_KIND_SLIM) {
            case 0: slim_tile_body<64, 64, SLIM_WAVES, 1, KC, MC>(h, tm * 64, tn * 64, tid, lds); break;
            case 1: slim_tile_body<64, 64, SLIM_WAVES, 1, KC, KC>(h, tm * 64, tn * 64, tid, lds); break;
            default: slim_tile_body<64, 64, SLIM_WAVES, 1, MC, MC>(h, tm * 64, tn * 64, tid, lds); break;
        }
        return;
    }
    if (sg.kind >= GROUP_KIND_PAIR && sg.kind < GROUP_KIND_LINES) {
        // Two 64 x 64 tiles of a product, each on four waves and in its half of the LDS; the halves take the same number of
        // steps, so they share the barriers of both walks.
        using C = SmallCfg<false>;
        static_assert(2 * C::THREADS == TILE_THREADS && 2 * C::LDS_BYTES <= MIX_LDS_BYTES, "two tiles per workgroup");
        const int half = __builtin_amdgcn_readfirstlane(threadIdx.x / C::THREADS), tiles = sg.tiles_m * sg.cols;
        const int t = 2 * xcd_run(bid - sg.first_block, sg.n_blocks) + half, tid = threadIdx.x % C::THREADS;
        int tm, tn;
        tile_of_index(min(t, tiles - 1), sg.tiles_m, sg.cols, sg.group_m, tm, tn);
        char* const lds = smem + half * C::LDS_BYTES;
        const int j0 = inside_col<64>(g, tn * 64);
        switch (sg.kind - GROUP_KIND_PAIR) {
            case 0: gemm_ring_body<64, 64, 2, 2, 4, KC, MC>(g, inside_row<64, KC>(g, tm * 64), j0, lds, tid, t < tiles); break;
            case 1: gemm_ring_body<64, 64, 2, 2, 4, KC, KC>(g, inside_row<64, KC>(g, tm * 64), j0, lds, tid, t < tiles); break;
            default: gemm_ring_body<64, 64, 2, 2, 4, MC, MC>(g, inside_row<64, MC>(g, tm * 64), j0, lds, tid, t < tiles); break;
        }
        return;
    }
    int tm, tn;
    // workgroup ids with equal id % 8 share an XCD whatever the segment's first id is
    tile_of_index(xcd_run(bid - sg.first_block, sg.n_blocks), sg.tiles_m, sg.cols, sg.group_m, tm, tn);
    if constexpr (LINES) {
        switch (sg.kind - GROUP_KIND_LINES) {
            case 0: gemm_tile_body<256, 256, 2, 4, KC, MC, true>(g, inside_row<256, KC>(g, tm * 256), inside_col<256>(g, sg.col0 + tn * 256), smem); return;
            case 2: gemm_tile_body<256, 256, 2, 4, KC, KC, true>(g, inside_row<256, KC>(g, tm * 256), inside_col<256>(g, sg.col0 + tn * 256), smem); return;
            case 3: gemm_ring_body<256, 128, 4, 2, 3, KC, KC, true>(g, inside_row<256, KC>(g, tm * 256), inside_col<128>(g, sg.col0 + tn * 128), smem, threadIdx.x); return;
            default: break;
        }
    }
    switch (sg.kind) {
        case 0: gemm_tile_body<256, 256, 2, 4, KC, MC>(g, inside_row<256, KC>(g, tm * 256), inside_col<256>(g, sg.col0 + tn * 256), smem); break;
        case 1: gemm_ring_body<256, 128, 4, 2, 3, KC, MC>(g, inside_row<256, KC>(g, tm * 256), inside_col<128>(g, sg.col0 + tn * 128), smem, threadIdx.x); break;
        case 2: gemm_tile_body<256, 256, 2, 4, KC, KC>(g, inside_row<256, KC>(g, tm * 256), inside_col<256>(g, sg.col0 + tn * 256), smem); break;
        case 3: gemm_ring_body<256, 128, 4, 2, 3, KC, KC>(g, inside_row<256, KC>(g, tm * 256), inside_col<128>(g, sg.col0 + tn * 128), smem, threadIdx.x); break;
        case 4: gemm_tile_body<256, 256, 2, 4, MC, MC>(g, inside_row<256, MC>(g, tm * 256), inside_col<256>(g, sg.col0 + tn * 256), smem); break;
        default: gemm_ring_body<256, 128, 4, 2, 3, MC, MC>(g, inside_row<256, MC>(g, tm * 256), inside_col<128>(g, sg.col0 + tn * 128), smem, threadIdx.x); break;
    }
}

// The same for products that all run on small tiles, at a small tile's own launch geometry: on its
// own a product of a few dozen tiles leaves most of the chip idle, and a chain of such launches pays a start and
// an end each.  Blocks of four layers, whose products take these two kinds of group, against one launch per product: 64 tokens
// of width 256 12.3 us and 43.9, 512 of width 512 24.5 and 58.9.
constexpr int SLIM_GROUP_MAX = 12;
struct SlimGroupArgs {
    int n;
    int first_block[SLIM_GROUP_MAX];  // ascending; products with the longest reductions come first
    int pair[SLIM_GROUP_MAX];         // layouts, 0: KC/MC, 1: KC/KC, 2: MC/MC
    SlimSched sched[SLIM_GROUP_MAX];
    GemmArgs g[SLIM_GROUP_MAX];
};

template <int ROWS>
__global__ void __launch_bounds__(SLIM_WAVES * 64) gemm_slim_group_kernel(SlimGroupArgs ga) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int k = 0;
    for (int i = 1; i < ga.n; ++i)
        if ((int)blockIdx.x >= ga.first_block[i]) k = i;
    const SlimSched sc = ga.sched[k];
    const GemmArgs g = ga.g[k];
    int tm, tn;
    tile_of_index(xcd_run((int)blockIdx.x - ga.first_block[k], sc.tiles_m * sc.tiles_n), sc.tiles_m, sc.tiles_n, sc.group_m, tm, tn);
    switch (ga.pair[k]) {
        case 0: slim_tile_body<ROWS, ROWS, SLIM_WAVES, 1, KC, MC>(g, tm * ROWS, tn * ROWS, threadIdx.x, smem); break;
        case 1: slim_tile_body<ROWS, ROWS, SLIM_WAVES, 1, KC, KC>(g, tm * ROWS, tn * ROWS, threadIdx.x, smem); break;
        default: slim_tile_body<ROWS, ROWS, SLIM_WAVES, 1, MC, MC>(g, tm * ROWS, tn * ROWS, threadIdx.x, smem); break;
    }
}

}  // namespace axo
