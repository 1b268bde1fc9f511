// C ABI of the shard-GEMM library: host-side validation, shard derivation, kernel selection and
// launch.  Every check runs before the first HIP call, so all statuses except AXO_ERR_HIP can be
// exercised on a machine without a GPU.
#include "../../include/axo.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <map>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "axo_common.hpp"
#include "bias_grad.hpp"
#include "gemm_generic.hpp"
#include "gemm_group.hpp"
#include "gemm_slim.hpp"
#include "gemm_tile.hpp"
#include "tile_bands.hpp"

// Scratch memory of the allocation-free entry point (axo_bias_grad_static): arrival counters and
// slice sums of the split bias gradient, laid out as BiasSplit says.  One copy per GPU, held from
// the moment the library is loaded on it until the process ends; zero-initialised by the loader,
// and every call leaves the counters at zero.  In host code this name only stands for the symbol:
// the device address comes from hipGetSymbolAddress (static_scratch() below), per device.
constexpr size_t STATIC_SCRATCH_BYTES = 256 * 1024;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

namespace {

using axo::GemmArgs;

struct Shard {
    int64_t M, Kl, Nl, row0, k0, n0;
    int k_coord;  // coordinate along the axis that splits K
};

int derive_shard(const axo_problem_t* p, Shard* s) {
    if (!p) return AXO_ERR_NULL_PTR;
    if (p->reserved != 0 || (p->transposed != 0 && p->transposed != 1)) return AXO_ERR_BAD_ARG;
    if (p->Gx < 1 || p->Gy < 1 || p->Gz < 1) return AXO_ERR_BAD_GRID;
    if (p->ix < 0 || p->ix >= p->Gx || p->iy < 0 || p->iy >= p->Gy || p->iz < 0 || p->iz >= p->Gz)
        return AXO_ERR_BAD_COORD;
    if (p->T < 0 || p->K < 0 || p->N < 0) return AXO_ERR_BAD_SIZE;
    // Section 3.2: I is cut over the token axis (Z) and the reduction axis, W over the reduction
    // axis and the output axis.  transposed swaps which of X / Y plays which role.
    const int gk = p->transposed ? p->Gy : p->Gx, ik = p->transposed ? p->iy : p->ix;
    const int gn = p->transposed ? p->Gx : p->Gy, in = p->transposed ? p->ix : p->iy;
    if (p->T % p->Gz != 0 || p->K % gk != 0 || p->N % gn != 0) return AXO_ERR_INDIVISIBLE;
    s->M = p->T / p->Gz;
    s->Kl = p->K / gk;
    s->Nl = p->N / gn;
    if (s->M > INT32_MAX || s->Kl > INT32_MAX || s->Nl > INT32_MAX) return AXO_ERR_BAD_SIZE;
    s->row0 = s->M * p->iz;
    s->k0 = s->Kl * ik;
    s->n0 = s->Nl * in;
    s->k_coord = ik;
    return AXO_OK;
}

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

// One matrix argument: pointer, leading dimension, row length.  A matrix without elements is
// never dereferenced, so nothing about it is checked.
int check_matrix(const void* ptr, int64_t ld, int64_t rows, int64_t row_len) {
    if (rows == 0 || row_len == 0) return AXO_OK;
    if (!ptr) return AXO_ERR_NULL_PTR;
    if (ld < row_len) return AXO_ERR_BAD_LD;
    if (!aligned16(ptr) || (ld % 8) != 0) return AXO_ERR_MISALIGNED;
    return AXO_OK;
}

// A launch's threads per grid dimension have to stay below 2^32.  Thin outputs of hundreds of millions of rows or
// columns pass that with the smaller tiles; the choices below then fall through to a kernel that takes them.
bool grid_fits(int64_t blocks, int threads) { return blocks <= (int64_t)UINT32_MAX / threads; }
int64_t tiles_in(int n, int size) { return ((int64_t)n + size - 1) / size; }

int launch_generic(const GemmArgs& g, int la, int lb, hipStream_t st) {
    dim3 grid((g.No + axo::GEN_BN - 1) / axo::GEN_BN, (g.Mo + axo::GEN_BM - 1) / axo::GEN_BM, 1);
    dim3 block(256, 1, 1);
    if (grid.y > 65535u) return AXO_ERR_BAD_SIZE;
    if (la == axo::KC && lb == axo::MC)
        hipLaunchKernelGGL((axo::gemm_generic_kernel<axo::KC, axo::MC>), grid, block, 0, st, g);
    else if (la == axo::KC && lb == axo::KC)
        hipLaunchKernelGGL((axo::gemm_generic_kernel<axo::KC, axo::KC>), grid, block, 0, st, g);
    else
        hipLaunchKernelGGL((axo::gemm_generic_kernel<axo::MC, axo::MC>), grid, block, 0, st, g);
    return hipGetLastError() == hipSuccess ? AXO_OK : AXO_ERR_HIP;
}

// The tuned kernel covers the output with 256x256 tiles and, to balance tile counts that do not
// fill the last round of CUs, a region of 256x128 tiles.  The CU count is a design constant
// (MI355X: 256 CUs) so that planning needs no device.
constexpr int NUM_CU = 256;
// relative cost of a half-width tile (half the flops at lower efficiency: more operand traffic
// per flop), in units of one big tile; measured on MI355X
constexpr double SMALL_TILE_COST = 0.60;

// The tuned kernel addresses an operand tile through a buffer descriptor with 32-bit byte offsets:
// the span a workgroup walks (256 rows of a KC operand, or the whole reduction of an MC operand)
// has to stay below 4 GiB.
bool span_ok(int layout, int64_t ld, int64_t R) {
    const int64_t elems = layout == axo::KC ? 256 * ld + R : R * ld + 256;
    return elems * 2 < (int64_t)0xFFFF0000;
}

// The span is that of the rows the kernels walk: the reduction rounded up to the unrolled loop's 128
// (the surplus rows of wgrad read as zeros, but their offsets are still formed in 32 bits).
bool spans_ok(const GemmArgs& g, int la, int lb) {
    const int64_t walked = ((int64_t)g.R + 2 * axo::TILE_BK - 1) / (2 * axo::TILE_BK) * (2 * axo::TILE_BK);
    return span_ok(la, g.lda, walked) && span_ok(lb, g.ldb, walked);
}

// Time (in big-tile units) a greedy dispatch of n_big big tiles followed by n_small small tiles
// takes on NUM_CU CUs: workgroups are handed out in order to whichever CU is free first.  The big tiles
// leave n_big % NUM_CU CUs busy one unit longer than the others.  Small tiles then start in batches: those CUs at 1, 1 + c,
// 1 + 2 c, ..., the others at 0, c, 2 c, ... (c the cost of a small tile), and from 1 on any span of c holds one start per
// CU, so that all but the last few batches can be counted off instead of simulated.
double makespan(int64_t n_big, int64_t n_small) {
    const int64_t late = n_big % NUM_CU, on_time = NUM_CU - late;
    double base = (double)(n_big / NUM_CU);
    if (n_small == 0) return base + (late > 0 ? 1.0 : 0.0);
    if (n_small > 3 * NUM_CU) {  // at most 2 NUM_CU of them start before 1
        const int64_t spans = n_small / NUM_CU - 3;
        base += SMALL_TILE_COST * (double)spans;
        n_small -= spans * NUM_CU;
    }
    double t0 = 0.0, t1 = late > 0 ? 1.0 : 1e30, end = late > 0 ? 1.0 : 0.0;  // next starts
    while (n_small > 0) {
        double& t = t0 < t1 ? t0 : t1;
        n_small -= t0 < t1 ? on_time : late;
        t += SMALL_TILE_COST;
        end = std::max(end, t);
    }
    return base + end;
}

// 128-wide tile columns that cover what `big_cols` 256-wide ones leave of No.
int half_cols(int No, int big_cols) { return (int)std::max<int64_t>(0, ((int64_t)No - (int64_t)big_cols * 256 + 127) / 128); }

// Choose how many 256-wide tile columns to use; the remaining columns become 128-wide tiles.  Only the
// last columns come into question: every column cut in two adds 2 SMALL_TILE_COST - 1 = 0.2 tiles of work per tile row (one
// that the output only half fills saves 0.4 once), and a plan with more work than NUM_CU tiles above that of whole columns
// cannot end before them.  Of plans that end together the one with the least work is taken: a last column that fits
// one half-width tile is not given a whole one (dgrad 2176 x 5504, reduction 16384, 385 us with a whole one and 323
// with a half; forward 7552 x 1152 x 9984 213 and 182; over 365 such shapes the half is 3 % quicker on average).  Plans are cached per tile count, so all sizes of a tile share one; a search takes
// 1 us for 4000 x 6000 and 15 us for a single row of millions of tiles.  (Simulated tile by tile for every split and cached per exact
// size, a new batch length cost 0.4 ms at 4000 x 6000 and 88 ms at 16384 x 50257, in every call.)
axo::TileSched plan_tiles(int Mo, int No) {
    static std::mutex mu;
    static std::map<std::pair<int, int>, axo::TileSched> cache;
    axo::TileSched sc{};
    sc.tiles_m = Mo / 256 + (Mo % 256 != 0);
    const int halves = No / 128 + (No % 128 != 0), max_big_cols = (halves + 1) / 2;  // the last one may reach over the edge
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find({sc.tiles_m, halves});
    if (it != cache.end()) return it->second;
    int best_cols = max_big_cols;
    double best = 1e30, best_work = 1e30;
    const int min_cols = (int)std::max<int64_t>(0, max_big_cols - 4 - (int64_t)(NUM_CU / 0.2) / sc.tiles_m);
    for (int cb = max_big_cols; cb >= min_cols; --cb) {
        const int small = std::max(0, halves - 2 * cb);
        const double t = makespan((int64_t)sc.tiles_m * cb, (int64_t)sc.tiles_m * small), work = cb + SMALL_TILE_COST * small;
        if (t < best - 1e-9 || (t < best + 1e-9 && work < best_work - 1e-9)) {
            best = t;
            best_work = work;
            best_cols = cb;
        }
    }
    sc.big_cols = best_cols;
    sc.small_cols = std::max(0, halves - 2 * best_cols);
    sc.n_big = sc.tiles_m * sc.big_cols;
    sc.group_m = sc.tiles_m < 4 ? sc.tiles_m : 4;
    if (cache.size() < 4096) cache[{sc.tiles_m, halves}] = sc;
    return sc;
}

// The tuned kernels' dynamic LDS size is above the default limit, so the limit is raised once per
// kernel and device (`raised` holds one bit per device ordinal; a process rarely sees more than
// 8, and beyond 64 the attribute is simply set on every launch).
bool raise_lds_limit(const void* kernel, int bytes, std::atomic<uint64_t>* raised) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
    if (bit && (raised->load(std::memory_order_acquire) & bit)) return true;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess)
        return false;
    raised->fetch_or(bit, std::memory_order_release);
    return true;
}

int64_t steps_in(int R) { return tiles_in(R, axo::TILE_BK); }
int64_t rounds_of(int64_t tiles) { return (tiles + NUM_CU - 1) / NUM_CU; }

// Estimated kernel time in microseconds of a product on its own, from its sizes alone.
// 256-row tiles: half-width tiles where they have a CU each, else large ones, else rounds of either.  A reduction step of a
// large tile takes 1.0 us on a chip that is nearly idle and 1.27 on a full one, which runs at its power limit.  Fitted to 3400
// measured products; half of the estimates are within 11 %, nine of ten within 25 %.  (With 1.33 us at any load, few tiles with
// long reductions were taken for slower than they are, and 64 x 64 tiles chosen instead: wgrad 1616 x 2960 of 8136
// tokens 181 us, 87 on these; 1536 x 3072 of 6016 98 and 61; dgrad 2408 x 3264 with reduction 9288 357 and 266.)
double tile_time(int Mo, int No, int R) {
    const int64_t tm = tiles_in(Mo, 256), big = tm * tiles_in(No, 256), half = tm * tiles_in(No, 128);
    const double rounds = half <= NUM_CU ? SMALL_TILE_COST : std::min((double)rounds_of(big), SMALL_TILE_COST * rounds_of(half));
    const double busy = std::min<int64_t>(half <= NUM_CU ? half : big, NUM_CU) / (double)NUM_CU;
    return 3.4 + rounds * (steps_in(R) + 4.4) * (1.0 + 0.27 * busy * busy);
}
// 128 x 128 tiles, 0.42 us per step.
double mid_time(int Mo, int No, int R) {
    if (tiles_in(Mo, 128) * tiles_in(No, 128) > NUM_CU) return 1e30;  // more than one tile per CU: see below
    return 4.5 + steps_in(R) * 0.42;
}

// 64 x 64 tiles of a ring: a step takes 0.235 us with a CU to itself, and 0.15 us on a busy one, where two run beside
// each other (wgrad 1024 x 1024 of 8192 tokens: 29 us measured, 33 estimated).  These times are from before the ring's loop was peeled:
// forward 2048 x 1024 x 1024 takes 8.7 us now where 9.5 are estimated, 64 steps of one round 14.6 where 18.2 are, so tiles that split
// the reduction are still taken for some products that these would be quicker for.
double small_time(int Mo, int No, int R) {
    const int64_t n = rounds_of(tiles_in(Mo, 64) * tiles_in(No, 64));
    return n <= 1 ? 3.2 + steps_in(R) * 0.235 : 3.0 + n * (0.85 + steps_in(R) * 0.15);
}
// What several rounds of them lose beyond 32 steps, where the operands leave the L2 (1408 x 11008 x 7296 dgrad: 427 us measured,
// 272 without this part).  Counts against the larger tiles only, not where split reductions are weighed against these
// tiles: there the two kinds slow down alike.
double small_time_long(int Mo, int No, int R) {
    const int64_t n = rounds_of(tiles_in(Mo, 64) * tiles_in(No, 64)), late = steps_in(R) - 32;
    return n <= 1 || late <= 0 ? 0.0 : n * late * 0.05;
}

// Launch of one product on tiles of ROWS x COLS.  Weight gradients take the bands of band_height, the others 8 tile rows.
template <typename C, int ROWS, int COLS, int LA>
int launch_tiles(void (*kern)(GemmArgs, int, int, int), std::atomic<uint64_t>* raised, const GemmArgs& g, hipStream_t st) {
    if (!raise_lds_limit(reinterpret_cast<const void*>(kern), C::LDS_BYTES, raised)) return AXO_ERR_HIP;
    const int tm = (int)tiles_in(g.Mo, ROWS), tn = (int)tiles_in(g.No, COLS);
    hipLaunchKernelGGL(kern, dim3((unsigned)tm * (unsigned)tn), dim3(C::THREADS), C::LDS_BYTES, st, g, tm, tn,
                       LA == axo::MC ? axo::band_height(tm, tn, ROWS, COLS, axo::NUM_XCD) : std::min(tm, 8));
    return hipGetLastError() == hipSuccess ? AXO_OK : AXO_ERR_HIP;
}

// The tiles of a product on its own, whichever are estimated quickest (all give
// the same bits).  128 x 128 tiles only where every tile has a CU of its own: beyond that they are bound by the rate at which a CU takes in
// operands (384 tiles: 4096 x 1536 x 1536 forward 28.6 us against 23.5; 1504 tiles: 4000 x 2000 x 6000 125 against 97).
// Halves of those, 64 x 128 or 128 x 64 (`wide`, `tall`), where every one has a CU of its own, 64 x 64 tiles would take clearly more than one
// round and the reduction has at least 16 steps: there they are the quickest by 8 to 45 % (gemm_rect_kernel; with 16 tiles too many for one round 64 x 64
// ones are as quick: 1001 x 1027 x 1300 13.2 us, 13.4).  The line at 16 steps was drawn when they were level at 8 (forward 2000 x 1000 x 512 6.2 us either
// way).  By now they are the quicker from 8 on, and the line has not been moved: 64 x 64 / these in us 2048 x 1024 x 512 6.3 / 5.9, x 768 7.5 / 6.9,
// dgrad 7.3 / 7.0, wgrad 7.4 / 6.8, wgrad 2000 x 1000 of 512 tokens 7.8 / 6.75, dgrad 6.15 / 6.0.  Of the two kinds the one with fewer tiles, else the
// wide one, which reads the rows of a forward's W in segments of 256 bytes (1000 x 2000 x 3000 19.7 us, 20.1 on the tall ones, dgrad 17.9 and 18.2,
// wgrad either way 21.0; wgrad 900 x 1300 of 6000 38.3 and 36.5).
enum class Tiles { small, wide, tall, mid, big };
Tiles tiles_of(int Mo, int No, int R) {
    const int64_t wide = tiles_in(Mo, 64) * tiles_in(No, 128), tall = tiles_in(Mo, 128) * tiles_in(No, 64);
    if (std::min(wide, tall) <= NUM_CU && 8 * tiles_in(Mo, 64) * tiles_in(No, 64) > 9 * NUM_CU && steps_in(R) >= 16) return wide <= tall ? Tiles::wide : Tiles::tall;
    const double small_us = small_time(Mo, No, R) + small_time_long(Mo, No, R), mid_us = mid_time(Mo, No, R), big_us = tile_time(Mo, No, R);
    if (small_us < mid_us && small_us < big_us && grid_fits(tiles_in(Mo, 64) * tiles_in(No, 64), axo::SmallCfg<false>::THREADS)) return Tiles::small;
    return mid_us < big_us ? Tiles::mid : Tiles::big;
}

// Units of the start-up phase shift of a launch on 256-row tiles (see start_shift): short reductions over more
// than one round of tiles.  Without / with 3 units: 4864 x 12288, reduction 128, 36.8 / 29.7 us; 8192 x 12416 x 256 77.8 / 66.2;
// 4352 x 8704 x 128 24.0 / 21.1; medians of 1200 sizes at two rounds or more 1.12 times quicker up to 4 steps, 1.06 up to 12, 1.03 up
// to 24, 1.02 up to 32 (4096 x 16384 x 2048 200 / 195.5), none beyond.  Between one round and two 2 units are the better choice (1.02 up to 16 steps).  Launches of at most one round
// lose by it (0.7 up to 6 steps, 0.86 at 24).
int shift_units(int Mo, int No, int R) {
    const int64_t tiles = tiles_in(Mo, 256) * tiles_in(No, 256), steps = tiles_in(R, axo::TILE_BK);
    if (tiles > 2 * NUM_CU) return steps <= 32 ? 3 : 0;
    return tiles > NUM_CU && steps <= 16 ? 2 : 0;
}

// The plan of a product on 256-row tiles: plan_tiles' split of the columns, the start-up shift, and for short reductions
// into rows that do not end on cache lines another order.  There the launch is bound by its output, whose lines at a
// tile's sides are written in two parts: tiles beside each other follow each other on one XCD (bands of one tile row),
// so that the parts meet in its L2, instead of four tile rows at a time for the sake of the operands.  Medians of 400 sizes
// with more tiles than CUs: 1.05 times quicker up to 4 steps, no matter at 8, slower beyond.  Data gradients of such reductions
// also take half-width tiles throughout, whose ring walks exactly the steps there are and masks the end of both operands
// in registers: 1.27 / 1.16 / 1.16 times quicker at 1 / 2 / 3-4 steps (10600 x 7736, reduction 48, 101 us, in this order 85, with half-width
// tiles 74).
axo::TileSched plan_product(const GemmArgs& g, int la, int lb) {
    axo::TileSched sc = plan_tiles(g.Mo, g.No);
    sc.shift = shift_units(g.Mo, g.No, g.R);
    const int64_t pitch = g.ldc * (g.epilogue == axo::EPI_ACC_F32 ? 4 : 2);
    if (pitch % 128 != 0 && g.R <= 4 * axo::TILE_BK && tiles_in(g.Mo, 256) * tiles_in(g.No, 256) > NUM_CU) {
        sc.group_m = 1;
        if (la == axo::KC && lb == axo::KC) {
            sc.big_cols = sc.n_big = sc.shift = 0;
            sc.small_cols = half_cols(g.No, 0);
        }
    }
    return sc;
}

// Rows, of eight that follow each other, that start elsewhere than on a cache line: 7 where the pitch is an odd number of 16-byte
// chunks, 6 or 4 where it is an odd number of 2 or of 4, none or (by the first one's address) all where it is whole lines.
int straddling(const axo::bf16_t* p, int64_t ld) {
    int n = 0;
    for (int64_t r = 0; r < 8; ++r) n += ((int64_t)(reinterpret_cast<uintptr_t>(p) >> 4) + r * (ld >> 3)) % 8 != 0;
    return n;
}

// Whether a product fetches operands whose reduction runs inside the rows by whole cache lines (line_phase) on tiles of this kind:
// where enough rows straddle lines and the reduction is long enough to pay for the later start and the one stage more.
//   64 x 64, 128 x 128 and its halves  a stage was added for it, or there were four: wherever either operand has such rows.  Without / with it, rows 16
//              bytes off, in us: dgrad 1024 x 1024 with 8 / 16 / 32 steps 4.70 / 5.11, 7.82 / 6.83, 12.0 / 9.3; 2048 x 1024 (two
//              tiles per CU) with 8 6.66 / 6.35; 2048 x 2048 with 8 / 16 / 32 9.62 / 9.33, 14.6 / 13.3, 23.3 / 18.0; one operand
//              off and half its rows straddling 1024 x 1024 x 2048 8.98 / 8.73, 2048 x 2048 x 2048 19.1 / 18.2
//   256 x 128  dgrad only.  Its three stages are then requested one step ahead instead of two, whatever the rows: 4096 x 1536 x 6144 takes
//              77 us in any place.  Without it 64 on lines, 76 or 67 with 16 bytes off dY or W, 85 with both, 81 with 32 bytes
//              off both, 81 with 16 and 64 and 72 with 64 (2304 x 2176 x 2240 32 with it and 25, 31, 26, 34, 33, 33, 29): by the
//              share of a step's 384 rows that straddle, the line lies at two thirds, 18 of 24 is on the right side of it.  With
//              operands from HBM, behind the forward, 4000 x 2000 x 6000 (18 of 24) takes 97 us without and 88 with it: the
//              same bytes fetched, the texture path busy 0.95 of the time without and 0.55 with it.
//   256 x 256  of the first operand only, so only where that one's rows straddle: dgrad 4096 x 4096 x 8192 260 / 226 us, 8192 x 8192
//              x 2000 272 / 233, 5120 x 5120 x 1024 58.6 / 53.4, forward 4096 x 4096 x 8192 225 / 205; with 64 bytes off, half the
//              rows, 4096 x 4096 with 12 / 16 / 24 / 32 steps 26.5 / 27.0, 32.1 / 32.6, 43.6 / 43.6, 53.5 / 53.4.
enum class Tile { t64, t128, half, whole };
bool takes_lines(const GemmArgs& g, int la, int lb, Tile tile) {
    if (la != axo::KC) return false;
    const int a = straddling(g.A, g.lda), b = lb == axo::KC ? straddling(g.B, g.ldb) : 0;
    const int64_t steps = steps_in(g.R);
    if (steps < 8) return false;
    // the ring then walks one stage more of the other operand, too, which spans_ok does not count where there are an even number of steps
    const bool in_span = lb == axo::KC || span_ok(axo::MC, g.ldb, (steps + 1) * axo::TILE_BK);
    switch (tile) {
        case Tile::t64: return in_span && a + b > 0 && (steps >= 12 || 2 * tiles_in(g.Mo, 64) * tiles_in(g.No, 64) > 3 * NUM_CU);
        case Tile::t128: return in_span && a + b > 0;
        case Tile::half: return lb == axo::KC && 2 * a + b >= 18;
        default: return a > 4 || (a > 0 && steps >= 24);
    }
}
// The same for a launch on 256-row tiles: on none of them, on whole ones, on all.
enum Lines { LINES_NONE = 0, LINES_WHOLE = 1, LINES_ALL = 2 };
Lines lines_of(const GemmArgs& g, int la, int lb, const axo::TileSched& sc) {
    if (sc.small_cols > 0 && takes_lines(g, la, lb, Tile::half)) return LINES_ALL;  // more than half of A's rows straddle, too
    return sc.n_big > 0 && takes_lines(g, la, lb, Tile::whole) ? LINES_WHOLE : LINES_NONE;
}

// Launch of one product on those tiles.
template <int LA, int LB, int LINES>
int launch_mixed(const GemmArgs& g, const axo::TileSched& sc, hipStream_t st) {
    // rows whose pitch makes them straddle cache lines, behind a short reduction: stored plainly (store_row)
    const bool plain = g.epilogue != axo::EPI_ACC_F32 && g.ldc % 64 != 0 && steps_in(g.R) <= 16;
    auto kern = plain ? axo::gemm_mixed_kernel<LA, LB, LINES, true> : axo::gemm_mixed_kernel<LA, LB, LINES, false>;
    constexpr int lds = LINES != LINES_NONE ? axo::LINES_LDS_BYTES : axo::MIX_LDS_BYTES;
    static std::atomic<uint64_t> raised[2]{{0}, {0}};
    if (!raise_lds_limit(reinterpret_cast<const void*>(kern), lds, &raised[plain])) return AXO_ERR_HIP;
    const int blocks = sc.n_big + sc.tiles_m * sc.small_cols;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(axo::TILE_THREADS), lds, st, g, sc);
    return hipGetLastError() == hipSuccess ? AXO_OK : AXO_ERR_HIP;
}
template <int LA, int LB, bool LINES>
int launch_ring_tiles(const GemmArgs& g, Tiles tiles, hipStream_t st) {
    static std::atomic<uint64_t> raised[4]{{0}, {0}, {0}, {0}};
    if (tiles == Tiles::small) return launch_tiles<axo::SmallCfg<LINES>, 64, 64, LA>(axo::gemm_small_kernel<LA, LB, LINES>, &raised[0], g, st);
    if (tiles == Tiles::wide) return launch_tiles<axo::RectCfg<true>, 64, 128, LA>(axo::gemm_rect_kernel<LA, LB, true, LINES>, &raised[1], g, st);
    if (tiles == Tiles::tall) return launch_tiles<axo::RectCfg<false>, 128, 64, LA>(axo::gemm_rect_kernel<LA, LB, false, LINES>, &raised[2], g, st);
    return launch_tiles<axo::MidCfg, 128, 128, LA>(axo::gemm_mid_kernel<LA, LB, LINES>, &raised[3], g, st);
}
template <int LA, int LB>
int launch_tile(const GemmArgs& g, hipStream_t st) {
    const Tiles tiles = tiles_of(g.Mo, g.No, g.R);
    if (tiles != Tiles::big) {
        if constexpr (LA == axo::KC)
            if (takes_lines(g, LA, LB, tiles == Tiles::small ? Tile::t64 : Tile::t128)) return launch_ring_tiles<LA, LB, true>(g, tiles, st);
        return launch_ring_tiles<LA, LB, false>(g, tiles, st);
    }
    const axo::TileSched sc = plan_product(g, LA, LB);
    const Lines lines = lines_of(g, LA, LB, sc);
    if constexpr (LA == axo::KC && LB == axo::KC) if (lines == LINES_ALL) return launch_mixed<LA, LB, LINES_ALL>(g, sc, st);
    if constexpr (LA == axo::KC) if (lines == LINES_WHOLE) return launch_mixed<LA, LB, LINES_WHOLE>(g, sc, st);
    return launch_mixed<LA, LB, LINES_NONE>(g, sc, st);
}

int launch_tile_layout(const GemmArgs& g, int la, int lb, hipStream_t st) {
    if (la == axo::KC && lb == axo::MC) return launch_tile<axo::KC, axo::MC>(g, st);
    if (la == axo::KC && lb == axo::KC) return launch_tile<axo::KC, axo::KC>(g, st);
    return launch_tile<axo::MC, axo::MC>(g, st);
}

// ---- small-tile launch (gemm_slim.hpp) ---------------------------------------------------------
// Estimated kernel time in microseconds of a product on small tiles, from its sizes alone.  Fitted to 177
// measured products (M 1..8000, K and N 94..13312, all three layout pairs); 85-89 % of the estimates are within 20 %.
// A small tile costs a fixed part (start, first load,
// addition of the partial tiles, store) plus its operand bytes at the rate a CU pulls them in; a
// product with few tiles is bound by one workgroup's chain of chunks instead.
struct SlimModel {
    int rows;          // square tile
    int slots;         // workgroups that fit one CU beside each other
    double fixed;      // us per tile on a busy CU
    double chunk_us;   // us per chunk of one wave when nothing else runs on the CU
    double rate[3];    // KB per us of a busy CU, by layout pair
};
constexpr SlimModel SLIM_MODEL[2] = {{32, 5, 0.2, 0.24, {80.0, 106.0, 60.0}}, {64, 2, 1.5, 0.47, {112.0, 115.0, 95.0}}};
int64_t slim_tiles(const SlimModel& m, int Mo, int No) { return m.rows == 32 ? tiles_in(Mo, 32) * tiles_in(No, 32) : tiles_in(Mo, 64) * tiles_in(No, 64); }
double slim_tile_us(const SlimModel& m, int R, int pair) {  // one tile on a busy CU
    return steps_in(R) * (2.0 * m.rows * axo::TILE_BK * 2 / 1024.0) / m.rate[pair] + m.fixed;
}
double slim_chain_us(const SlimModel& m, int R) {  // one tile on a CU of its own
    return 0.7 + tiles_in(R, axo::SLIM_WAVES * axo::TILE_BK) * m.chunk_us;
}
double slim_time(const SlimModel& m, int Mo, int No, int R, int pair) {
    const int64_t rounds = rounds_of(slim_tiles(m, Mo, No));
    return 2.5 + std::max(rounds * slim_tile_us(m, R, pair), (rounds + m.slots - 1) / m.slots * slim_chain_us(m, R));
}
int layout_pair(int la, int lb) { return (la == axo::KC && lb == axo::MC) ? 0 : (la == axo::KC ? 1 : 2); }

// Whether all tiles of one size go into one launch: square split-reduction tiles, 256-row tiles (none wider than half).
bool slim_fits(const GemmArgs& g, int rows) { return grid_fits(tiles_in(g.Mo, rows) * tiles_in(g.No, rows), axo::SLIM_WAVES * 64); }
int64_t most_tile_blocks(const GemmArgs& g) { return tiles_in(g.Mo, 256) * tiles_in(g.No, 128); }

// Rows of the small tile (32 or 64) that is quicker for this product.
int slim_rows(const GemmArgs& g, int pair) {
    if (!slim_fits(g, 32)) return 64;
    return slim_time(SLIM_MODEL[0], g.Mo, g.No, g.R, pair) <= slim_time(SLIM_MODEL[1], g.Mo, g.No, g.R, pair) ? 32 : 64;
}
// Share of the chip's time that a product's 256-row tiles take in a launch that fills it.
double tile_share(int Mo, int No, int R) {
    return tiles_in(Mo, 256) * std::min(tiles_in(No, 256) * 1.0, tiles_in(No, 128) * SMALL_TILE_COST) * (steps_in(R) + 4.0) * 1.33 / NUM_CU;
}
// Whether a product runs on tiles whose waves split the reduction: where those are estimated at least 15 % quicker than
// the others, and where a chain's grouped launch, in which the larger tiles of other products keep the chip
// full, loses no more than about a microsecond by it.  A function of sizes and layouts only, because these tiles sum
// in another order: a product has the same bits on its own and in a chain.  (Without the second condition a block of
// four layers, 2048 tokens of width 1024, took 181 us instead of 127.)
bool prefers_slim(const GemmArgs& g, int la, int lb) {
    const int pair = layout_pair(la, lb);
    double us = 1e30, share = 1e30;
    for (const SlimModel& m : SLIM_MODEL) {
        us = std::min(us, slim_time(m, g.Mo, g.No, g.R, pair));
        share = std::min(share, slim_tiles(m, g.Mo, g.No) * slim_tile_us(m, g.R, pair) / NUM_CU);
    }
    return us < 0.85 * std::min({tile_time(g.Mo, g.No, g.R), mid_time(g.Mo, g.No, g.R), small_time(g.Mo, g.No, g.R)}) &&
           share < 1.3 * tile_share(g.Mo, g.No, g.R) + 1.0;
}

template <int ROWS, int ST, int LA, int LB>
int launch_slim_rows(const GemmArgs& g, hipStream_t st) {
    using C = axo::SlimCfg<ROWS, ROWS, axo::SLIM_WAVES, ST>;
    auto kern = axo::gemm_slim_kernel<ROWS, ROWS, axo::SLIM_WAVES, ST, LA, LB>;
    static std::atomic<uint64_t> raised{0};
    if (!raise_lds_limit(reinterpret_cast<const void*>(kern), C::LDS_BYTES, &raised)) return AXO_ERR_HIP;
    axo::SlimSched sc{(g.Mo + ROWS - 1) / ROWS, (g.No + ROWS - 1) / ROWS, 0};
    sc.group_m = std::min(sc.tiles_m, 8);  // 8 tile rows share the column panels in an XCD's L2
    hipLaunchKernelGGL(kern, dim3((unsigned)sc.tiles_m * (unsigned)sc.tiles_n), dim3(C::THREADS), C::LDS_BYTES, st, g, sc);
    return hipGetLastError() == hipSuccess ? AXO_OK : AXO_ERR_HIP;
}
// Whether a product on 32 x 32 tiles keeps two LDS stages per wave.  Two stages leave room for two workgroups on a
// CU, one stage for five; below 16 chunks per wave the second stage's longer start costs what it gains (200 x 2000 x 512
// forward 5.5 us with one, 5.8 with two).
bool slim_two_stages(const GemmArgs& g) {
    const int64_t tiles = ((int64_t)g.Mo + 31) / 32 * (((int64_t)g.No + 31) / 32);
    return tiles <= 2 * NUM_CU && g.R >= 16 * axo::SLIM_WAVES * axo::TILE_BK;
}
template <int LA, int LB>
int launch_slim_layout(const GemmArgs& g, int rows, hipStream_t st) {
    if (rows == 64) return launch_slim_rows<64, 1, LA, LB>(g, st);
    return slim_two_stages(g) ? launch_slim_rows<32, 2, LA, LB>(g, st) : launch_slim_rows<32, 1, LA, LB>(g, st);
}
int launch_slim(const GemmArgs& g, int la, int lb, hipStream_t st) {
    const int rows = slim_rows(g, layout_pair(la, lb));
    if (la == axo::KC && lb == axo::MC) return launch_slim_layout<axo::KC, axo::MC>(g, rows, st);
    if (la == axo::KC && lb == axo::KC) return launch_slim_layout<axo::KC, axo::KC>(g, rows, st);
    return launch_slim_layout<axo::MC, axo::MC>(g, rows, st);
}

// ---- grouped launch ------------------------------------------------------------------------
// Cost of one tile in reduction steps of a big tile: the steps themselves plus a fixed share for
// the tile's first loads and its epilogue (measured: a two-step tile takes about as long as six
// steps of a long one).
constexpr double TILE_OVERHEAD_STEPS = 4.0;
double tile_cost(int R, bool small) {
    return (R / (double)axo::TILE_BK + TILE_OVERHEAD_STEPS) * (small ? SMALL_TILE_COST : 1.0);
}

struct GroupItem {
    int Mo, No, R, pair;
    bool operator<(const GroupItem& o) const {
        if (Mo != o.Mo) return Mo < o.Mo;
        if (No != o.No) return No < o.No;
        if (R != o.R) return R < o.R;
        return pair < o.pair;
    }
};

struct SegCost {
    double cost;
    int count, item, small;  // small: 1 half-width tiles, 2 pairs of 64 x 64 tiles
};

// A bias gradient inside a grouped launch (GroupItem::pair == PAIR_BIAS_GRAD, Mo = rows, No =
// columns): strips of 64 columns, each a workgroup that streams Mo rows of 128 bytes.  A strip
// is bound by memory latency, not bandwidth: measured 19 us for 4096 rows, which is what 15
// reduction steps of a big tile take.
constexpr int PAIR_BIAS_GRAD = 3;
// A product on small tiles inside a grouped launch (GroupItem::pair == PAIR_SLIM + its layout pair): a workgroup
// takes two 64 x 64 tiles; their cost in reduction steps of a big tile (1.33 us).
constexpr int PAIR_SLIM = 4;
double slim_pair_cost(int R, int pair) { return 2.0 * slim_tile_us(SLIM_MODEL[1], R, pair) / 1.33; }
int slim_pair_blocks(int Mo, int No) { return (int)((tiles_in(Mo, 64) * tiles_in(No, 64) + 1) / 2); }
// The same for a product that could take 256-row tiles: a pair of 64 x 64 ring tiles takes 2.2 us and 0.33 per step.  The planner
// weighs them as one more split (PAIRS in place of a number of columns); all these tiles give the same bits.
constexpr int PAIRS = -1, MOST_PAIRS = 8 * NUM_CU;
double pair_cost(int R) { return (2.2 + 0.33 * steps_in(R)) / 1.33; }
double bias_strip_cost(int rows) { return 1.0 + 15.0 * rows / 4096.0; }
int bias_strips(int cols) { return (cols + axo::GROUP_BIAS_COLS - 1) / axo::GROUP_BIAS_COLS; }
// The standalone launch picks its strip width by shape; only shapes for which it picks the
// grouped launch's 64 columns may ride along, so that both give the same bits.
bool bias_grad_groupable(const axo::BiasGradArgs& g) { return g.Nl > 0 && bias_strips(g.Nl) >= NUM_CU / 4; }

// segments of a group for a choice of big_cols per item, most expensive tiles first
std::vector<SegCost> group_segments(const std::vector<GroupItem>& items, const std::vector<int>& big_cols) {
    std::vector<SegCost> segs;
    for (size_t i = 0; i < items.size(); ++i) {
        if (items[i].pair == PAIR_BIAS_GRAD) {
            segs.push_back({bias_strip_cost(items[i].Mo), bias_strips(items[i].No), (int)i, 0});
            continue;
        }
        if (items[i].pair >= PAIR_SLIM) {
            segs.push_back({slim_pair_cost(items[i].R, items[i].pair - PAIR_SLIM), slim_pair_blocks(items[i].Mo, items[i].No), (int)i, 0});
            continue;
        }
        if (big_cols[i] == PAIRS) {
            segs.push_back({pair_cost(items[i].R), slim_pair_blocks(items[i].Mo, items[i].No), (int)i, 2});
            continue;
        }
        const int tiles_m = (items[i].Mo + 255) / 256, cb = big_cols[i], cs = half_cols(items[i].No, cb);
        if (cb > 0) segs.push_back({tile_cost(items[i].R, false), tiles_m * cb, (int)i, 0});
        if (cs > 0) segs.push_back({tile_cost(items[i].R, true), tiles_m * cs, (int)i, 1});
    }
    std::stable_sort(segs.begin(), segs.end(), [](const SegCost& a, const SegCost& b) { return a.cost > b.cost; });
    return segs;
}

// Time a greedy dispatch of the segments in their order takes on NUM_CU CUs.  CUs that fall free together take their
// tiles together, and a segment adds at most one more time to the few at which CUs fall free.
double group_makespan(const std::vector<SegCost>& segs) {
    struct Free {
        double t;
        int cus;
    };
    std::vector<Free> free_at{{0.0, NUM_CU}};  // latest first
    free_at.reserve(segs.size() + 2);
    for (const SegCost& sg : segs)
        for (int left = sg.count; left > 0;) {
            Free& first = free_at.back();
            const int n = std::min(first.cus, left);
            const double t = first.t + sg.cost;
            left -= n;
            first.cus -= n;
            if (first.cus == 0) free_at.pop_back();
            auto at = free_at.begin();
            while (at != free_at.end() && at->t > t) ++at;
            if (at != free_at.end() && at->t == t) at->cus += n;
            else free_at.insert(at, {t, n});
        }
    return free_at.front().t;
}

// big_cols per item that minimise the simulated makespan of the whole group: coordinate descent
// from "all big tiles, and a half-width one where that covers the last column", two sweeps.  That start is the plan with
// the least work, and another one has to be quicker (started from whole tiles over the edge, a layer step of
// 7168 x 1152 x 4096 took 172 us, now 159; 9160 / 8 tokens of 128 x 104 with extras 50 and 26; over 500 chains 1.5 % less).  A split
// with more work than NUM_CU CUs can do before the best plan so far ends is not simulated, nor is a product looked at again
// when no other has changed since.  Cached per list of shapes, so every new token count is a search: a block of
// width 2056 with 200-1000 tokens 2114 us a step when all were simulated, tile by tile, 212 so and 210 with plans at hand.  With
// pairs of small tiles among the choices a search takes 6 us of host time for a layer, 50 for a block of four.
std::vector<int> plan_group(const std::vector<GroupItem>& items) {
    static std::mutex mu;
    static std::map<std::vector<GroupItem>, std::vector<int>> cache;
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find(items);
    if (it != cache.end()) return it->second;
    std::vector<int> cols(items.size());
    for (size_t i = 0; i < items.size(); ++i) cols[i] = items[i].pair >= PAIR_BIAS_GRAD ? 0 : (int)(tiles_in(items[i].No, 128) / 2);
    const std::vector<SegCost> start = group_segments(items, cols);
    double best = group_makespan(start), work = 0.0;  // work: of all tiles, in the units of the makespan on one CU
    for (const SegCost& sg : start) work += sg.cost * sg.count;
    const int n = (int)items.size();
    int changed = 0;  // when a split was last changed
    for (int k = 0; k < 2 * n && k - changed < n; ++k) {
        const GroupItem& it = items[k % n];
        int& c = cols[k % n];
        if (it.pair >= PAIR_BIAS_GRAD) continue;
        const double tiles_m = (double)tiles_in(it.Mo, 256), big = tile_cost(it.R, false), half = tile_cost(it.R, true);
        const int64_t pairs = (tiles_in(it.Mo, 64) * tiles_in(it.No, 64) + 1) / 2;
        auto work_of = [&](int big_cols) {
            return big_cols == PAIRS ? pairs * pair_cost(it.R) : tiles_m * (big_cols * big + half_cols(it.No, big_cols) * half);
        };
        const int max_cols = (int)tiles_in(it.No, 256), now = c;
        const int stride = max_cols > 16 ? (max_cols + 15) / 16 : 1;
        const double others = work - work_of(now);
        int best_c = now;
        auto consider = [&](int to, double margin) {
            if (to == now || (others + work_of(to)) / NUM_CU > best * (1.0 + 1e-9)) return;
            c = to;
            const double t = group_makespan(group_segments(items, cols));
            if (t < best * margin - 1e-9) {
                best = t;
                best_c = to;
            }
        };
        for (int to = max_cols; to >= 0; to -= stride) consider(to, 1.0);
        if (pairs <= MOST_PAIRS) consider(PAIRS, 0.92);  // only for a clear gain: among large tiles they cost more than estimated
        c = best_c;
        if (best_c != now) {
            work = others + work_of(best_c);
            changed = k;
        }
    }
    if (cache.size() < 1024) cache[items] = cols;
    return cols;
}

int check_workspace(const axo_problem_t* p, int op, const void* ws, size_t ws_bytes) {
    const size_t need = axo_workspace_bytes(p, op);
    if (need == 0) return AXO_OK;
    if (!ws || ws_bytes < need) return AXO_ERR_WORKSPACE;
    if (!aligned16(ws)) return AXO_ERR_MISALIGNED;
    return AXO_OK;
}

// Validated, launch-ready description of one unit of work of a chain: a product (the usual
// case) or a bias gradient.
struct Plan {
    GemmArgs g{};
    int la = 0, lb = 0;
    bool small = false;       // the product runs on small tiles (filled in when it is enqueued with others)
    bool bias_grad = false;   // bg is valid instead of g
    axo::BiasGradArgs bg{};
    bool nothing_to_do() const { return bias_grad ? bg.Nl == 0 : (g.Mo == 0 || g.No == 0); }
};

// The segments of one launch over the tiles of all given units of work: products on 256-row tiles (Kernel::tiles), products on
// small tiles that ride along (Plan::small), bias gradients; at most GROUP_MAX_PRODUCTS of them, together no more
// workgroups than a grid holds.  Returns the number of workgroups.
int group_launch(const Plan* const* plans, int n, axo::GroupArgs& ga, bool& lines) {
    std::vector<GroupItem> items(n);
    for (int i = 0; i < n; ++i)
        items[i] = plans[i]->bias_grad ? GroupItem{plans[i]->bg.M, plans[i]->bg.Nl, 0, PAIR_BIAS_GRAD}
                                       : GroupItem{plans[i]->g.Mo, plans[i]->g.No, plans[i]->g.R,
                                                   layout_pair(plans[i]->la, plans[i]->lb) + (plans[i]->small ? PAIR_SLIM : 0)};
    const std::vector<int> cols = plan_group(items);
    const std::vector<SegCost> segs = group_segments(items, cols);
    ga.n_seg = (int)segs.size();
    int blocks = 0;
    lines = false;
    for (int k = 0; k < ga.n_seg; ++k) {
        const SegCost& sc = segs[k];
        axo::GroupSeg& sg = ga.seg[k];
        sg.first_block = blocks;
        sg.n_blocks = sc.count;
        sg.product = sc.item;
        if (items[sc.item].pair == PAIR_BIAS_GRAD) {
            sg.kind = axo::GROUP_KIND_BIAS_GRAD;
            sg.tiles_m = 1;
            sg.cols = sc.count;
            sg.col0 = 0;
            sg.group_m = 1;
        } else if (items[sc.item].pair >= PAIR_SLIM) {
            sg.kind = axo::GROUP_KIND_SLIM + items[sc.item].pair - PAIR_SLIM;
            sg.tiles_m = (items[sc.item].Mo + 63) / 64;
            sg.cols = (items[sc.item].No + 63) / 64;
            sg.col0 = 0;
            sg.group_m = std::min(sg.tiles_m, 8);
        } else if (sc.small == 2) {
            sg.kind = axo::GROUP_KIND_PAIR + items[sc.item].pair;
            sg.tiles_m = (items[sc.item].Mo + 63) / 64;
            sg.cols = (items[sc.item].No + 63) / 64;
            sg.col0 = 0;
            sg.group_m = std::min(sg.tiles_m, 8);
        } else {
            sg.kind = 2 * items[sc.item].pair + sc.small;
            const Plan& pl = *plans[sc.item];
            if (takes_lines(pl.g, pl.la, pl.lb, sc.small ? Tile::half : Tile::whole)) {
                sg.kind += axo::GROUP_KIND_LINES;
                lines = true;
            }
            sg.tiles_m = (items[sc.item].Mo + 255) / 256;
            sg.cols = sc.count / sg.tiles_m;
            sg.col0 = sc.small ? cols[sc.item] * 256 : 0;
            sg.group_m = sg.tiles_m < 4 ? sg.tiles_m : 4;
        }
        blocks += sc.count;
    }
    for (int i = 0; i < n; ++i) {
        if (!plans[i]->bias_grad) {
            ga.g[i] = plans[i]->g;
            continue;
        }
        GemmArgs b{};  // the bias gradient's arguments in a GemmArgs, as gemm_group_kernel reads them
        b.A = plans[i]->bg.dY;
        b.lda = plans[i]->bg.lddy;
        b.C = reinterpret_cast<axo::bf16_t*>(plans[i]->bg.db);
        b.Mo = plans[i]->bg.M;
        b.No = plans[i]->bg.Nl;
        b.epilogue = plans[i]->bg.accumulate;
        ga.g[i] = b;
    }
    return blocks;
}
int launch_group(const Plan* const* plans, int n, hipStream_t st) {
    axo::GroupArgs ga{};
    bool lines;
    const int blocks = group_launch(plans, n, ga, lines);
    static std::atomic<uint64_t> raised[2]{{0}, {0}};
    auto kern = lines ? axo::gemm_group_kernel<true> : axo::gemm_group_kernel<false>;
    const int lds = lines ? axo::LINES_LDS_BYTES : axo::MIX_LDS_BYTES;
    if (!raise_lds_limit(reinterpret_cast<const void*>(kern), lds, &raised[lines])) return AXO_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(axo::TILE_THREADS), lds, st, ga);
    return hipGetLastError() == hipSuccess ? AXO_OK : AXO_ERR_HIP;
}

// Which kernel a product takes; a function of its sizes, layouts and leading dimensions.
enum class Kernel { none, tiles, small_tiles, general };
Kernel kernel_of(const GemmArgs& g, int la, int lb) {
    if (g.Mo == 0 || g.No == 0) return Kernel::none;
    // 64-bit addressing, an order of magnitude slower; and what an empty reduction leaves: epilogue(0)
    if (!spans_ok(g, la, lb) || g.R == 0) return Kernel::general;
    if (prefers_slim(g, la, lb) && slim_fits(g, 64)) return Kernel::small_tiles;
    return grid_fits(most_tile_blocks(g), axo::TILE_THREADS) ? Kernel::tiles : Kernel::general;
}

int launch(const GemmArgs& g, int la, int lb, hipStream_t st) {
    switch (kernel_of(g, la, lb)) {
        case Kernel::none: return AXO_OK;
        case Kernel::tiles: return launch_tile_layout(g, la, lb, st);
        case Kernel::small_tiles: return launch_slim(g, la, lb, st);
        default: return launch_generic(g, la, lb, st);
    }
}

// The same choice as axo_fc_kernel reports it, down to the tile sizes of a call on its own.
int kernel_id(const GemmArgs& g, int la, int lb) {
    switch (kernel_of(g, la, lb)) {
        case Kernel::none: return AXO_KERNEL_NONE;
        case Kernel::general: return AXO_KERNEL_GENERAL;
        case Kernel::small_tiles:
            if (slim_rows(g, layout_pair(la, lb)) == 64) return AXO_KERNEL_SPLIT_64;
            return slim_two_stages(g) ? AXO_KERNEL_SPLIT_32_TWO_STAGES : AXO_KERNEL_SPLIT_32;
        default: break;
    }
    switch (tiles_of(g.Mo, g.No, g.R)) {
        case Tiles::small: return AXO_KERNEL_TILES_64;
        case Tiles::wide: return AXO_KERNEL_TILES_64_128;
        case Tiles::tall: return AXO_KERNEL_TILES_128_64;
        case Tiles::mid: return AXO_KERNEL_TILES_128;
        default: break;
    }
    const axo::TileSched sc = plan_product(g, la, lb);
    return sc.small_cols == 0 ? AXO_KERNEL_TILES_256 : sc.big_cols == 0 ? AXO_KERNEL_TILES_256_HALF : AXO_KERNEL_TILES_256_MIXED;
}

// The kinds of tiles of a call on its own, as axo_fc_tiles reports them.
int tile_bits(int kernel, bool lines) { return (1 << kernel) | (lines ? AXO_TILES_BY_LINES << kernel : 0); }
int tiles_id(const GemmArgs& g, int la, int lb) {
    const int kernel = kernel_id(g, la, lb);
    if (kernel == AXO_KERNEL_NONE) return 0;
    if (kernel < AXO_KERNEL_TILES_256 || kernel > AXO_KERNEL_TILES_256_MIXED) {
        const bool ring = kernel >= AXO_KERNEL_TILES_64;
        return tile_bits(kernel, ring && takes_lines(g, la, lb, kernel == AXO_KERNEL_TILES_64 ? Tile::t64 : Tile::t128));
    }
    const axo::TileSched sc = plan_product(g, la, lb);
    const Lines lines = lines_of(g, la, lb, sc);
    return (sc.n_big > 0 ? tile_bits(AXO_KERNEL_TILES_256, lines != LINES_NONE) : 0) |
           (sc.small_cols > 0 ? tile_bits(AXO_KERNEL_TILES_256_HALF, lines == LINES_ALL) : 0);
}

// How the shape fits the 256 x 128 granularity of the tiles, for axo_fc_route.
int route_of(const GemmArgs& g, int la, int lb) {
    if (g.Mo == 0 || g.No == 0) return AXO_ROUTE_NONE;
    if (!spans_ok(g, la, lb) || g.R == 0 || g.Mo < 256 || g.No < 128) return AXO_ROUTE_GENERAL;
    return g.Mo % 256 == 0 && g.No % 128 == 0 ? AXO_ROUTE_TILED : AXO_ROUTE_COVERED;
}

int check_no_alias(const Plan& pl);  // defined with the byte-range code below

int plan_fwd(const axo_problem_t* p, const void* X, int64_t ldx, const void* W, int64_t ldw, const void* bias,
             int epilogue, void* Y, int64_t ldy, void* ws, size_t ws_bytes, Plan* out) {
    Shard s;
    int rc = derive_shard(p, &s);
    if (rc) return rc;
    if (epilogue < AXO_EPI_NONE || epilogue > AXO_EPI_BIAS_GELU_ERF) return AXO_ERR_BAD_EPILOGUE;
    if (epilogue != AXO_EPI_NONE && !bias) return AXO_ERR_BAD_EPILOGUE;
    if ((rc = check_matrix(X, ldx, s.M, s.Kl))) return rc;
    if ((rc = check_matrix(W, ldw, s.Kl, s.Nl))) return rc;
    if ((rc = check_matrix(Y, ldy, s.M, s.Nl))) return rc;
    if (epilogue != AXO_EPI_NONE && !aligned16(bias)) return AXO_ERR_MISALIGNED;
    if ((rc = check_workspace(p, AXO_OP_FWD, ws, ws_bytes))) return rc;
    GemmArgs& g = out->g;
    g.A = static_cast<const axo::bf16_t*>(X); g.lda = ldx;
    g.B = static_cast<const axo::bf16_t*>(W); g.ldb = ldw;
    g.C = static_cast<axo::bf16_t*>(Y); g.ldc = ldy;
    g.bias = static_cast<const axo::bf16_t*>(bias);
    g.aux = nullptr; g.ldaux = 0;
    g.Mo = (int)s.M; g.No = (int)s.Nl; g.R = (int)s.Kl;
    g.epilogue = epilogue;
    g.add_bias = (epilogue != AXO_EPI_NONE && s.k_coord == 0) ? 1 : 0;
    out->la = axo::KC; out->lb = axo::MC;
    return check_no_alias(*out);
}

int plan_dgrad(const axo_problem_t* p, const void* dY, int64_t lddy, const void* W, int64_t ldw, void* dX,
               int64_t lddx, void* ws, size_t ws_bytes, Plan* out) {
    Shard s;
    int rc = derive_shard(p, &s);
    if (rc) return rc;
    if ((rc = check_matrix(dY, lddy, s.M, s.Nl))) return rc;
    if ((rc = check_matrix(W, ldw, s.Kl, s.Nl))) return rc;
    if ((rc = check_matrix(dX, lddx, s.M, s.Kl))) return rc;
    if ((rc = check_workspace(p, AXO_OP_DGRAD, ws, ws_bytes))) return rc;
    GemmArgs& g = out->g;
    g.A = static_cast<const axo::bf16_t*>(dY); g.lda = lddy;
    g.B = static_cast<const axo::bf16_t*>(W); g.ldb = ldw;
    g.C = static_cast<axo::bf16_t*>(dX); g.ldc = lddx;
    g.bias = nullptr;
    g.aux = nullptr; g.ldaux = 0;
    g.Mo = (int)s.M; g.No = (int)s.Kl; g.R = (int)s.Nl;
    g.epilogue = AXO_EPI_NONE; g.add_bias = 0;
    out->la = axo::KC; out->lb = axo::KC;
    return check_no_alias(*out);
}

int plan_wgrad(const axo_problem_t* p, const void* X, int64_t ldx, const void* dY, int64_t lddy, void* dW,
               int64_t lddw, void* ws, size_t ws_bytes, Plan* out) {
    Shard s;
    int rc = derive_shard(p, &s);
    if (rc) return rc;
    if ((rc = check_matrix(X, ldx, s.M, s.Kl))) return rc;
    if ((rc = check_matrix(dY, lddy, s.M, s.Nl))) return rc;
    if ((rc = check_matrix(dW, lddw, s.Kl, s.Nl))) return rc;
    if ((rc = check_workspace(p, AXO_OP_WGRAD, ws, ws_bytes))) return rc;
    GemmArgs& g = out->g;
    g.A = static_cast<const axo::bf16_t*>(X); g.lda = ldx;
    g.B = static_cast<const axo::bf16_t*>(dY); g.ldb = lddy;
    g.C = static_cast<axo::bf16_t*>(dW); g.ldc = lddw;
    g.bias = nullptr;
    g.aux = nullptr; g.ldaux = 0;
    g.Mo = (int)s.Kl; g.No = (int)s.Nl; g.R = (int)s.M;
    g.epilogue = AXO_EPI_NONE; g.add_bias = 0;
    out->la = axo::MC; out->lb = axo::MC;
    return check_no_alias(*out);
}

int plan_bias_grad(const axo_problem_t* p, const void* dY, int64_t lddy, float* db, int accumulate, Plan* out) {
    Shard s;
    int rc = derive_shard(p, &s);
    if (rc) return rc;
    if (accumulate != 0 && accumulate != 1) return AXO_ERR_BAD_ARG;
    if ((rc = check_matrix(dY, lddy, s.M, s.Nl))) return rc;
    out->bias_grad = true;
    out->bg.dY = static_cast<const axo::bf16_t*>(dY);
    out->bg.lddy = lddy;
    out->bg.db = db;
    out->bg.M = (int)s.M;
    out->bg.Nl = (int)s.Nl;
    out->bg.accumulate = accumulate;
    if (s.Nl == 0) return AXO_OK;
    if (!db) return AXO_ERR_NULL_PTR;
    if (reinterpret_cast<uintptr_t>(db) & 3u) return AXO_ERR_MISALIGNED;
    return check_no_alias(*out);
}

int launch_bias_grad(const axo::BiasGradArgs& g, hipStream_t st) {
    if (g.Nl == 0) return AXO_OK;
    auto blocks = [&](int cols) { return (unsigned)((g.Nl + cols - 1) / cols); };
    // the widest column block that still gives a quarter (an eighth) of the CUs a workgroup
    if (blocks(64) >= (unsigned)NUM_CU / 4)
        hipLaunchKernelGGL(axo::bias_grad_kernel<64>, dim3(blocks(64)), dim3(axo::BG_THREADS), 0, st, g);
    else if (blocks(32) >= (unsigned)NUM_CU / 8)
        hipLaunchKernelGGL(axo::bias_grad_kernel<32>, dim3(blocks(32)), dim3(axo::BG_THREADS), 0, st, g);
    else
        hipLaunchKernelGGL(axo::bias_grad_kernel<16>, dim3(blocks(16)), dim3(axo::BG_THREADS), 0, st, g);
    return hipGetLastError() == hipSuccess ? AXO_OK : AXO_ERR_HIP;
}

// ---- bias gradient with the rows split over workgroups (needs scratch memory) ----------------
// How a shape is cut at most, and what its workspace is sized for: 64-column strips, each cut into S row slices
// of a multiple of 64 rows so that about BIAS_SPLIT_WORKGROUPS workgroups are in flight, no slice below 128 rows.  A
// launch uses launch_slices() of them, up to eight times fewer.  Both are functions of the shape alone, so the
// summation order (and with it every bit of the result) is too.  Measured on 4096 rows (time per call in a loop, launch included; 6144 / 16384 / 1536 columns): 128
// workgroups 14.6 / 25.0 / 9.0 us, 256: 12.6 / 22.0 / 8.4, 384: 11.6 / 22.4 / 10.5, 512: 11.6 / 22.2 /
// 10.6, 1024: 15.2 / 27.4 / 17.1 (every slice costs a publication and a share of the final
// addition); the strips of axo_bias_grad: 15.6 / 24.6 / 14.7.
constexpr int BIAS_SPLIT_WORKGROUPS = 384;
struct BiasSplit {
    int strips, S, rows_per_slice;
    size_t counter_bytes, partial_bytes;  // scratch layout: [counters][partial sums]
    size_t bytes() const { return S > 1 ? counter_bytes + partial_bytes : 0; }
};
BiasSplit plan_bias_split(int64_t M, int64_t Nl) {
    BiasSplit b{};
    b.strips = (int)((Nl + axo::BGS_COLS - 1) / axo::BGS_COLS);
    b.S = 1;
    b.rows_per_slice = (int)((M + axo::BGS_ROW_LANES - 1) / axo::BGS_ROW_LANES * axo::BGS_ROW_LANES);
    if (b.strips > 0 && M > 0) {
        int64_t want = (BIAS_SPLIT_WORKGROUPS + b.strips / 2) / b.strips;
        want = std::min<int64_t>(std::min<int64_t>(want, axo::BGS_MAX_SPLIT), M / 128);
        if (b.strips * (int64_t)sizeof(uint32_t) > axo::BGS_MAX_COUNTER_BYTES) want = 1;  // (it already is there)
        if (want > 1) {
            const int64_t rows = ((M + want - 1) / want + axo::BGS_ROW_LANES - 1) / axo::BGS_ROW_LANES * axo::BGS_ROW_LANES;
            b.rows_per_slice = (int)rows;
            b.S = (int)((M + rows - 1) / rows);
        }
    }
    b.counter_bytes = ((size_t)b.strips * sizeof(uint32_t) + 255) / 256 * 256;
    b.partial_bytes = (size_t)b.S * (size_t)Nl * sizeof(float);
    return b;
}

// Slices that a launch really uses, of the plan's at most: one per 1024 rows, none below 1536.  Publishing and
// adding slices costs 1.5 us and some 0.08 us per slice (their counts meet in one cache line), a batch of 512 rows
// of one workgroup 0.5 us.  Measured with the plan's own count / with this one: 7296 x 512 8.6 us (29 slices) / 6.0,
// 4096 x 1536 8.1 (16) / 5.2, 16384 x 256 7.5 (32) / 6.1, 1000 x 1000 5.3 (7) / 4.2, 300 x 300 4.6 (2) / 3.5.
BiasSplit launch_slices(BiasSplit b, int M) {
    const int64_t want = M <= 1536 ? 1 : ((int64_t)M + 1023) / 1024;
    if (want >= b.S) return b;
    b.rows_per_slice = (int)(((M + want - 1) / want + axo::BGS_ROW_LANES - 1) / axo::BGS_ROW_LANES * axo::BGS_ROW_LANES);
    b.S = M > 0 ? (int)(((int64_t)M + b.rows_per_slice - 1) / b.rows_per_slice) : 1;
    return b;
}

// Enqueues the split kernel on scratch memory laid out as BiasSplit says (ignored when S == 1).
int launch_bias_grad_split(const axo::BiasGradArgs& g, const BiasSplit& plan, void* scratch, hipStream_t st) {
    if (g.Nl == 0) return AXO_OK;
    const BiasSplit b = launch_slices(plan, g.M);
    axo::BiasGradSplitArgs a{};
    a.dY = g.dY;
    a.lddy = g.lddy;
    a.db = g.db;
    a.M = g.M;
    a.Nl = g.Nl;
    a.accumulate = g.accumulate;
    a.S = b.S;
    a.rows_per_slice = b.rows_per_slice;
    a.counters = static_cast<uint32_t*>(scratch);
    a.partial = reinterpret_cast<float*>(static_cast<char*>(scratch) + b.counter_bytes);
    hipLaunchKernelGGL(axo::bias_grad_split_kernel, dim3((unsigned)b.strips * (unsigned)b.S), dim3(axo::BGS_THREADS), 0, st, a);
    return hipGetLastError() == hipSuccess ? AXO_OK : AXO_ERR_HIP;
}

// Device address of this GPU's copy of `scratch`: asked for once per device, with that device
// current, and kept (each GPU holds its own copy at its own address).  No allocation.
int static_scratch(void** out) {
    static std::atomic<void*> known[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return AXO_ERR_HIP;
    const bool slot = dev >= 0 && dev < 64;
    if (slot) {
        if (void* p = known[dev].load(std::memory_order_acquire)) {
            *out = p;
            return AXO_OK;
        }
    }
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return AXO_ERR_HIP;
    if (slot) known[dev].store(p, std::memory_order_release);
    *out = p;
    return AXO_OK;
}

// one unit of work on its own
int launch_plan(const Plan& pl, hipStream_t st) {
    return pl.bias_grad ? launch_bias_grad(pl.bg, st) : launch(pl.g, pl.la, pl.lb, st);
}

// Validates a chain and lists its products in the order of Section 4.1: forwards of layers
// 0..n-1, then for layers n-1..0 dgrad followed by wgrad.  Nothing is launched here, so a chain
// with a malformed product enqueues nothing.
int plan_chain(const axo_layer_t* layers, int n_layers, void* ws, size_t ws_bytes, std::vector<Plan>* out) {
    if (n_layers < 0) return AXO_ERR_BAD_ARG;
    if (n_layers == 0) return AXO_OK;
    if (!layers) return AXO_ERR_NULL_PTR;
    if (n_layers > 4096) return AXO_ERR_BAD_ARG;
    out->resize(3 * (size_t)n_layers);
    for (int i = 0; i < n_layers; ++i) {
        const axo_layer_t& L = layers[i];
        if (L.reserved != 0) return AXO_ERR_BAD_ARG;
        int rc = plan_fwd(&L.p, L.X, L.ldx, L.W, L.ldw, L.bias, L.epilogue, L.Y, L.ldy, ws, ws_bytes, &(*out)[i]);
        if (rc) return rc;
        const size_t b = (size_t)n_layers + 2 * (size_t)(n_layers - 1 - i);
        rc = plan_dgrad(&L.p, L.dY, L.lddy, L.W, L.ldw, L.dX, L.lddx, ws, ws_bytes, &(*out)[b]);
        if (rc) return rc;
        rc = plan_wgrad(&L.p, L.X, L.ldx, L.dY, L.lddy, L.dW, L.lddw, ws, ws_bytes, &(*out)[b + 1]);
        if (rc) return rc;
    }
    return AXO_OK;
}

// dgrad with the activation's derivative fused in (see axo_fc_dgrad_act)
int plan_dgrad_act(const axo_problem_t* p, const void* dY, int64_t lddy, const void* W, int64_t ldw, const void* pre,
                   int64_t ldpre, int act, void* dX, int64_t lddx, void* ws, size_t ws_bytes, Plan* out) {
    if (act != AXO_EPI_BIAS_GELU_TANH && act != AXO_EPI_BIAS_GELU_ERF) return AXO_ERR_BAD_EPILOGUE;
    int rc = plan_dgrad(p, dY, lddy, W, ldw, dX, lddx, ws, ws_bytes, out);
    if (rc) return rc;
    if ((rc = check_matrix(pre, ldpre, out->g.Mo, out->g.No))) return rc;
    out->g.aux = static_cast<const axo::bf16_t*>(pre);
    out->g.ldaux = ldpre;
    out->g.epilogue = act == AXO_EPI_BIAS_GELU_TANH ? axo::EPI_MUL_DGELU_TANH : axo::EPI_MUL_DGELU_ERF;
    return check_no_alias(*out);
}

// wgrad accumulated into an fp32 matrix (see axo_fc_wgrad_acc)
int plan_wgrad_acc(const axo_problem_t* p, const void* X, int64_t ldx, const void* dY, int64_t lddy, float* dW32,
                   int64_t lddw, void* ws, size_t ws_bytes, Plan* out) {
    Shard s;
    int rc = derive_shard(p, &s);
    if (rc) return rc;
    if (s.Kl > 0 && s.Nl > 0) {  // the fp32 output: 16-byte aligned rows of 4-byte elements
        if (!dW32) return AXO_ERR_NULL_PTR;
        if (lddw < s.Nl) return AXO_ERR_BAD_LD;
        if (!aligned16(dW32) || (lddw % 4) != 0) return AXO_ERR_MISALIGNED;
    }
    // the bf16 checks of the output do not apply; validate the inputs through plan_wgrad with a stand-in
    rc = plan_wgrad(p, X, ldx, dY, lddy, dW32, (lddw + 7) / 8 * 8, ws, ws_bytes, out);
    if (rc) return rc;
    out->g.C = reinterpret_cast<axo::bf16_t*>(dW32);
    out->g.ldc = lddw;
    out->g.epilogue = axo::EPI_ACC_F32;
    return check_no_alias(*out);
}

// The chain of axo_layer_step_ext: 3 or 4 units per layer, in program order.
int plan_chain_ext(const axo_layer_ext_t* layers, int n_layers, void* ws, size_t ws_bytes, std::vector<Plan>* out) {
    if (n_layers < 0) return AXO_ERR_BAD_ARG;
    if (n_layers == 0) return AXO_OK;
    if (!layers) return AXO_ERR_NULL_PTR;
    if (n_layers > 4096) return AXO_ERR_BAD_ARG;
    out->clear();
    out->resize((size_t)n_layers);  // the forwards; the backward units are appended in order
    for (int i = 0; i < n_layers; ++i) {
        const axo_layer_t& L = layers[i].layer;
        if (L.reserved != 0) return AXO_ERR_BAD_ARG;
        const int rc = plan_fwd(&L.p, L.X, L.ldx, L.W, L.ldw, L.bias, L.epilogue, L.Y, L.ldy, ws, ws_bytes, &(*out)[i]);
        if (rc) return rc;
    }
    for (int i = n_layers - 1; i >= 0; --i) {
        const axo_layer_ext_t& E = layers[i];
        const axo_layer_t& L = E.layer;
        if (E.accumulate_db != 0 && E.accumulate_db != 1) return AXO_ERR_BAD_ARG;
        Plan pl;
        int rc;
        if (E.pre) {
            rc = plan_dgrad_act(&L.p, L.dY, L.lddy, L.W, L.ldw, E.pre, E.ldpre, E.act_below, L.dX, L.lddx, ws, ws_bytes, &pl);
        } else {
            if (E.act_below != 0) return AXO_ERR_BAD_EPILOGUE;
            rc = plan_dgrad(&L.p, L.dY, L.lddy, L.W, L.ldw, L.dX, L.lddx, ws, ws_bytes, &pl);
        }
        if (rc) return rc;
        out->push_back(pl);
        pl = Plan();
        rc = E.dW32 ? plan_wgrad_acc(&L.p, L.X, L.ldx, L.dY, L.lddy, E.dW32, E.lddw32, ws, ws_bytes, &pl)
                    : plan_wgrad(&L.p, L.X, L.ldx, L.dY, L.lddy, L.dW, L.lddw, ws, ws_bytes, &pl);
        if (rc) return rc;
        out->push_back(pl);
        if (E.db) {
            pl = Plan();
            rc = plan_bias_grad(&L.p, L.dY, L.lddy, E.db, E.accumulate_db, &pl);
            if (rc) return rc;
            out->push_back(pl);
        }
    }
    return AXO_OK;
}

// ---- dependence analysis of a chain --------------------------------------------------------
// Byte range [lo, hi) that a matrix argument covers (rows x row_len elements of elem bytes, rows
// ld elements apart); empty matrices cover nothing.  The matrix itself is kept beside its range
// for the exact overlap test.
struct Range {
    uintptr_t lo, hi;
    int64_t pitch, rows, width;  // bytes between rows, row count, bytes per row
    bool overlaps(const Range& o) const { return lo < o.hi && o.lo < hi; }
    // Do the two matrices share a byte?  (Ranges that overlap need not: two column blocks of one
    // buffer interleave.)  Row r of this matrix covers [a, a + width) relative to the other's
    // base; row q of the other covers [q * pitch, q * pitch + width_o); they meet iff
    // q * pitch < a + width and q * pitch + width_o > a, an interval of q that is clamped to the
    // other's rows.  Only called when the ranges overlap, which no well-formed call makes them do.
    bool shares_bytes_with(const Range& o) const {
        if (!overlaps(o)) return false;
        auto floor_div = [](int64_t x, int64_t y) { return x / y - ((x % y != 0) && ((x < 0) != (y < 0)) ? 1 : 0); };
        const int64_t op = o.rows > 1 ? o.pitch : (int64_t)(o.hi - o.lo) + 1;  // one row: any positive pitch
        for (int64_t r = 0; r < rows; ++r) {
            const int64_t a = (int64_t)(lo - o.lo) + r * pitch;
            const int64_t q_hi = std::min<int64_t>(floor_div(a + width - 1, op), o.rows - 1);
            const int64_t q_lo = std::max<int64_t>(floor_div(a - o.width, op) + 1, 0);
            if (q_lo <= q_hi) return true;
        }
        return false;
    }
};
bool matrix_range(const void* ptr, int64_t ld, int64_t rows, int64_t row_len, int elem, Range* r) {
    if (!ptr || rows <= 0 || row_len <= 0) return false;
    r->lo = reinterpret_cast<uintptr_t>(ptr);
    r->hi = r->lo + (uintptr_t)(((rows - 1) * ld + row_len) * elem);
    r->pitch = ld * elem;
    r->rows = rows;
    r->width = row_len * elem;
    return true;
}
// What one product reads and writes.  (Ranges, not elements: two column blocks interleaved in one
// buffer count as overlapping, which only costs concurrency.)
struct Footprint {
    Range in[4];
    int n_in = 0;
    Range out{0, 0, 0, 0, 0};
    bool has_out = false;
    bool conflicts_with_later(const Footprint& later) const {
        if (has_out) {
            if (later.has_out && out.overlaps(later.out)) return true;                 // write after write
            for (int k = 0; k < later.n_in; ++k)
                if (out.overlaps(later.in[k])) return true;                            // read after write
        }
        if (later.has_out)
            for (int k = 0; k < n_in; ++k)
                if (in[k].overlaps(later.out)) return true;                            // write after read
        return false;
    }
    // the output shares bytes with one of the product's own inputs
    bool output_aliases_input() const {
        if (!has_out) return false;
        for (int k = 0; k < n_in; ++k)
            if (out.shares_bytes_with(in[k])) return true;
        return false;
    }
};
Footprint footprint(const Plan& pl) {
    const GemmArgs& g = pl.g;
    Footprint f;
    if (pl.nothing_to_do()) return f;  // nothing is launched for it
    Range r;
    if (pl.bias_grad) {  // reads dY, writes (or updates) db
        if (matrix_range(pl.bg.dY, pl.bg.lddy, pl.bg.M, pl.bg.Nl, 2, &r)) f.in[f.n_in++] = r;
        f.has_out = matrix_range(pl.bg.db, pl.bg.Nl, 1, pl.bg.Nl, 4, &f.out);
        return f;
    }
    // A(i, r): KC is Mo rows of R elements, MC is R rows of Mo elements; B likewise with No
    if (pl.la == axo::KC ? matrix_range(g.A, g.lda, g.Mo, g.R, 2, &r) : matrix_range(g.A, g.lda, g.R, g.Mo, 2, &r))
        f.in[f.n_in++] = r;
    if (pl.lb == axo::KC ? matrix_range(g.B, g.ldb, g.No, g.R, 2, &r) : matrix_range(g.B, g.ldb, g.R, g.No, 2, &r))
        f.in[f.n_in++] = r;
    if (g.add_bias && matrix_range(g.bias, g.No, 1, g.No, 2, &r)) f.in[f.n_in++] = r;
    if (matrix_range(g.aux, g.ldaux, g.Mo, g.No, 2, &r)) f.in[f.n_in++] = r;
    f.has_out = matrix_range(g.C, g.ldc, g.Mo, g.No, g.epilogue == axo::EPI_ACC_F32 ? 4 : 2, &f.out);
    return f;
}
// The rule of the header, checked: an output that shares bytes with an input of its own product is
// refused.  The kernels write an output tile while other workgroups still read the operands, and
// the tiles along a ragged output's edge overlap and compute what they share twice, so an in-place call
// (say dX written over the pre-activation it is multiplied with) would silently go wrong.
int check_no_alias(const Plan& pl) { return footprint(pl).output_aliases_input() ? AXO_ERR_BAD_ARG : AXO_OK; }
// Dependence level of every product of a chain given in program order: 0 when it conflicts with
// no earlier product, otherwise one more than the highest level among the earlier products it
// conflicts with.  Products of one level are independent of each other, and every product a
// given one depends on sits on a lower level, so enqueueing level by level on one stream gives
// the results of the program order.  The pairwise comparison is quadratic; beyond
// MAX_ANALYSED products the chain simply keeps its order (level = position).  Returns the
// number of levels.
constexpr size_t MAX_ANALYSED = 768;  // 256 layers
int dependence_levels(const std::vector<Plan>& plans, std::vector<int>* level) {
    const size_t n = plans.size();
    level->assign(n, 0);
    if (n == 0) return 0;
    if (n > MAX_ANALYSED) {
        for (size_t j = 0; j < n; ++j) (*level)[j] = (int)j;
        return (int)n;
    }
    std::vector<Footprint> fp(n);
    for (size_t j = 0; j < n; ++j) fp[j] = footprint(plans[j]);
    int levels = 1;
    for (size_t j = 1; j < n; ++j) {
        int lv = 0;
        for (size_t i = 0; i < j; ++i)
            if ((*level)[i] >= lv && fp[i].conflicts_with_later(fp[j])) lv = (*level)[i] + 1;
        (*level)[j] = lv;
        if (lv + 1 > levels) levels = lv + 1;
    }
    return levels;
}

// One launch over the small tiles of several products (Kernel::small_tiles each, at most
// SLIM_GROUP_MAX, together no more tiles than a grid holds).  Both tile sizes sum in the same order, so the size is the group's to choose.
template <int ROWS>
int launch_slim_group_rows(const std::vector<const Plan*>& plans, hipStream_t st) {
    using C = axo::SlimCfg<ROWS, ROWS, axo::SLIM_WAVES, 1>;
    auto kern = axo::gemm_slim_group_kernel<ROWS>;
    static std::atomic<uint64_t> raised{0};
    if (!raise_lds_limit(reinterpret_cast<const void*>(kern), C::LDS_BYTES, &raised)) return AXO_ERR_HIP;
    axo::SlimGroupArgs ga{};
    ga.n = (int)plans.size();
    int64_t blocks = 0;
    for (int i = 0; i < ga.n; ++i) {
        const GemmArgs& g = plans[i]->g;
        ga.first_block[i] = (int)blocks;
        ga.pair[i] = layout_pair(plans[i]->la, plans[i]->lb);
        ga.sched[i] = {(g.Mo + ROWS - 1) / ROWS, (g.No + ROWS - 1) / ROWS, 0};
        ga.sched[i].group_m = std::min(ga.sched[i].tiles_m, 8);
        ga.g[i] = g;
        blocks += (int64_t)ga.sched[i].tiles_m * ga.sched[i].tiles_n;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(C::THREADS), C::LDS_BYTES, st, ga);
    return hipGetLastError() == hipSuccess ? AXO_OK : AXO_ERR_HIP;
}
// Rows of its tiles, 0 where the products are launched one by one, each of which fits.  Puts long reductions first.
int slim_group_rows(std::vector<const Plan*>& plans) {
    int64_t blocks[2] = {0, 0};
    for (const Plan* pl : plans)
        for (int m = 0; m < 2; ++m) blocks[m] += tiles_in(pl->g.Mo, SLIM_MODEL[m].rows) * tiles_in(pl->g.No, SLIM_MODEL[m].rows);
    if (plans.size() == 1 || !grid_fits(blocks[1], axo::SLIM_WAVES * 64)) return 0;
    std::stable_sort(plans.begin(), plans.end(), [](const Plan* a, const Plan* b) { return a->g.R > b->g.R; });
    double us[2];
    for (int m = 0; m < 2; ++m) {
        double busy = 0.0, chain = 0.0;
        for (const Plan* pl : plans) {
            const double tile = slim_tile_us(SLIM_MODEL[m], pl->g.R, layout_pair(pl->la, pl->lb));
            busy += slim_tiles(SLIM_MODEL[m], pl->g.Mo, pl->g.No) * tile / NUM_CU;
            chain = std::max(chain, slim_chain_us(SLIM_MODEL[m], pl->g.R));
        }
        us[m] = std::max(busy, chain);
    }
    return us[0] <= us[1] && grid_fits(blocks[0], axo::SLIM_WAVES * 64) ? 32 : 64;
}
int launch_slim_group(std::vector<const Plan*> plans, hipStream_t st) {
    const int rows = slim_group_rows(plans);
    if (rows == 0) {
        int rc = AXO_OK;
        for (size_t i = 0; i < plans.size() && rc == AXO_OK; ++i) rc = launch_slim(plans[i]->g, plans[i]->la, plans[i]->lb, st);
        return rc;
    }
    return rows == 32 ? launch_slim_group_rows<32>(plans, st) : launch_slim_group_rows<64>(plans, st);
}

// What becomes of the launches that a chain is cut into: enqueued on a stream, or reported (axo_layer_step_tiles).
struct Enqueue {
    hipStream_t st;
    int group(const Plan* const* plans, int n) { return launch_group(plans, n, st); }
    int small_group(const std::vector<const Plan*>& plans) { return launch_slim_group(plans, st); }
    int one(const Plan& pl) { return launch_plan(pl, st); }
};
struct Report {
    const Plan* first;  // of the chain
    int* tiles;         // per unit of work
    int group(const Plan* const* plans, int n) {
        axo::GroupArgs ga{};
        bool lines;
        group_launch(plans, n, ga, lines);
        for (int k = 0; k < ga.n_seg; ++k) {
            const int kind = ga.seg[k].kind;
            if (kind == axo::GROUP_KIND_BIAS_GRAD) continue;
            const bool by_lines = kind >= axo::GROUP_KIND_LINES;
            const int kernel = !by_lines && kind >= axo::GROUP_KIND_PAIR ? AXO_KERNEL_TILES_64
                               : !by_lines && kind >= axo::GROUP_KIND_SLIM ? AXO_KERNEL_SPLIT_64
                               : kind % 2 ? AXO_KERNEL_TILES_256_HALF : AXO_KERNEL_TILES_256;
            tiles[plans[ga.seg[k].product] - first] |= tile_bits(kernel, by_lines);
        }
        return AXO_OK;
    }
    int small_group(std::vector<const Plan*> plans) {
        const int rows = slim_group_rows(plans);
        for (const Plan* pl : plans)
            if (rows == 0) one(*pl);
            else tiles[pl - first] |= tile_bits(rows == 32 ? AXO_KERNEL_SPLIT_32 : AXO_KERNEL_SPLIT_64, false);
        return AXO_OK;
    }
    int one(const Plan& pl) {
        if (!pl.bias_grad) tiles[&pl - first] |= tiles_id(pl.g, pl.la, pl.lb);
        return AXO_OK;
    }
};

// Cuts a chain into launches level by level: the products of a level that the tiled kernel takes share
// grouped launches (GROUP_MAX_PRODUCTS per launch), those on small tiles likewise, the others get a launch of their own.
template <typename Sink>
int by_level(std::vector<Plan>& plans, const std::vector<int>& level, int levels, Sink sink) {
    int rc = AXO_OK;
    std::vector<const Plan*> group;   // products of the level the tiled kernel takes
    std::vector<const Plan*> small;   // products of the level that run on small tiles
    auto flush_small = [&]() {
        if (!small.empty() && rc == AXO_OK) rc = sink.small_group(small);
        small.clear();
    };
    std::vector<const Plan*> riders;  // bias gradients of the level that may share their launch
    int64_t group_blocks = 0;         // at most so many workgroups in the group so far
    auto blocks_of = [](const Plan& pl) -> int64_t {
        return pl.bias_grad ? bias_strips(pl.bg.Nl) : pl.small ? slim_pair_blocks(pl.g.Mo, pl.g.No) : std::max<int64_t>(most_tile_blocks(pl.g), MOST_PAIRS);
    };
    auto joins = [&](const Plan& pl) { return grid_fits(group_blocks + blocks_of(pl), axo::TILE_THREADS); };
    auto join = [&](const Plan* pl) {
        group_blocks += blocks_of(*pl);
        group.push_back(pl);
    };
    auto flush = [&]() {
        group_blocks = 0;
        if (group.empty() || rc != AXO_OK) return;
        rc = group.size() == 1 ? sink.one(*group[0]) : sink.group(group.data(), (int)group.size());
        group.clear();
    };
    // the last launch of a level takes the level's small products and bias gradients along, as many as fit
    auto flush_level = [&]() {
        for (std::vector<const Plan*>* list : {&small, &riders})
            while (!list->empty() && !group.empty() && (int)group.size() < axo::GROUP_MAX_PRODUCTS && joins(*list->back())) {
                join(list->back());
                list->pop_back();
            }
        flush();
        flush_small();
        for (size_t k = 0; k < riders.size() && rc == AXO_OK; ++k) rc = sink.one(*riders[k]);
        riders.clear();
    };
    for (int lv = 0; lv < levels && rc == AXO_OK; ++lv) {
        for (size_t i = 0; i < plans.size() && rc == AXO_OK; ++i) {
            Plan& pl = plans[i];
            if (level[i] != lv || pl.nothing_to_do()) continue;
            if (pl.bias_grad) {
                if (bias_grad_groupable(pl.bg)) riders.push_back(&pl);
                else rc = sink.one(pl);
                continue;
            }
            const Kernel kernel = kernel_of(pl.g, pl.la, pl.lb);
            if (kernel == Kernel::small_tiles) {
                pl.small = true;
                small.push_back(&pl);
                if ((int)small.size() == axo::SLIM_GROUP_MAX) flush_small();
                continue;
            }
            if (kernel != Kernel::tiles) {
                rc = sink.one(pl);
                continue;
            }
            if (!group.empty() && !joins(pl)) flush();
            join(&pl);
            if ((int)group.size() == axo::GROUP_MAX_PRODUCTS) flush();
        }
        flush_level();
    }
    return rc;
}

// A validated chain, scheduled by dependence level.
template <typename Sink>
int scheduled(std::vector<Plan>& plans, Sink sink) {
    if (plans.size() > MAX_ANALYSED) {  // not analysed: program order, one unit per launch
        int rc = AXO_OK;
        for (size_t i = 0; i < plans.size() && rc == AXO_OK; ++i) rc = sink.one(plans[i]);
        return rc;
    }
    std::vector<int> level;
    const int levels = dependence_levels(plans, &level);
    return by_level(plans, level, levels, sink);
}

// The product that a query asks about: the planners compare pointers, never follow them.
int plan_query(const axo_problem_t* p, int op, const void* a, int64_t ld_a, const void* b, int64_t ld_b, void* c, int64_t ld_out, Plan* pl) {
    if (op < AXO_OP_FWD || op > AXO_OP_WGRAD) return AXO_ERR_BAD_ARG;
    if (op == AXO_OP_FWD) return plan_fwd(p, a, ld_a, b, ld_b, nullptr, AXO_EPI_NONE, c, ld_out, nullptr, 0, pl);
    if (op == AXO_OP_DGRAD) return plan_dgrad(p, a, ld_a, b, ld_b, c, ld_out, nullptr, 0, pl);
    return plan_wgrad(p, a, ld_a, b, ld_b, c, ld_out, nullptr, 0, pl);
}
void* made_up(int n) { return reinterpret_cast<void*>((uintptr_t)n << 40); }  // well-separated and aligned
int plan_query(const axo_problem_t* p, int op, int64_t ld_a, int64_t ld_b, int64_t ld_out, Plan* pl) {
    return plan_query(p, op, made_up(1), ld_a, made_up(2), ld_b, made_up(3), ld_out, pl);
}

// No exception leaves the library: the planners keep their lists and caches in standard
// containers, whose allocations can fail.
template <typename F>
int guarded(F&& body) noexcept {
    try {
        return body();
    } catch (const std::bad_alloc&) {
        return AXO_ERR_NO_MEMORY;
    } catch (...) {
        return AXO_ERR_BAD_ARG;
    }
}

}  // namespace

extern "C" {

int axo_version(void) { return AXO_VERSION; }

const char* axo_status_string(int status) {
    switch (status) {
        case AXO_OK: return "ok";
        case AXO_ERR_BAD_GRID: return "grid dimension < 1";
        case AXO_ERR_BAD_COORD: return "grid coordinate outside the grid";
        case AXO_ERR_INDIVISIBLE: return "T, K or N not divisible by its grid dimension";
        case AXO_ERR_NULL_PTR: return "required pointer is NULL";
        case AXO_ERR_MISALIGNED: return "pointer not 16-byte aligned or leading dimension not a multiple of 8";
        case AXO_ERR_BAD_LD: return "leading dimension smaller than the row length";
        case AXO_ERR_WORKSPACE: return "workspace too small";
        case AXO_ERR_BAD_EPILOGUE: return "unknown epilogue or epilogue without bias";
        case AXO_ERR_HIP: return "HIP launch failed";
        case AXO_ERR_BAD_SIZE: return "negative size or shard dimension beyond 2^31-1";
        case AXO_ERR_BAD_ARG: return "malformed argument";
        case AXO_ERR_NO_MEMORY: return "host allocation failed";
        case AXO_ERR_TOO_LARGE: return "problem needs more scratch memory than the allocation-free entry point holds";
        default: return "unknown status";
    }
}

int axo_shard_dims(const axo_problem_t* p, int64_t* M, int64_t* Kl, int64_t* Nl, int64_t* row0, int64_t* k0,
                   int64_t* n0) {
    Shard s;
    int rc = derive_shard(p, &s);
    if (rc) return rc;
    if (M) *M = s.M;
    if (Kl) *Kl = s.Kl;
    if (Nl) *Nl = s.Nl;
    if (row0) *row0 = s.row0;
    if (k0) *k0 = s.k0;
    if (n0) *n0 = s.n0;
    return AXO_OK;
}

size_t axo_workspace_bytes(const axo_problem_t* p, int op) {
    Shard s;
    if (derive_shard(p, &s) != AXO_OK) return 0;
    if (op < AXO_OP_FWD || op > AXO_OP_WGRAD) return 0;
    return 0;  // no product needs workspace at present; the argument is kept for split reductions
}

int axo_fc_route(const axo_problem_t* p, int op, int64_t ld_a, int64_t ld_b, int64_t ld_out, int* route) {
    return guarded([&]() -> int {
        if (!route) return AXO_ERR_NULL_PTR;
        Plan pl;
        const int rc = plan_query(p, op, ld_a, ld_b, ld_out, &pl);
        if (rc) return rc;
        *route = route_of(pl.g, pl.la, pl.lb);
        return AXO_OK;
    });
}

int axo_fc_kernel(const axo_problem_t* p, int op, int64_t ld_a, int64_t ld_b, int64_t ld_out, int* kernel) {
    return guarded([&]() -> int {
        if (!kernel) return AXO_ERR_NULL_PTR;
        Plan pl;
        const int rc = plan_query(p, op, ld_a, ld_b, ld_out, &pl);
        if (rc) return rc;
        *kernel = kernel_id(pl.g, pl.la, pl.lb);
        return AXO_OK;
    });
}

int axo_fc_tiles(const axo_problem_t* p, int op, const void* a, int64_t ld_a, const void* b, int64_t ld_b, int64_t ld_out, int* tiles) {
    return guarded([&]() -> int {
        if (!tiles) return AXO_ERR_NULL_PTR;
        Plan pl;
        const int rc = plan_query(p, op, a, ld_a, b, ld_b, made_up(1 << 20), ld_out, &pl);  // an output far from any input
        if (rc) return rc;
        *tiles = tiles_id(pl.g, pl.la, pl.lb);
        return AXO_OK;
    });
}

int axo_fc_fwd(const axo_problem_t* p, const void* X, int64_t ldx, const void* W, int64_t ldw, const void* bias,
               int epilogue, void* Y, int64_t ldy, void* ws, size_t ws_bytes, void* hip_stream) {
    return guarded([&]() -> int {
        Plan pl;
        int rc = plan_fwd(p, X, ldx, W, ldw, bias, epilogue, Y, ldy, ws, ws_bytes, &pl);
        if (rc) return rc;
        return launch(pl.g, pl.la, pl.lb, static_cast<hipStream_t>(hip_stream));
    });
}

int axo_fc_dgrad(const axo_problem_t* p, const void* dY, int64_t lddy, const void* W, int64_t ldw, void* dX,
                 int64_t lddx, void* ws, size_t ws_bytes, void* hip_stream) {
    return guarded([&]() -> int {
        Plan pl;
        int rc = plan_dgrad(p, dY, lddy, W, ldw, dX, lddx, ws, ws_bytes, &pl);
        if (rc) return rc;
        return launch(pl.g, pl.la, pl.lb, static_cast<hipStream_t>(hip_stream));
    });
}

int axo_fc_wgrad(const axo_problem_t* p, const void* X, int64_t ldx, const void* dY, int64_t lddy, void* dW,
                 int64_t lddw, void* ws, size_t ws_bytes, void* hip_stream) {
    return guarded([&]() -> int {
        Plan pl;
        int rc = plan_wgrad(p, X, ldx, dY, lddy, dW, lddw, ws, ws_bytes, &pl);
        if (rc) return rc;
        return launch(pl.g, pl.la, pl.lb, static_cast<hipStream_t>(hip_stream));
    });
}

int axo_fc_dgrad_act(const axo_problem_t* p, const void* dY, int64_t lddy, const void* W, int64_t ldw, const void* pre,
                     int64_t ldpre, int act, void* dX, int64_t lddx, void* ws, size_t ws_bytes, void* hip_stream) {
    return guarded([&]() -> int {
        Plan pl;
        int rc = plan_dgrad_act(p, dY, lddy, W, ldw, pre, ldpre, act, dX, lddx, ws, ws_bytes, &pl);
        if (rc) return rc;
        return launch(pl.g, pl.la, pl.lb, static_cast<hipStream_t>(hip_stream));
    });
}

int axo_fc_wgrad_acc(const axo_problem_t* p, const void* X, int64_t ldx, const void* dY, int64_t lddy, float* dW,
                     int64_t lddw, void* ws, size_t ws_bytes, void* hip_stream) {
    return guarded([&]() -> int {
        Plan pl;
        int rc = plan_wgrad_acc(p, X, ldx, dY, lddy, dW, lddw, ws, ws_bytes, &pl);
        if (rc) return rc;
        return launch(pl.g, pl.la, pl.lb, static_cast<hipStream_t>(hip_stream));
    });
}

int axo_bias_grad(const axo_problem_t* p, const void* dY, int64_t lddy, float* db, int accumulate, void* hip_stream) {
    Plan pl;
    const int rc = plan_bias_grad(p, dY, lddy, db, accumulate, &pl);
    if (rc) return rc;
    return launch_bias_grad(pl.bg, static_cast<hipStream_t>(hip_stream));
}

size_t axo_bias_grad_workspace_bytes(const axo_problem_t* p) {
    Shard s;
    if (derive_shard(p, &s) != AXO_OK) return 0;
    return plan_bias_split(s.M, s.Nl).bytes();
}

int axo_bias_grad_ws(const axo_problem_t* p, const void* dY, int64_t lddy, float* db, int accumulate, void* ws,
                     size_t ws_bytes, void* hip_stream) {
    Plan pl;
    const int rc = plan_bias_grad(p, dY, lddy, db, accumulate, &pl);
    if (rc) return rc;
    const BiasSplit b = plan_bias_split(pl.bg.M, pl.bg.Nl);
    if (b.bytes() > 0) {
        if (!ws || ws_bytes < b.bytes()) return AXO_ERR_WORKSPACE;
        if (!aligned16(ws)) return AXO_ERR_MISALIGNED;
    }
    return launch_bias_grad_split(pl.bg, b, ws, static_cast<hipStream_t>(hip_stream));
}

int axo_bias_grad_static(const axo_problem_t* p, const void* dY, int64_t lddy, float* db, int accumulate,
                         void* hip_stream) {
    Plan pl;
    const int rc = plan_bias_grad(p, dY, lddy, db, accumulate, &pl);
    if (rc) return rc;
    if (pl.bg.Nl == 0) return AXO_OK;
    const BiasSplit b = plan_bias_split(pl.bg.M, pl.bg.Nl);
    if (b.bytes() > STATIC_SCRATCH_BYTES) return AXO_ERR_TOO_LARGE;
    void* dev_scratch = nullptr;
    if (b.bytes() > 0) {
        const int sc = static_scratch(&dev_scratch);
        if (sc) return sc;
    }
    return launch_bias_grad_split(pl.bg, b, dev_scratch, static_cast<hipStream_t>(hip_stream));
}

size_t axo_bias_grad_static_limit(void) { return STATIC_SCRATCH_BYTES; }

size_t axo_layer_step_workspace_bytes(const axo_layer_t* layers, int n_layers) {
    size_t need = 0;
    if (!layers) return 0;
    for (int i = 0; i < n_layers; ++i)
        for (int op = AXO_OP_FWD; op <= AXO_OP_WGRAD; ++op) {
            size_t b = axo_workspace_bytes(&layers[i].p, op);
            if (b > need) need = b;
        }
    return need;
}

int axo_layer_step(const axo_layer_t* layers, int n_layers, void* ws, size_t ws_bytes, void* hip_stream) {
    return guarded([&]() -> int {
        std::vector<Plan> plans;
        const int rc = plan_chain(layers, n_layers, ws, ws_bytes, &plans);
        if (rc != AXO_OK) return rc;
        return scheduled(plans, Enqueue{static_cast<hipStream_t>(hip_stream)});
    });
}

int axo_layer_step_ext(const axo_layer_ext_t* layers, int n_layers, void* ws, size_t ws_bytes, void* hip_stream) {
    return guarded([&]() -> int {
        std::vector<Plan> plans;
        const int rc = plan_chain_ext(layers, n_layers, ws, ws_bytes, &plans);
        if (rc != AXO_OK) return rc;
        return scheduled(plans, Enqueue{static_cast<hipStream_t>(hip_stream)});
    });
}

int axo_layer_step_ordered(const axo_layer_t* layers, int n_layers, void* ws, size_t ws_bytes, void* hip_stream) {
    return guarded([&]() -> int {
        std::vector<Plan> plans;
        int rc = plan_chain(layers, n_layers, ws, ws_bytes, &plans);
        for (size_t i = 0; i < plans.size() && rc == AXO_OK; ++i)
            rc = launch_plan(plans[i], static_cast<hipStream_t>(hip_stream));
        return rc;
    });
}

int axo_layer_step_levels(const axo_layer_t* layers, int n_layers, int* n_levels, int* levels) {
    return guarded([&]() -> int {
        if (!n_levels) return AXO_ERR_NULL_PTR;
        std::vector<Plan> plans;
        const int rc = plan_chain(layers, n_layers, nullptr, 0, &plans);
        if (rc != AXO_OK) return rc;
        std::vector<int> level;
        *n_levels = dependence_levels(plans, &level);
        if (levels)
            for (size_t i = 0; i < level.size(); ++i) levels[i] = level[i];
        return AXO_OK;
    });
}

int axo_layer_step_tiles(const axo_layer_ext_t* layers, int n_layers, int* tiles) {
    return guarded([&]() -> int {
        if (!tiles) return AXO_ERR_NULL_PTR;
        std::vector<Plan> plans;
        const int rc = plan_chain_ext(layers, n_layers, nullptr, 0, &plans);
        if (rc != AXO_OK) return rc;
        std::fill(tiles, tiles + plans.size(), 0);
        return scheduled(plans, Report{plans.data(), tiles});
    });
}

}  // extern "C"
