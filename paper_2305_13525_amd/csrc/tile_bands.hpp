// Host side: band height of the tile order of a weight gradient that runs at once.  Each XCD gets a run of tiles (xcd_run), and what its 4 MB of L2
// have to take in are the operand panels of the tile rows and columns that the run touches, so the run should be as square as bands
// allow.  Panels come over the fabric, at 4.5 TB/s for all XCDs, which is what such launches with long reductions are bound by.  8 rows / the best
// in us: 512 x 512 of 4096 tokens 19.1 / 14.9 (bands of 4), 768 x 768 of 2048 9.0 / 8.3, 1536 x 1536 of 4096 on 128 x 128 tiles 26.3 / 25.9; nothing
// lost at 1024 x 1024 of 512.  Products whose A lies along the reduction gain less by it and lose where rows are a power of two
// apart (forward 512 x 1024 x 1024 5.7 us with 8 rows, 6.0 with 4; 5.9 and 5.8 with 64 elements of padding): those keep 8.
#pragma once
#include <algorithm>
#include <array>
#include <atomic>
#include <climits>
#include <cstdint>

namespace axo {

constexpr int BAND_MAX_TILES = 512;  // at most two tiles per CU: beyond that they do not run at once
constexpr int BAND_MAX_ROWS = 16;

// What the XCDs have to take in, in rows and columns of operand panels, if tiles of rows x cols are ordered in bands of h tile rows and each of
// `xcds` takes a run of them (xcd_run, tile_of_index).
inline int band_cost(int tiles_m, int tiles_n, int rows, int cols, int xcds, int h) {
    const int n = tiles_m * tiles_n, band = h * tiles_n;
    // tiles t0 to t1 of band b
    auto part = [=](int b, int t0, int t1) {
        const int height = std::min(h, tiles_m - b * h), first = b * band;
        return std::min(height, t1 - t0) * rows + ((t1 - 1 - first) / height - (t0 - first) / height + 1) * cols;
    };
    int cost = 0;
    for (int x = 0, t0 = 0; x < xcds && t0 < n; ++x) {
        const int t1 = t0 + n / xcds + (x < n % xcds), b0 = t0 / band, b1 = (t1 - 1) / band;
        if (t1 == t0) continue;
        if (b0 == b1) cost += part(b0, t0, t1);
        else cost += part(b0, t0, (b0 + 1) * band) + (b1 - b0 - 1) * (h * rows + tiles_n * cols) + part(b1, b1 * band, t1);
        t0 = t1;
    }
    return cost;
}

// The height of the bands: the tallest of the cheapest.  Kept per grid of tiles, in a table that has a place for each, without a lock; a grid's
// first search takes about 1 us on a host core, also where there are hundreds of bands.  (Walking them one by one took up to 21 us, under a lock,
// and on every call once a map of 4096 grids was full.)  In a single row or column of tiles any height gives the same order.
inline int band_height(int tiles_m, int tiles_n, int rows, int cols, int xcds) {
    if (tiles_m == 1 || tiles_n == 1 || (int64_t)tiles_m * tiles_n > BAND_MAX_TILES) return std::min(tiles_m, 8);
    // place of (tiles_m, 1): behind the columns that fit beside fewer rows
    static constexpr auto place = [] {
        std::array<uint16_t, BAND_MAX_TILES + 2> p{};
        for (int m = 1; m <= BAND_MAX_TILES; ++m) p[m + 1] = (uint16_t)(p[m] + BAND_MAX_TILES / m);
        return p;
    }();
    static std::atomic<uint8_t> known[3][place[BAND_MAX_TILES + 1]];  // by whether tiles are square, wide or tall; 0: not yet
    std::atomic<uint8_t>& entry = known[rows == cols ? 0 : rows < cols ? 1 : 2][place[tiles_m] + tiles_n - 1];
    if (const int h = entry.load(std::memory_order_relaxed)) return h;
    int best = 1, best_cost = INT_MAX;
    for (int h = std::min(tiles_m, BAND_MAX_ROWS); h >= 1; --h) {
        const int cost = band_cost(tiles_m, tiles_n, rows, cols, xcds, h);
        if (cost < best_cost) {
            best_cost = cost;
            best = h;
        }
    }
    entry.store((uint8_t)best, std::memory_order_relaxed);
    return best;
}

}  // namespace axo
