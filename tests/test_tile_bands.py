"""Band heights of the tile order of weight gradients (csrc/tile_bands.hpp), compiled for the host: for every grid of tiles the choice of a walk over
all tiles, and a search whose time does not grow with the number of bands and which each grid needs once."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2305_13525_amd", "csrc")
SOURCE = r"""
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <thread>
#include <vector>
#include "tile_bands.hpp"
using namespace axo;

// every tile by itself, in the order of tile_of_index
static int walk(int tm, int tn, int rows, int cols, int h) {
    const int n = tm * tn;
    int cost = 0;
    for (int x = 0, t = 0; x < 8; ++x) {
        const int end = t + n / 8 + (x < n % 8);
        std::set<int> seen_rows, seen_cols;
        int band = -1;
        for (; t < end; ++t) {
            const int b = t / (h * tn), height = std::min(h, tm - b * h), in_band = t - b * h * tn;
            if (b != band) {
                cost += (int)seen_rows.size() * rows + (int)seen_cols.size() * cols;
                seen_rows.clear(), seen_cols.clear(), band = b;
            }
            seen_rows.insert(b * h + in_band % height);
            seen_cols.insert(in_band / height);
        }
        cost += (int)seen_rows.size() * rows + (int)seen_cols.size() * cols;
    }
    return cost;
}
static int fail(const char* what, int a, int b, int c) { return std::printf("%s: %d %d %d\n", what, a, b, c), 1; }
template <typename F>
static double least(F f) {
    double t = 1e30;
    for (int i = 0; i < 7; ++i) {
        const auto t0 = std::chrono::steady_clock::now();
        f();
        t = std::min(t, std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
    }
    return t;
}

int main() {
    const int shapes[3][2] = {{64, 64}, {64, 128}, {128, 64}};
    auto all = [&](auto f) {
        for (auto& s : shapes)
            for (int m = 1; m <= 512; ++m)
                for (int n = 1; m * n <= 512; ++n) f(m, n, s[0], s[1]);
    };
    volatile int sink = 0;
    const auto t0 = std::chrono::steady_clock::now();
    all([&](int m, int n, int r, int c) { sink = sink + band_height(m, n, r, c, 8); });
    const double first = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    const double again = least([&] { all([&](int m, int n, int r, int c) { sink = sink + band_height(m, n, r, c, 8); }); });
    if (5 * again > first) return fail("searched again, ns", (int)(first * 1e9), (int)(again * 1e9), 0);
    auto search = [&](int m, int n) {
        return least([&] { for (int i = 0; i < 300; ++i) for (int h = 16; h >= 1; --h) sink = sink + band_cost(m, n, 64, 64, 8, std::min(h, m)); });
    };
    const double square = search(16, 16);
    for (auto& g : {std::pair<int, int>{512, 1}, {256, 2}, {128, 4}, {24, 21}})
        if (search(g.first, g.second) > 4 * square) return fail("a long search", g.first, g.second, 0);
    int bad = 0;
    all([&](int m, int n, int r, int c) {
        const int h = band_height(m, n, r, c, 8);
        if (m == 1 || n == 1) {  // any height gives the same order
            bad |= h != std::min(m, 8);
            return;
        }
        int best = 0, cost = 1 << 30;
        for (int i = std::min(m, 16); i >= 1; --i) {
            const int w = walk(m, n, r, c, i);
            if (w != band_cost(m, n, r, c, 8, i)) bad = fail("cost", m, n, i);
            if (w < cost) cost = w, best = i;
        }
        if (h != best) bad = fail("height", m, n, h);
    });
    if (band_height(513, 1, 64, 64, 8) != 8 || band_height(3, 200, 64, 64, 8) != 3 || band_height(1 << 20, 1 << 20, 64, 64, 8) != 8) return 1;
    std::vector<std::thread> threads;
    for (int i = 0; i < 4; ++i) threads.emplace_back([&] { all([&](int m, int n, int r, int c) { if (band_height(m, n, r, c, 8) < 1) std::abort(); }); });
    for (auto& t : threads) t.join();
    return bad;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")
def test_heights_are_those_of_a_walk_and_searched_once(tmp_path):
    (tmp_path / "bands.cpp").write_text(SOURCE)
    exe = tmp_path / "bands"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-pthread", "-I", CSRC, str(tmp_path / "bands.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
