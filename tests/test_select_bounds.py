"""The bisections that cut a full candidate buffer down (csrc/knnf_select.h), on the CPU
under UndefinedBehaviorSanitizer: the kept candidates hold the K smallest in (distance,
index) order, no more of them than asked for, after at most as many counts as there are
bits, over distance bits and indices up to the ends of their ranges.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = r'''
#define __device__
#define __forceinline__ inline
#include "knnf_select.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>
using namespace knnf;
struct C { uint32_t d, i; };
static int calls;
// The cut as the kernels make it; returns the number kept, or -1 for a lost neighbour.
static int cut(const std::vector<C>& v, uint32_t bound, int K, int few, int room) {
    auto count = [&](uint32_t t) { ++calls; int c = 0; for (auto& x : v) c += x.d <= t; return c; };
    int n = 2 * room;
    uint32_t hi = cut_distance(bound, K, few, n, count);
    std::vector<C> keep;
    uint32_t ih = 0xffffffffu;
    if (n > room) {
        if (hi == 1 && count(0u) >= K) hi = 0;
        n = 0;
        for (auto& x : v) n += x.d <= hi;
        if (n > room)
            ih = cut_index(K, few, n, [&](uint32_t i) {
                ++calls; int c = 0; for (auto& x : v) c += x.d < hi || (x.d == hi && x.i < i); return c; });
    }
    for (auto& x : v) if (x.d < hi || (x.d == hi && x.i < ih)) keep.push_back(x);
    if ((int)keep.size() != n || n > room || n < K) return -2;
    auto less = [](const C& a, const C& b) { return a.d != b.d ? a.d < b.d : a.i < b.i; };
    std::vector<C> s = v;
    std::sort(s.begin(), s.end(), less);
    std::sort(keep.begin(), keep.end(), less);
    for (int k = 0; k < K; ++k) if (keep[k].d != s[k].d || keep[k].i != s[k].i) return -1;
    return n;
}
int main() {
    std::mt19937 g(3);
    const uint32_t inf = 0x7f800000u;
    int worst = 0;
    for (int t = 0; t < 40000; ++t) {
        const int room = t % 3 ? 64 : 128;
        const int K = 1 + (int)(g() % 64), total = room + 1 + (int)(g() % 64), few = K + (int)(g() % (room - K + 1));
        const int kind = t % 7;
        std::vector<C> v;
        std::set<uint32_t> used;
        for (int k = 0; k < total; ++k) {
            uint32_t d = kind == 0 ? g() % (inf + 1) : kind == 1 ? 0 : kind == 2 ? g() % 3 : kind == 3 ? inf - g() % 2
                       : kind == 4 ? inf : kind == 5 ? 0x3f000000u + g() % 1000 : 1;
            uint32_t i;
            do i = t % 2 ? g() % 0x7fffffffu : t % 5 ? 0x7ffffffeu - g() % 300 : g() % 300; while (!used.insert(i).second);
            v.push_back({d, i});
        }
        uint32_t bound = 0;
        for (auto& x : v) bound = std::max(bound, x.d);
        calls = 0;
        const int n = cut(v, bound, K, few, room);
        if (n < 0) { std::printf("FAIL %d: case %d K %d few %d\n", n, t, K, few); return 1; }
        worst = std::max(worst, calls);
    }
    std::printf("ok %d\n", worst);
    return worst > 70;
}
'''


def test_cuts_hold_the_nearest(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    src, exe = str(tmp_path / "cut.cpp"), str(tmp_path / "cut")
    with open(src, "w") as f:
        f.write(CODE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_2404_10631_amd", "csrc"), src, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
