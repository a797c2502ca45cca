"""The selection's bins of entropies (csrc/tahq_bins.hpp), compiled for the host and run over every bin of many scales."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <vector>

#define __device__
#define __forceinline__ inline
static uint32_t __float_as_uint(float f) { uint32_t u; std::memcpy(&u, &f, 4); return u; }
static float __uint_as_float(uint32_t u) { float f; std::memcpy(&f, &u, 4); return f; }
// median of three; with a NaN among them the smaller of the other two
static float med3(float a, float b, float c)
{
    if (std::isnan(a)) return std::min(b, c);
    return std::max(std::min(a, b), std::min(std::max(a, b), c));
}
#define __builtin_amdgcn_fmed3f med3
#include "tahq_bins.hpp"
using namespace tahq;

static void check(bool ok, const char *what, double x, unsigned b)
{
    if (!ok) { std::printf("%s: %.9g, bin %u\n", what, x, b); std::exit(1); }
}

int main()
{
    std::vector<double> widths;
    for (unsigned a = 8; a <= 8192; a += 8) widths.push_back(a);
    for (unsigned s = 14; s < 32; ++s) { widths.push_back(std::ldexp(1.0, s)); widths.push_back(std::ldexp(1.0, s) - 8.0); }
    for (double a : widths) {
        const float scale = (float)((double)kLinBins / std::log(a));
        for (uint32_t b = 1; b < kLinBins; ++b) {
            const int e = linear_bin_edge(b, scale);
            check(linear_bin(__uint_as_float(e), scale) == b, "an edge lies in its bin", a, b);
            check(linear_bin(__uint_as_float(e - 1), scale) == b - 1, "the float below it in the one below", a, b);
        }
        // beyond the last bin: the search ends, at the last bin's edge
        for (uint32_t b : {kLinBins, kLinBins + 1, 2 * kLinBins, 1u << 20, 1u << 31, 0xffffffffu})
            check(linear_bin_edge(b, scale) == linear_bin_edge(kLinBins - 1, scale), "no such bin", a, b);
    }
    for (float scale : {0.0f, -1.0f, INFINITY, NAN, 1e-30f, 1e30f})          // none occurs: the search ends all the same
        for (uint32_t b : {0u, 1u, 5u, kLinBins - 1, 0xffffffffu}) (void)linear_bin_edge(b, scale);

    // bins and sub-bins never decrease in the order of the keys
    const float scale = (float)((double)kLinBins / std::log(64.0));
    std::vector<uint32_t> v = {0x7f800000u, 0xff800000u, 0x7fc00000u, 0xffc00000u, 0x7fffffffu, 0xffffffffu, 0u, 1u, 0x80000001u};
    uint32_t state = 1;
    for (int i = 0; i < 400000; ++i) {
        state = state * 1664525u + 1013904223u;
        v.push_back(i % 4 == 0 ? state : __float_as_uint(4.2f * (state >> 8) / 16777216.0f));
    }
    std::sort(v.begin(), v.end(), [](uint32_t x, uint32_t y) { return order_key(__uint_as_float(x)) < order_key(__uint_as_float(y)); });
    for (size_t i = 1; i < v.size(); ++i) {
        const float p = __uint_as_float(v[i - 1]), q = __uint_as_float(v[i]);
        const uint32_t bp = linear_bin(p, scale), bq = linear_bin(q, scale);
        check(bp <= bq && bq < kLinBins, "bins in key order", q, bq);
        if (bp == bq) check(linear_sub_bin(p, scale, bp) <= linear_sub_bin(q, scale, bq), "sub-bins in key order", q, bq);
        if (bp == bq) check(crowd_sub_bin(p, scale, bp) <= crowd_sub_bin(q, scale, bq) && crowd_sub_bin(q, scale, bq) < kSubBins, "a crowd's sub-bins in key order", q, bq);
        if (bq == 0 && v[i] != 0x80000000u) check((crowd_sub_bin(q, scale, 0) == 1) == (v[i] == 0), "all-zero tiles by themselves", q, bq);
        check(__float_as_uint(key_to_float(order_key(q))) == v[i], "a key turns back into its entropy", q, bq);
    }
    return 0;
}
"""


def test_bins_of_entropies_on_the_host(tmp_path):
    source, binary = tmp_path / "bins.cpp", tmp_path / "bins"
    source.write_text(HARNESS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-Wno-unknown-pragmas",
                    "-I", os.path.join(ROOT, "paper_2506_01352_amd", "csrc"), str(source), "-o", str(binary)], check=True)
    try:
        done = subprocess.run([str(binary)], timeout=60, capture_output=True, text=True)
    except subprocess.TimeoutExpired:
        pytest.fail("the search for a bin's edge does not end")
    assert done.returncode == 0, done.stdout
