"""Rank steps of the output compaction (prefix_advance, hrr_compact.hpp): the rank
of a linear walk, in a number of reads that does not grow with the empty entries
between two ranks."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1907_12343_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "hrr_compact.hpp"
using namespace hrr;
struct Counted {
    const std::vector<unsigned long long>& v;
    mutable unsigned long reads = 0;
    unsigned long long operator[](unsigned long long i) const {
        if (i >= v.size()) abort();
        ++reads;
        return v[i];
    }
};
int main(int, char** argv) {
    const unsigned long long n = strtoull(argv[1], 0, 10);
    const int empty = atoi(argv[2]);   // percent of the entries
    std::mt19937_64 rng(n * 100 + empty);
    std::vector<unsigned long long> prefix(n + 1, 0);
    for (unsigned long long q = 0; q < n; ++q)
        prefix[q + 1] = prefix[q] + ((int)(rng() % 100) < empty ? 0 : 1 + rng() % 7);
    if (!prefix[n]) prefix[n] = 3;
    const unsigned long long total = prefix[n];
    for (unsigned long long stride : {1ull, 64ull, 1000ull}) {
        unsigned long long q = prefix_rank(prefix.data(), n, 0);
        for (unsigned long long e = 0; e < total; e += stride) {
            unsigned long long want = q;
            while (prefix[want + 1] <= e) ++want;
            const Counted c{prefix};
            const unsigned long long got = prefix_advance(c, n, q, e);
            if (got != want || want != prefix_rank(prefix.data(), n, e)) return printf("rank %llu %llu\n", got, want), 1;
            unsigned long bits = 0;
            while ((want - q) >> bits) ++bits;
            if (c.reads > 2 * bits + 2) return printf("%lu reads over %llu entries\n", c.reads, want - q), 1;
            q = got;
        }
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    d = tmp_path_factory.mktemp("compact_advance")
    (d / "t.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t")], check=True)
    return str(d / "t")


@pytest.mark.parametrize("empty", [0, 30, 95, 100])
@pytest.mark.parametrize("n", [1, 2, 3, 64, 1000, 8191, 16385])
def test_prefix_advance(harness, n, empty):
    r = subprocess.run([harness, str(n), str(empty)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
