"""The spread of a light set's block tree (hrr_types.hpp): small where the sort
order follows the lights' places, large where it does not."""
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1907_12343_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "hrr_build.hpp"
#include "hrr_devbuild.hpp"
#include "hrr_types.hpp"
using namespace hrr;
// stdin: n lights (3 floats each); prints the spread over all smallest blocks
int main(int, char** argv) {
    const uint32_t n = (uint32_t)atoi(argv[1]);
    std::vector<float> xyz(3 * (size_t)n);
    if (fread(xyz.data(), 12, n, stdin) != n) return 1;
    HostHierarchy H;
    if (!build_hierarchy(xyz.data(), n, 8, false, nullptr, H)) return 1;
    const uint32_t small = 1u << block_leaf_log(block_tree_log(n));
    double sum = 0.0;
    for (uint32_t first = 0; first < n; first += small) {
        const float* p = &H.sorted_xyz[3 * (size_t)first];
        float lo[3] = {p[0], p[1], p[2]}, hi[3] = {p[0], p[1], p[2]};
        for (uint32_t i = first; i < n && i < first + small; ++i)
            for (int k = 0; k < 3; ++k) {
                lo[k] = min_first(lo[k], H.sorted_xyz[3 * (size_t)i + k]);
                hi[k] = max_first(hi[k], H.sorted_xyz[3 * (size_t)i + k]);
            }
        sum += block_share(lo, hi, H.box, H.box + 3);
    }
    printf("%.6f\n", sum);
    return 0;
}
"""


@pytest.fixture(scope="module")
def spread(tmp_path_factory):
    d = tmp_path_factory.mktemp("block_spread")
    (d / "t.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(d / "t.cpp"),
                    os.path.join(CSRC, "hrr_build.cpp"), "-o", str(d / "t")], check=True)

    def run(points):
        p = np.ascontiguousarray(points, np.float32)
        r = subprocess.run([str(d / "t"), str(len(p))], input=p.tobytes(), capture_output=True)
        assert r.returncode == 0
        return float(r.stdout)
    return run


@pytest.mark.parametrize("n", [1000, 30011, 1 << 17, (1 << 17) + 1])
def test_spread(spread, n):
    u = synth.uniform_points(n, 7)
    m = synth.mixture_points(n, synth.mixture_centers(3), 8)
    # in order: no threshold of the walks' choice (128 and more) is near
    assert 0.0 < spread(m) < 16.0 and 0.0 < spread(u) < 16.0
    flat = u.copy()
    flat[:, 2] = 0.25
    for shift in (0.0, 10.0):
        assert spread(flat + shift) == 0.0               # a plane
    assert spread(np.full((n, 3), 0.5, np.float32)) == 0.0
    # beside the unit cube that orders them every code is one: a good part of all blocks
    blocks = -(-n // 16)
    assert spread(u + 10.0) > 0.4 * blocks
