"""Host rules of the block walk's launches (hrr_layout.hpp, hrr_types.hpp): the
task split, the output's shape and the lights' second order."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1907_12343_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <vector>
#include "hrr_layout.hpp"
using namespace hrr;
uint32_t bit_reverse(uint32_t x) {
    uint32_t r = 0;
    for (int b = 0; b < 32; ++b) r |= (x >> b & 1u) << (31 - b);
    return r;
}
#define CHECK(x) do { if (!(x)) { printf("line %d: %s (n %u)\n", __LINE__, #x, n); return 1; } } while (0)
int main(int, char** argv) {
    uint32_t n = 0;
    sscanf(argv[1], "%u", &n);
    const uint32_t S = block_tree_log(n), leaf = block_leaf_log(S), small = 1u << leaf;
    CHECK((1ull << S) >= n && (S - leaf) % 2 == 0 && S > leaf);
    // every light has a place of its own inside its smallest block, and the
    // place is the one the walk derives from the light's reversed index
    const uint32_t padded = block_tree_lights(n);
    CHECK(padded >= n && padded - n < small && padded % small == 0);
    CHECK(padded - 1u == ((n - 1u) | (small - 1u)));
    CHECK(block_tree_floats(n) == block_lights_at(n) + 4ull * padded);
    std::vector<bool> taken(padded, false);
    for (uint32_t i = 0; i < n; ++i) {
        const uint32_t built = (i & ~(small - 1u)) + (bit_reverse(i & (small - 1u)) >> (32u - leaf));
        const uint32_t walked = (i & (0u - small)) | bit_reverse(i) >> (32u - leaf);
        CHECK(built == walked && built < padded && !taken[built]);
        taken[built] = true;
    }
    // a task holds at most a wave's 64 eye slots; an eye is cut into 1, 4 or 16
    // blocks, all of them above the smallest ones; dense launches only
    for (double eyes = 1; eyes < 1e8; eyes *= 7)
        for (uint64_t waves : {1ull, 64ull, 8192ull})
            for (int dense = 0; dense < 2; ++dense) {
                uint32_t shift = 99, sub = 99;
                block_task_split(n, eyes * eye_cost(n), waves, dense != 0, &shift, &sub);
                CHECK(shift <= 6u && (sub == 0 || sub == 2 || sub == 4));
                CHECK(sub == 0 || (dense && shift == 0 && S - leaf >= sub + 2u));
                const uint32_t cs = block_chunk_shift((uint64_t)eyes * n, waves);
                CHECK(cs >= kMinChunkShift && cs <= kMaxChunkShift);
            }
    CHECK(block_walk_dense(1, 1e30) && block_walk_dense(1u << 24, 0) && !block_walk_dense((1u << 24) + 1u, 0));
    CHECK(block_walk_dense(0, 1.0) && !block_walk_dense(0, 268435456.0));
    CHECK(block_walk_takes(1e-4f) && block_walk_takes(0x1p-60f) && block_walk_takes(0x1p60f));
    CHECK(!block_walk_takes(0x1p-61f) && !block_walk_takes(0x1p61f) && !block_walk_takes(-1.0f));
    return 0;
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    d = tmp_path_factory.mktemp("block_layout")
    (d / "t.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t")], check=True)
    return str(d / "t")


@pytest.mark.parametrize("n", [1, 7, 8, 9, 31, 32, 33, 63, 64, 65, 100003, 1 << 20, (1 << 20) + 1])
def test_block_layout(harness, n):
    r = subprocess.run([harness, str(n)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
