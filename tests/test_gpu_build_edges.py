"""GPU hierarchy build around the sizes where its sort changes tiles and scans,
and on blocks of memory that freed hierarchies left behind: record for record
equal to the host build."""
import numpy as np
import pytest

import synth
from test_gpu_build import _same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1907_12343_amd as hrr
    c = hrr.Context(synth.dither_tile(100))
    yield c
    c.close()


# 2 rounds of 256 keys a tile below 2^16 lights, 4 below 2^18, then 8; fused
# offsets up to 48 tiles (24,576 lights in tiles of 512), beyond them each
# digit's tile counts are scanned 2048 at a time (2^22 lights in tiles of 2048)
@pytest.mark.parametrize("n", [511, 512, 513, 24576, 24577, 65535, 65536, 131072, 131073, 262143, 262144, 262145,
                               (1 << 22) + 1])
def test_sort_tiles(ctx, n):
    import torch
    lights = synth.mixture_points(n, synth.mixture_centers(n), n + 1)
    lights[n // 3: n // 3 + 300] = lights[n // 3]          # a run of equal codes
    lights = np.ascontiguousarray(lights)
    split = "pow2" if n & 1 else "radix"
    hh = ctx.build_hierarchy(lights, leaf_size=1 + n % 3, split=split)
    hd = ctx.build_hierarchy_device(torch.from_numpy(lights).to(ctx.torch_device), leaf_size=1 + n % 3, split=split)
    _same(hh, hd)
    hh.free()
    hd.free()


def test_rebuilt_hierarchies_share_no_memory(ctx):
    """Hierarchies freed and rebuilt in turn, two alive at a time: each keeps its
    own records while the other's memory is reused."""
    import torch
    alive, want = [], []
    for k in range(12):
        n = 20000 + 37 * (k % 4)
        lights = torch.from_numpy(synth.uniform_points(n, 500 + k)).to(ctx.torch_device)
        h = ctx.build_hierarchy_device(lights, split="radix" if k % 2 else "pow2")
        alive.append(h)
        want.append((h.permutation(), h.records().tobytes()))
        if len(alive) > 2:
            old, (perm, rec) = alive.pop(0), want.pop(0)
            assert np.array_equal(old.permutation(), perm) and old.records().tobytes() == rec
            old.free()
    for h, (perm, rec) in zip(alive, want):
        assert np.array_equal(h.permutation(), perm) and h.records().tobytes() == rec
        h.free()
