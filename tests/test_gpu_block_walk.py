"""GPU parity of the block walk (the default traversal) at the edges of its
block tree: light counts around the leaf blocks (8 or 16 lights, by the
parity of the tree's depth) and around each level's four children, with a
ragged last task, against the oracle's all-pairs set."""
import numpy as np
import pytest

import synth
from _helpers import pair_keys_from_gpu, pair_keys_from_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1907_12343_amd as hrr
    c = hrr.Context(synth.dither_tile(100))
    yield c
    c.close()


@pytest.mark.parametrize("n_l", [1, 2, 7, 8, 9, 31, 32, 33, 63, 64, 65, 127, 129, 255, 257, 1023, 1024, 1025, 4097])
def test_block_tree_edges(ctx, orc, n_l):
    import torch
    # enough eyes for the block walk (work 2^21), an odd number
    n_e = int(2 ** 21 / n_l ** 0.6) + 13
    lights = synth.mixture_points(n_l, np.random.default_rng(40 + n_l).random((4, 3)), 50 + n_l)
    eyes = synth.uniform_points(n_e, 60 + n_l)
    eyes[5] = lights[0]
    s = 0.5 / n_l                    # near and far blocks, saturated and sparse
    tile = synth.dither_tile(100)
    sel = np.unique(np.concatenate([np.arange(0, n_e, max(1, n_e // 6000)), [5, n_e - 1]]))
    out = orc.accept_eyes(eyes, sel, 64, 0, tile, lights[orc.morton_order(lights)], s, lists=True)
    want = pair_keys_from_oracle(out, sel)
    h = ctx.build_hierarchy(lights, leaf_size=3)
    e = torch.from_numpy(eyes).to(ctx.torch_device)
    pairs, n, _ = ctx.traverse_all(h, e, s, 64)
    assert ctx.traverse_all(h, e, s, 64, rmq_method=4)[1] == n      # the node walk's count
    got = pair_keys_from_gpu(pairs)
    assert np.unique(got).size == n
    assert np.array_equal(got[np.isin(got >> np.uint64(32), sel.astype(np.uint64))], want)
    h.free()
