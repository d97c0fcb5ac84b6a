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
    # an odd number of eyes, more for small light sets
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


@pytest.mark.parametrize("n_e", [1, 3, 64, 65, 1000])
@pytest.mark.parametrize("n_l", [447, 448, 449, 512, 513, 4096 + 1])
def test_dense_output_edges(ctx, n_l, n_e):
    """Every pair accepted (s beyond every squared distance): outputs around
    the 512 staged pairs of a wave, one eye cut into the tree's first blocks,
    counting calls and outputs smaller than the count."""
    import paper_1907_12343_amd as hrr
    import torch
    lights = synth.uniform_points(n_l, 70 + n_l)
    e = torch.from_numpy(synth.uniform_points(n_e, 80 + n_e)).to(ctx.torch_device)
    h = ctx.build_hierarchy(lights)
    n = ctx.count(h, e, 1e3, 64)
    assert n == n_e * n_l
    pairs, m, _, w = ctx.traverse(h, e, 1e3, 64, capacity=n + 7, with_weights=True)
    assert m == n
    assert np.array_equal(pair_keys_from_gpu(pairs),
                          (np.arange(n_e, dtype=np.uint64)[:, None] << np.uint64(32)
                           | np.arange(n_l, dtype=np.uint64)[None, :]).ravel())
    assert bool((w == 1.0).all())
    cap = n - n // 3
    buf = torch.full((cap, 2), -1, dtype=torch.int32, device=e.device)
    with pytest.raises(hrr.OverflowResult) as ei:
        ctx.traverse(h, e, 1e3, 64, pairs=buf)
    assert ei.value.count == n
    keys = pair_keys_from_gpu(buf)
    assert np.unique(keys).size == cap and int(buf.min()) >= 0
    h.free()


def test_dense_output_of_many_small_items(ctx):
    """Items of a few eyes: the waves of a block hold pairs of different items
    when they end, and every item's pairs are dense in its own slice."""
    import torch
    rng = np.random.default_rng(9)
    items, want, at = [], [], 0
    for k in range(23):
        n_l, n_e = int(rng.integers(1, 3000)), int(rng.integers(0, 70))
        lights = synth.uniform_points(n_l, 300 + k)
        h = ctx.build_hierarchy(lights, leaf_size=1 + k % 8)
        e = torch.from_numpy(synth.uniform_points(n_e, 400 + k).reshape(-1, 3)).to(ctx.torch_device)
        ref = pair_keys_from_gpu(ctx.traverse_all(h, e, 0.02, 64, rmq_method=1)[0])   # the node walk
        items.append(dict(h=h, eyes=e, s=0.02, width=64, out_offset=at, out_capacity=ref.size + 5))
        want.append(ref)
        at += ref.size + 5
    pairs = torch.empty((at, 2), dtype=torch.int32, device=ctx.torch_device)
    counts, _ = ctx.traverse_batched(items, pairs)
    for it, ref, n in zip(items, want, counts):
        assert int(n) == ref.size
        o = it["out_offset"]
        assert np.array_equal(pair_keys_from_gpu(pairs[o:o + int(n)]), ref)
        it["h"].free()
