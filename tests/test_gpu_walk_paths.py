"""GPU parity of both walks where the default call no longer takes them: the
node walk of the default method and of the ablations (tops of mixed depths,
chunks that straddle the capacity, overflow, interleaved queues, the
allocation-free call), the block walk's chunked output, eyes that are not
finite, the largest light sets, and calls of several launches."""
import numpy as np
import pytest

import synth
from _helpers import pair_keys_from_gpu, pair_keys_from_oracle, select_pairs_of_eyes

pytestmark = pytest.mark.gpu

TILE = synth.dither_tile(100)
FAR = np.float32(2.0 ** 31)      # scales distances exactly; s scales with its square


@pytest.fixture(scope="module")
def hrr():
    import paper_1907_12343_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(hrr):
    c = hrr.Context(TILE)
    yield c
    c.close()


def _dev(ctx, a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(ctx.torch_device)


def _oracle(orc, h, eyes, sel, s):
    return pair_keys_from_oracle(orc.accept_eyes(eyes, sel, 64, 0, TILE, h.sorted_lights(), s, lists=True), sel)


@pytest.mark.parametrize("split", ["radix", "pow2"])
@pytest.mark.parametrize("n_l,leaf", [(1, 1), (2, 1), (3, 1), (5, 8), (8, 8), (9, 8), (17, 4), (33, 1), (64, 1), (65, 1),
                                      (100, 3), (127, 1), (128, 3), (129, 1), (200, 3), (300, 8)])
def test_node_walk_tops_and_leaves(ctx, orc, n_l, leaf, split):
    """Hierarchies that are one leaf, and tops that mix leaves of every depth with
    nodes.  The node walk in its three ways: counting statistics, an ablation, and
    the default method with s beyond the block walk's range (the scene and s
    scaled by powers of two, so every probability stays the same)."""
    lights = synth.mixture_points(n_l, np.random.default_rng(700 + n_l).random((4, 3)), 710 + n_l)
    eyes = synth.uniform_points(300, 720 + n_l)
    eyes[7] = lights[0]
    sel = np.arange(300)
    h = ctx.build_hierarchy(lights, leaf_size=leaf, split=split)
    f = ctx.build_hierarchy(lights * FAR, leaf_size=leaf, split=split, box=[0.0] * 3 + [float(FAR)] * 3)
    want = _oracle(orc, h, eyes, sel, 0.02)
    e, e_far = _dev(ctx, eyes), _dev(ctx, eyes * FAR)
    for epw in (1, 2, 8):
        for opt in (dict(stats=True), dict(rmq_method=1)):
            pairs, n, _ = ctx.traverse_all(h, e, 0.02, 64, eyes_per_wave=epw, **opt)
            assert np.array_equal(pair_keys_from_gpu(pairs), want), (epw, opt)
        pairs, n, _ = ctx.traverse_all(f, e_far, float(np.float32(0.02)) * 2.0 ** 62, 64, eyes_per_wave=epw)
        assert np.array_equal(pair_keys_from_gpu(pairs), want), epw
    h.free()
    f.free()


@pytest.fixture(scope="module")
def tiny(orc):
    t = synth.tiny()
    t["sorted"] = t["lights"][orc.morton_order(t["lights"])]
    sel = np.arange(t["eyes"].shape[0])
    t["keys"] = pair_keys_from_oracle(orc.accept_eyes(t["eyes"], sel, t["width"], 0, t["tile"], t["sorted"], t["s"],
                                                      lists=True), sel)
    return t


@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("opt", [dict(rmq_method=1, eyes_per_wave=1), dict(rmq_method=4, eyes_per_wave=8), dict(stats=True)],
                         ids=str)
def test_node_walk_output_edges(ctx, hrr, tiny, opt, weights):
    """Capacities around the count: chunks straddle it and the pairs past it live in
    the slack area until the compaction; smaller ones hold distinct pairs and the
    call reports the true count."""
    import torch
    h = ctx.build_hierarchy(tiny["lights"])
    eyes = _dev(ctx, tiny["eyes"])
    total = tiny["keys"].size
    for cap in (total, total + 1, total + 77, total + 1000, 2 * total, total - 1, total // 2, total // 3, 1):
        buf = torch.full((cap, 2), -1, dtype=torch.int32, device=eyes.device)
        w = torch.full((cap,), -1.0, device=eyes.device) if weights else None
        if cap >= total:
            out = ctx.traverse(h, eyes, tiny["s"], tiny["width"], pairs=buf, weights=w, **opt)
            assert out[1] == total and np.array_equal(pair_keys_from_gpu(out[0]), tiny["keys"])
        else:
            with pytest.raises(hrr.OverflowResult) as ei:
                ctx.traverse(h, eyes, tiny["s"], tiny["width"], pairs=buf, weights=w, **opt)
            assert ei.value.count == total
            keys = pair_keys_from_gpu(buf)
            assert np.unique(keys).size == cap and np.isin(keys, tiny["keys"]).all()
        if weights:
            assert bool((w[:min(cap, total)] >= 1.0).all())
    h.free()


def test_node_walk_interleaved_queues(ctx, hrr):
    """2^19 tasks of several items: interleaved chunks of tasks, items that overflow
    and items with room to spare."""
    import torch
    n_e, n_l = 1 << 15, 700
    hs = [ctx.build_hierarchy(synth.uniform_points(n_l + k, 800 + k), leaf_size=1 + k % 3) for k in range(17)]
    eyes = [_dev(ctx, synth.uniform_points(n_e, 900 + k)) for k in range(17)]
    want = [pair_keys_from_gpu(ctx.traverse_all(h, e, 1e-4, 64)[0]) for h, e in zip(hs, eyes)]    # the block walk
    caps = [w.size for w in want]
    caps[5] //= 2
    caps[9] += 777
    offs = np.concatenate([[0], np.cumsum(caps)])
    buf = torch.full((int(offs[-1]), 2), -1, dtype=torch.int32, device=ctx.torch_device)
    items = [dict(h=h, eyes=e, s=1e-4, width=64, out_offset=int(offs[k]), out_capacity=caps[k])
             for k, (h, e) in enumerate(zip(hs, eyes))]
    with pytest.raises(hrr.OverflowResult) as ei:
        ctx.traverse_batched(items, buf, rmq_method=1, eyes_per_wave=1)
    assert ei.value.counts.tolist() == [w.size for w in want]
    for k, w in enumerate(want):
        keys = pair_keys_from_gpu(buf[offs[k]:offs[k] + min(caps[k], w.size)])
        assert np.unique(keys).size == keys.size and np.isin(keys, w).all() and keys.size == min(caps[k], w.size)
        hs[k].free()


@pytest.mark.parametrize("opt", [dict(eyes_per_wave=8, stack_entries=256, rmq_method=1), dict(rmq_method=4),
                                 dict(far=True), dict(far=True, eyes_per_wave=8, stack_entries=192)], ids=str)
def test_noalloc_node_walk(ctx, tiny, opt):
    """The allocation-free call's node walk (an ablation, or the default method with
    s beyond the block walk's range): spill stacks carved from its scratch."""
    import torch
    opt = dict(opt)
    scale = FAR if opt.pop("far", False) else np.float32(1.0)
    h = ctx.build_hierarchy(tiny["lights"] * scale, box=[0.0] * 3 + [float(scale)] * 3)
    eyes = _dev(ctx, tiny["eyes"] * scale)
    s = float(np.float32(tiny["s"])) * float(scale) ** 2
    n = tiny["keys"].size
    for cap in (n, n + 1000, n // 2, 0):
        buf = torch.full((max(cap, 1), 2), -1, dtype=torch.int32, device=eyes.device)
        res = torch.full((2,), -7, dtype=torch.int64, device=eyes.device)
        ctx.traverse_noalloc(h, eyes, s, tiny["width"], buf, res, capacity=cap, **opt)
        torch.cuda.synchronize()
        assert res.tolist() == [n, 0]
        keys = pair_keys_from_gpu(buf[:min(cap, n)])
        assert keys.size == min(cap, n) and np.unique(keys).size == keys.size and np.isin(keys, tiny["keys"]).all()
    h.free()


@pytest.mark.parametrize("weights", [False, True])
def test_block_walk_chunked_output_edges(ctx, hrr, weights):
    """More than 2^24 pairs (every pair of 4200 eyes and 4100 lights): chunks that
    straddle the capacity, the slack area and its end, alone and as one item of a
    batch beside others."""
    import torch
    n_e, n_l, s = 4200, 4100, 1e3
    h = ctx.build_hierarchy_device(_dev(ctx, synth.uniform_points(n_l, 31)))
    e = _dev(ctx, synth.uniform_points(n_e, 32))
    n = n_e * n_l

    def check(pairs, w, stored):
        key = (pairs[:, 0].to(torch.int64) * n_l + pairs[:, 1])
        assert key.numel() == stored and int(key.min()) >= 0 and int(key.max()) < n
        assert int(torch.bincount(key, minlength=n).max()) == 1
        if weights:
            assert bool((w[:stored] == 1.0).all())

    for cap in (n, n + 1, n + 77, n + 100003, n - 1, n - 12345, (1 << 24) + 1):
        buf = torch.full((cap, 2), -1, dtype=torch.int32, device=e.device)
        w = torch.full((cap,), -1.0, device=e.device) if weights else None
        if cap >= n:
            assert ctx.traverse(h, e, s, 64, pairs=buf, weights=w)[1] == n
        else:
            with pytest.raises(hrr.OverflowResult) as ei:
                ctx.traverse(h, e, s, 64, pairs=buf, weights=w)
            assert ei.value.count == n
        check(buf[:min(cap, n)], w, min(cap, n))
        res = torch.full((2,), -7, dtype=torch.int64, device=e.device)
        buf.fill_(-1)
        ctx.traverse_noalloc(h, e, s, 64, buf, res, weights=w)
        torch.cuda.synchronize()
        assert res.tolist() == [n, 0]
        check(buf[:min(cap, n)], w, min(cap, n))
    # a batch: its first item overflows, the others have room to spare
    g = ctx.build_hierarchy_device(_dev(ctx, synth.uniform_points(999, 33)))
    caps, offs = [n - 4321, 4200 * 999 + 555, 4200 * 999], [0, n, n + 4200 * 999 + 999]
    buf = torch.full((offs[2] + caps[2], 2), -1, dtype=torch.int32, device=e.device)
    w = torch.full((buf.shape[0],), -1.0, device=e.device) if weights else None
    items = [dict(h=q, eyes=e, s=s, width=64, out_offset=o, out_capacity=c) for q, o, c in zip((h, g, g), offs, caps)]
    with pytest.raises(hrr.OverflowResult) as ei:
        ctx.traverse_batched(items, buf, weights=w)
    assert ei.value.counts.tolist() == [n, 4200 * 999, 4200 * 999]
    check(buf[:caps[0]], w, caps[0])
    assert int(buf[caps[0]:n].max()) == -1                  # nothing past the slice
    for o in offs[1:]:
        part = buf[o:o + 4200 * 999]
        key = part[:, 0].to(torch.int64) * 999 + part[:, 1]
        assert int(torch.bincount(key, minlength=4200 * 999).min()) == 1
    h.free()
    g.free()


@pytest.mark.parametrize("n_l", [1, 40, 3001])
def test_eyes_that_are_not_finite(ctx, n_l):
    """NaN and infinite coordinates beside ordinary eyes: the block walk keeps the
    pairs of the node walk, in dense and in chunked output."""
    import torch
    eyes = synth.uniform_points(6001, 50 + n_l)
    for k, bad in enumerate((np.nan, np.inf, -np.inf, 3e38, -3e38)):
        eyes[3 + 7 * k, k % 3] = bad
        eyes[5 + 7 * k, :] = bad
    h = ctx.build_hierarchy(synth.uniform_points(n_l, 60 + n_l), leaf_size=2)
    e = _dev(ctx, eyes)
    for s in (1e-4, 0.5):
        ref, n, _ = ctx.traverse_all(h, e, s, 64, rmq_method=1)
        want = pair_keys_from_gpu(ref)
        for cap in (n, n + (1 << 25)):
            pairs, m, _ = ctx.traverse(h, e, s, 64, capacity=max(cap, 1))
            assert m == n and np.array_equal(pair_keys_from_gpu(pairs), want)
    h.free()


@pytest.mark.parametrize("n_l", [1 << 24, (1 << 24) + 1, (1 << 25) - 1])
def test_the_largest_light_sets(ctx, orc, n_l):
    """Light numbers and block numbers at the widths they are packed with."""
    import torch
    g = torch.Generator(device=ctx.torch_device).manual_seed(n_l)
    lights = torch.rand((n_l, 3), device=ctx.torch_device, generator=g)
    h = ctx.build_hierarchy_device(lights, leaf_size=8)
    eyes = synth.uniform_points(70, 77)
    order = h.sorted_lights()
    eyes[3], eyes[4], eyes[5] = order[0], order[-1], order[n_l // 2]
    del lights
    sel = np.array([0, 3, 4, 5, 63, 64, 69])
    out = orc.accept_eyes(eyes, sel, 64, 0, TILE, order, 1e-6, lists=True)
    want = pair_keys_from_oracle(out, sel)
    e = _dev(ctx, eyes)
    pairs, n, _ = ctx.traverse_all(h, e, 1e-6, 64)
    assert np.array_equal(select_pairs_of_eyes(pairs, sel), want)
    assert ctx.count(h, e, 1e-6, 64, rmq_method=1) == n
    h.free()


@pytest.mark.parametrize("n_l,n_e,cap", [(4099, 30000, 1 << 25), (1 << 17, 30000, 1 << 22)])
def test_lights_in_no_order(ctx, orc, n_l, n_e, cap):
    """Lights beside the unit cube that orders them: the default method's node walk,
    with chunked and with exact output."""
    lights = synth.uniform_points(n_l, 90) + np.float32(10.0)
    eyes = synth.uniform_points(n_e, 91) + np.float32(10.0)
    h = ctx.build_hierarchy_device(_dev(ctx, lights))
    sel = np.arange(0, n_e, 997)
    pairs, n, _ = ctx.traverse(h, _dev(ctx, eyes), 1e-6, 64, capacity=cap)
    assert np.array_equal(select_pairs_of_eyes(pairs, sel), _oracle(orc, h, eyes, sel, 1e-6))
    assert np.unique(pair_keys_from_gpu(pairs)).size == n
    h.free()


@pytest.mark.parametrize("method", [0, 1])
def test_more_items_than_one_launch(ctx, method):
    """1500 items of two shapes."""
    import torch
    small = ctx.build_hierarchy(synth.uniform_points(100, 1))
    large = ctx.build_hierarchy_device(_dev(ctx, synth.uniform_points(1 << 16, 2)))
    eyes = _dev(ctx, synth.uniform_points(20, 3))
    ref = {h: pair_keys_from_gpu(ctx.traverse_all(h, eyes, 1e-4, 64, rmq_method=1 - method)[0]) for h in (small, large)}
    hs = [small if k % 2 else large for k in range(1500)]
    items, at = [], 0
    for h in hs:
        items.append(dict(h=h, eyes=eyes, s=1e-4, width=64, out_offset=at, out_capacity=ref[h].size))
        at += ref[h].size
    buf = torch.full((at, 2), -1, dtype=torch.int32, device=eyes.device)
    counts, _ = ctx.traverse_batched(items, buf, rmq_method=method)
    for h, it, n in zip(hs, items, counts):
        assert int(n) == ref[h].size
    for it, h in list(zip(items, hs))[::251]:
        o = it["out_offset"]
        assert np.array_equal(pair_keys_from_gpu(buf[o:o + ref[h].size]), ref[h])
    small.free()
    large.free()
