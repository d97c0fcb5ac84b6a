"""What the host side of a call launches and refuses, on a replaced HIP runtime."""
import re

import numpy as np
import pytest

import paper_1907_12343_amd as hrr
from _host_runtime import HostContext, build


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return build(tmp_path_factory.mktemp("host_launches"))


@pytest.fixture
def ctx(lib):
    c = HostContext(lib)
    yield c
    c.close()


def test_more_items_than_a_launch_holds(ctx):
    """A batched call of more than 1024 items runs when no shape (eyes per wave of
    an item's own hierarchy) has more than 1024 of them, one launch per shape,
    and is refused otherwise."""
    small, large = ctx.hierarchy(100), ctx.hierarchy(1 << 16)      # 8 and 4 eyes per wave
    for method in (0, 1):
        for n_s, n_l, ok in ((600, 600, True), (1024, 1024, True), (1025, 0, False), (1025, 3, False), (3, 1025, False)):
            st, counts = ctx.batched([(small, 7, 1e-4, 0)] * n_s + [(large, 5, 1e-4, 0)] * n_l, rmq_method=method)
            launches = [int(re.search(r"items=(\d+)", x).group(1)) for x in ctx.log() if "items=" in x]
            if ok:
                assert st == hrr.HRR_E_OVERFLOW                     # a counting call: no room for the pairs found
                assert launches == [n_l, n_s] and counts.tolist() == [7] * n_s + [5] * n_l
            else:
                assert st == hrr.HRR_E_INVALID and launches == []
        # a fixed shape, or one shape over both walks, is one launch
        assert ctx.batched([(small, 7, 1e-4, 0)] * 600 + [(large, 5, 1e-4, 0)] * 600, eyes_per_wave=4,
                           rmq_method=method)[0] == hrr.HRR_E_INVALID
        assert ctx.batched([(small, 7, 1e-4, 0)] * 600 + [(small, 5, 1e-30, 0)] * 600, rmq_method=method)[0] == \
            hrr.HRR_E_INVALID
        assert ctx.log() == []
    # up to 1024 items the default method is one launch
    st, _ = ctx.batched([(small, 7, 1e-4, 0)] * 512 + [(large, 5, 1e-4, 0)] * 512)
    assert [x.split()[0] for x in ctx.log()] == ["blocks"]
    ctx.free(small)
    ctx.free(large)


SHAPES = [(1, 192), (1, 256), (1, 512)] + [(e, c) for e in (2, 4, 8) for c in (512, 256, 1024)]


def test_autotuner_times_the_walk_whose_shape_it_chooses(ctx):
    """Every probe of both autotuners is a launch of the node walk in the shape
    that is tried (the block walk, which has no shape, takes no part)."""
    import ctypes
    hs = [ctx.hierarchy(5000, leaf=leaf) for leaf in (1, 4)]
    ctx.log()
    E, best = ctx.eyes(3000), hrr.HrrTuneResult()
    arr = (ctypes.c_void_p * 2)(*hs)
    assert ctx.lib.hrr_autotune(ctx.handle, arr, 2, ctypes.byref(E), 1e-4, 1000, ctypes.byref(best), None) == hrr.HRR_OK
    lines = [x for x in ctx.log() if "tasks=" in x]
    shapes = [tuple(int(v) for v in re.search(r"epw=(\d+) stack=(\d+)", x).groups()) for x in lines]
    per_leaf = [(1, 192)] + [q for q in SHAPES for _ in range(2)]     # a counting call, then two runs a shape
    assert shapes == per_leaf * 2 and all(x.startswith("nodes") and "method=0" in x for x in lines)
    items = (hrr.HrrWorkItem * 4)()
    for k in range(4):
        items[k] = hrr.HrrWorkItem(hs[k // 2], ctx.eyes(700 + 100 * (k % 2)), 1e-4, 0, 0, 0)
    assert ctx.lib.hrr_autotune_batched(ctx.handle, items, 2, 2, ctypes.byref(best), None) == hrr.HRR_OK
    lines = [x for x in ctx.log() if "tasks=" in x]
    shapes = [tuple(int(v) for v in re.search(r"epw=(\d+) stack=(\d+)", x).groups()) for x in lines]
    assert shapes == per_leaf * 2 and all(x.startswith("nodes") and "items=2" in x for x in lines)
    for h in hs:
        ctx.free(h)


@pytest.mark.parametrize("epw", [0, 1])
def test_a_bad_item_is_refused_before_anything_runs(ctx, epw):
    """One bad item among good ones: the call names it by its place in the call,
    and no item is launched (the output stays as it was)."""
    h, other = ctx.hierarchy(5000), HostContext(ctx.lib)
    foreign = other.hierarchy(10)
    good = (h, 7, 1e-4, 100)
    for bad, text in (((h, 7, float("nan"), 100), "s must be finite"), ((h, 7, 0.0, 100), "s must be finite"),
                      ((None, 7, 1e-4, 100), "null hierarchy"), ((foreign, 7, 1e-4, 100), "another context")):
        st, counts = ctx.batched([good, good, bad, (h, 7, 1e-30, 100)], eyes_per_wave=epw)
        assert st == hrr.HRR_E_INVALID and ctx.error().startswith("item 2: ") and text in ctx.error()
        assert [x for x in ctx.log() if "tasks=" in x] == [] and not counts.any()
    assert ctx.batched([good, good, (h, 7, 1e-30, 100)], eyes_per_wave=epw)[0] == hrr.HRR_OK
    assert [x.split()[0] for x in ctx.log() if "tasks=" in x] == ["blocks", "nodes"]
    other.free(foreign)
    other.close()
    ctx.free(h)


def _fields(line):
    return {k: int(v) for k, v in re.findall(r"(\w+)=(\d+)", line)}


@pytest.mark.parametrize("n_lights", [64, 4099, 16387, 262147])
@pytest.mark.parametrize("n_eyes", [1, 30, 300, 3000])
def test_a_large_buffer_does_not_idle_the_gpu(ctx, n_lights, n_eyes):
    """Few eyes into a buffer far larger than their pairs: the output is dense
    where the eyes have at most 2^24 lights in all, and a chunked launch makes a
    hundred tasks or one per eye.  Allocation-free calls follow the same rule."""
    h = ctx.hierarchy(n_lights, leaf=8)
    ctx.log()
    assert ctx.traverse(h, n_eyes, 1 << 26) == hrr.HRR_OK
    assert ctx.noalloc(h, n_eyes, 1 << 26) == hrr.HRR_OK
    lines = [_fields(x) for x in ctx.log() if x.startswith("blocks")]
    assert len(lines) == 2
    for f in lines:
        assert f["dense"] == (n_eyes * n_lights <= 1 << 24)
        assert f["tasks"] >= min(n_eyes, 100)
    ctx.free(h)


@pytest.mark.parametrize("device", [False, True])
def test_scattered_lights_take_the_node_walk(ctx, device):
    """Lights whose order says little about their place: the node walk, where the
    block walk is the slower one (node_walk_scattered)."""
    cases = [  # spread, lights, eyes, buffer, node walk
        (3.0, 1 << 18, 30000, 1 << 26, False), (3.0, 1 << 18, 30000, 1 << 20, False),
        (255.0, 1 << 18, 30000, 1 << 26, False), (256.0, 1 << 18, 30000, 1 << 26, True),
        (31.0, 4096, 30000, 1 << 26, False), (32.0, 4096, 30000, 1 << 26, True), (32.0, 4096, 3000, 1 << 26, False),
        (32.0, 4095, 30000, 1 << 26, False), (2047.0, 1 << 18, 1 << 17, 1 << 26, False),
        (2048.0, 1 << 18, 1 << 17, 1 << 26, True), (2048.0, 1 << 18, 1 << 17, 1 << 20, True),
        (1e4, 5000, 1 << 20, 1 << 20, False), (1e4, 1 << 18, 3000, 1 << 20, False), (1e4, 1 << 18, 6000, 1 << 20, True),
        (1e4, 1 << 18, 6000, 0, True), (511.0, 1 << 18, 300000, 1 << 20, False), (512.0, 1 << 18, 300000, 1 << 20, True),
        (1e4, 1 << 18, 5500, 1 << 20, False), (5e4, 1 << 18, 1199, 1 << 20, False), (5e4, 1 << 18, 1200, 1 << 20, True),
        (1000.0, 1 << 18, 23999, 1 << 20, False), (1000.0, 1 << 18, 24000, 1 << 20, True),
        (float("nan"), 1 << 18, 300000, 1 << 20, False)]
    hs = {}
    for spread, n_l, n_e, cap, nodes in cases:
        key = (spread, n_l)
        if key not in hs:
            ctx.lib.host_spread(spread)
            hs[key] = ctx.hierarchy(n_l, leaf=8, device=device)
            ctx.log()
        st = [ctx.traverse(hs[key], n_e, cap), ctx.noalloc(hs[key], n_e, cap)]
        assert all(q in (hrr.HRR_OK, hrr.HRR_E_OVERFLOW) for q in st)
        walks = [x.split()[0] for x in ctx.log() if "tasks=" in x]
        assert walks == ["nodes" if nodes else "blocks"] * 2, (spread, n_l, n_e, cap)
    # in a batch the two walks' items are launched side by side
    a, b = hs[(3.0, 1 << 18)], hs[(1e4, 1 << 18)]
    assert ctx.batched([(a, 3000, 1e-4, 1 << 20), (b, 6000, 1e-4, 1 << 20), (a, 10, 1e-4, 100)])[0] == hrr.HRR_OK
    assert [(x.split()[0], _fields(x)["items"]) for x in ctx.log() if "tasks=" in x] == [("blocks", 2), ("nodes", 1)]
    ctx.lib.host_spread(1.0)
    for h in hs.values():
        ctx.free(h)


@pytest.mark.parametrize("device", [False, True])
def test_repeated_readbacks_need_no_device_copy(ctx, device):
    """A program that asks for the light order again and again is served from a
    host copy: one built on the device is read twice at the most."""
    n = 5000
    h = ctx.hierarchy(n, device=device)
    ctx.log()
    for call, shape, dtype, size in ((ctx.lib.hrr_hierarchy_permutation, n, np.uint32, 4 * n),
                                     (ctx.lib.hrr_hierarchy_sorted_lights, 3 * n, np.float32, 16 * n)):
        outs = [np.zeros(shape, dtype) for _ in range(5)]
        for out in outs:
            assert call(h, out.ctypes.data) == hrr.HRR_OK
        assert all(np.array_equal(out, outs[0]) for out in outs) and len(np.unique(outs[0])) > n // 2
        assert ctx.log() == (["read %d" % size] * 2 if device else [])
    ctx.free(h)


def test_a_readback_without_room_for_its_copy(ctx):
    """The host copy is a convenience: a full heap costs the next call a device
    copy, not this one its result."""
    n = 5000
    h = ctx.hierarchy(n)
    out = [np.zeros(n, np.uint32) for _ in range(4)]
    assert ctx.lib.hrr_hierarchy_permutation(h, out[0].ctypes.data) == hrr.HRR_OK
    ctx.lib.host_fail_new(0)
    st = ctx.lib.hrr_hierarchy_permutation(h, out[1].ctypes.data)
    ctx.lib.host_fail_new(-1)
    assert st == hrr.HRR_OK
    for o in out[2:]:
        assert ctx.lib.hrr_hierarchy_permutation(h, o.ctypes.data) == hrr.HRR_OK
    assert all(np.array_equal(o, out[0]) for o in out) and out[0].any()
    ctx.free(h)


def _server(ctx, budget):
    import ctypes
    cfg = hrr.HrrServerConfig(budget, 1, 1 << 16, 64, 0, 64.0, 100.0)
    return ctx.lib.hrr_server_start(ctx.handle, ctypes.byref(cfg))


@pytest.mark.parametrize("what", ["traverse", "host build", "device build", "server"])
def test_kept_memory_is_given_back_when_room_is_short(ctx, what):
    """Blocks of freed hierarchies and the build scratch, which a context keeps for
    later builds, are no reason to refuse any other allocation."""
    lib = ctx.lib
    h = ctx.hierarchy(1000)
    before = lib.host_used()
    for g in [ctx.hierarchy(1 << 18) for _ in range(4)]:
        ctx.free(g)
    kept = lib.host_used() - before
    assert kept > 50 << 20
    lib.host_limit(before + kept + (1 << 20))             # room for 1 MiB beside what is kept
    try:
        if what == "traverse":
            st = ctx.traverse(h, 30000, 3 << 23)           # its chunks need tens of MiB of slack
        elif what == "host build":
            st, g = ctx.build(1 << 18, device=False, leaf=8)
        elif what == "device build":
            st, g = ctx.build(1 << 19)                      # outgrows every kept block
        else:
            st = _server(ctx, 40 << 20)
        assert st == hrr.HRR_OK, ctx.error()
        # what does not fit even so is refused, and the next call is not
        assert _server(ctx, 1 << 40) in (hrr.HRR_E_NOMEM, hrr.HRR_E_BUSY)
        assert ctx.traverse(h, 10, 100) == hrr.HRR_OK
    finally:
        lib.host_limit(2 ** 64 - 1)
    assert lib.host_last_error() == 0
    lib.hrr_server_stop(ctx.handle)
    if what.endswith("build"):
        ctx.free(g)
    ctx.free(h)


def test_freeing_a_hierarchy_fails_quietly(ctx):
    """hrr_free_hierarchy has no status: when the block cannot be kept (a stream is
    being captured, host memory is out, another context frees it) it is freed, and
    neither an exception nor an error is left behind."""
    lib = ctx.lib
    before = lib.host_used()
    other = HostContext(lib)
    base = lib.host_used()
    for how in ("sync", "new", "other", "no context"):
        h = ctx.hierarchy(5000)
        if how == "sync":
            lib.host_fail_device_sync(1)
            ctx.free(h)
            lib.host_fail_device_sync(0)
        elif how == "new":
            lib.host_fail_new(0)
            ctx.free(h)
            lib.host_fail_new(-1)
        elif how == "other":
            other.free(h)
        else:
            lib.hrr_free_hierarchy(None, h)
        assert lib.host_last_error() == 0, how
        g = ctx.hierarchy(5000)
        assert ctx.traverse(g, 10, 100) == hrr.HRR_OK
        ctx.free(g)
    ctx.free(ctx.hierarchy(5000))
    other.close()
    ctx.close()
    assert lib.host_used() <= before
    ctx.handle = HostContext(lib).handle       # for the fixture to close
