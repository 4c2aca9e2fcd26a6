"""The list walk's one call: lists of every length, in storage of their own size, whole on every stream when the call
returns, and a call without memory for them."""
import numpy as np
import pytest

import oracle as O
import paper_2008_05712_amd as gc
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("theta", [0.0, 0.05, 0.7, 1.5])
def test_lists_of_every_length(ctx, theta, noalloc):
    import torch
    w = W.build_grav(W.plummer(6000, 97), bucket=4, theta=0.7)
    leaf = np.ascontiguousarray(w.meta["leaf"], np.int32)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in
           (w.node_range.astype(np.int32), w.node_mom64[:, :3], w.node_side, w.rec, leaf)]
    got = gc.tree_walk(ctx, *dev, theta, noalloc=noalloc)
    want = O.bh_walk(w.node_range, w.node_parent, w.node_side, w.node_mom64[:, :3], w.rec, leaf, theta)
    print(f"[gpu] walk room theta={theta} nodes {got[1].numel()} ranges {got[3].shape[0]} buckets {leaf.size}", flush=True)
    for a, b in zip(got, want):
        assert np.array_equal(a.cpu().numpy(), b)
    for x in (got[1], got[3]):  # at most twice what the lists need (or one entry)
        assert x.untyped_storage().nbytes() <= max(8 * x.numel(), 16)


@pytest.mark.parametrize("noalloc", [False, True])
def test_lists_are_whole_on_the_callers_stream(ctx, noalloc):
    # The walk runs on a stream of the caller's while the current one is busy; its lists are used on the caller's
    # stream, and on a third one, with nothing to wait for.
    import torch
    w = W.build_grav(W.uniform_cube(20000, 98), bucket=16, theta=0.7)
    leaf = np.ascontiguousarray(w.meta["leaf"], np.int32)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in
           (w.node_range.astype(np.int32), w.node_mom64[:, :3], w.node_side, w.rec, leaf)]
    want = O.bh_walk(w.node_range, w.node_parent, w.node_side, w.node_mom64[:, :3], w.rec, leaf, w.theta)
    own, third = torch.cuda.Stream(), torch.cuda.Stream()
    busy = torch.ones((4096, 4096), device="cuda")
    for x in (want[1], want[3]):  # (memory that they may get holds nothing like them)
        torch.full(x.shape, -7, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    print("[gpu] walk on a stream of the caller's beside a busy one", flush=True)
    for _ in range(40):
        busy = busy @ busy * 1e-4
    got = gc.tree_walk(ctx, *dev, w.theta, stream=own, noalloc=noalloc)
    copies = []
    for s in (own, third):
        with torch.cuda.stream(s):
            copies.append([x.clone() for x in got])
        s.synchronize()
    for c in copies:
        for a, b in zip(c, want):
            assert np.array_equal(a.cpu().numpy(), b)


@pytest.mark.parametrize("noalloc", [False, True])
def test_lists_without_memory(ctx, noalloc, monkeypatch):
    # No memory for a list: the error is torch's, and the next call walks as if nothing had been.
    import torch
    w = W.build_grav(W.uniform_cube(20000, 98), bucket=16, theta=0.7)
    leaf = np.ascontiguousarray(w.meta["leaf"], np.int32)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in
           (w.node_range.astype(np.int32), w.node_mom64[:, :3], w.node_side, w.rec, leaf)]
    want = O.bh_walk(w.node_range, w.node_parent, w.node_side, w.node_mom64[:, :3], w.rec, leaf, w.theta)
    empty = torch.empty

    def none(size, **kw):
        if size in (want[1].size, tuple(want[3].shape)):
            raise torch.OutOfMemoryError("lists")
        return empty(size, **kw)

    with monkeypatch.context() as m:
        m.setattr(torch, "empty", none)
        with pytest.raises(torch.OutOfMemoryError, match="lists"):
            gc.tree_walk(ctx, *dev, w.theta, noalloc=noalloc)
    got = gc.tree_walk(ctx, *dev, w.theta, noalloc=noalloc)
    for a, b in zip(got, want):
        assert np.array_equal(a.cpu().numpy(), b)
        assert a.untyped_storage().nbytes() == 4 * a.numel()  # exactly the lists


@pytest.mark.parametrize("refused", [0, 1, 2, 3])
def test_scratch_that_does_not_fit(refused):
    # The group walk's scratch, then the per-bucket rooms, then the subtree ends alone; no memory for those is an error.
    import torch
    w = W.build_grav(W.plummer(6000, 97), bucket=16, theta=0.7)
    leaf = np.ascontiguousarray(w.meta["leaf"], np.int32)
    asked = []

    def alloc(nbytes, _user):
        asked.append(int(nbytes))
        return None if len(asked) <= refused else torch.cuda.caching_allocator_alloc(int(nbytes), 0)

    def free(ptr, _user):
        torch.cuda.caching_allocator_delete(ptr)

    c = gc.Context(0, allocator=(alloc, free))
    asked.clear()
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in
           (w.node_range.astype(np.int32), w.node_mom64[:, :3], w.node_side, w.rec, leaf)]
    n, nb = w.node_range.shape[0], leaf.size
    rings = next(r for r in range(1, 32) if 128 * (2 ** r - 1) >= n)
    head = 4 * n
    sizes = [head + 72 * n + nb * (44 + 120 * (8 * rings + 1)), head + nb * (4 * 2048 + 8 * 128), head]
    if refused == 3:
        with pytest.raises(gc.GcError) as e:
            gc.tree_walk(c, *dev, w.theta)
        assert e.value.status == gc.GC_E_NOMEM
    else:
        got = gc.tree_walk(c, *dev, w.theta)
        want = O.bh_walk(w.node_range, w.node_parent, w.node_side, w.node_mom64[:, :3], w.rec, leaf, w.theta)
        for a, b in zip(got, want):
            assert np.array_equal(a.cpu().numpy(), b)
    assert len(asked) == min(refused + 1, 3)
    for a, b in zip(asked, sizes):  # (the arrays are padded to 256 bytes, and the last group to 64 buckets)
        assert b <= a <= b + 4096 + 64 * 20000, (asked, sizes)
    c.close()
