"""The gravity adjoint's items (runs of tasks, or stretches of one long task, that share an LDS table of their
distinct sources) against the FP64 oracle VJP at their edges: a task whose lists exceed the table, lists that
repeat a node or come out of order, tasks without nodes or without direct ranges, target counts around the
register block, and enough tasks that items hold several.

Bar: relative error <= 1e-4 per gradient block, as for the adjoint elsewhere."""
import copy

import numpy as np
import pytest

import oracle as O
import paper_2008_05712_amd as gc
import workloads as W
from gpu_helpers import GravRig, whole
from test_gpu_adjoint import close, grav_vjp_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gc.Context(0)
    yield c
    c.close()


def _check(ctx, w, order, mode=gc.REORG_NONE, seed=7):
    g = np.random.default_rng(seed).normal(size=(w.n, 3)).astype(np.float32).astype(np.float64)
    gp, gm = grav_vjp_gpu(ctx, w, g, mode, order=order)
    rp, rm = O.vjp_grav(w, g, order=order)
    for name, a, b in (("positions", gp, rp), ("masses", gm, rm)):
        ok, e = close(a, b)
        assert ok, (name, e)


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("mode", [gc.REORG_NONE, gc.REORG_PACK])
def test_lists_longer_than_the_table(ctx, order, mode):
    # theta 0: every bucket's direct list is all 2,500 particles; theta 0.15, buckets of 2: thousands of nodes
    _check(ctx, W.build_grav(W.plummer(2500, 91), bucket=24, theta=0.0), order, mode)
    _check(ctx, W.build_grav(W.uniform_cube(9000, 92), bucket=2, theta=0.25), order, mode)


@pytest.mark.parametrize("bucket", [1, 7, 8, 9, 16, 17, 40])
def test_target_blocks(ctx, bucket):
    _check(ctx, W.build_grav(W.plummer(1500, 93), bucket=bucket, theta=0.8), 2)


def _with_lists(w, per):
    w = copy.copy(w)
    w.node_idx = np.concatenate(per).astype(np.int32) if sum(p.size for p in per) else np.zeros(1, np.int32)
    w.n_count = np.array([p.size for p in per], np.int32)
    w.n_first = np.concatenate([[0], np.cumsum(w.n_count)[:-1]]).astype(np.int32)
    return w


def _node_lists(w):
    return [w.node_idx[w.n_first[t]:w.n_first[t] + w.n_count[t]] for t in range(w.n_tasks)]


@pytest.mark.parametrize("lists", ["as_built", "repeated", "some_empty"])
def test_several_tasks_per_item(ctx, lists):
    # more than four tasks for each of four items per CU, so items hold runs of tasks
    w = W.build_grav(W.plummer(60000, 94), bucket=8, theta=1.0)
    assert w.n_tasks > 16 * 256
    rng = np.random.default_rng(97)
    if lists == "repeated":
        w = _with_lists(w, [np.concatenate([p, p[: rng.integers(0, 4)], p[-2:]]) for p in _node_lists(w)])
    elif lists == "some_empty":
        w = _with_lists(w, [p if rng.random() < 0.6 else p[:0] for p in _node_lists(w)])
        w.j_nr = np.where(rng.random(w.n_tasks) < 0.6, w.j_nr, 0).astype(np.int32)
    _check(ctx, w, 2, gc.REORG_PACK)


def test_long_tasks_among_many(ctx):
    # 4,200 tasks of one target, each with every particle in its direct list: stretches of one task's sources
    w = W.build_grav(W.uniform_cube(4200, 98), bucket=1, theta=0.0)
    assert w.n_tasks > 16 * 256
    _check(ctx, w, 1)


def test_long_tasks_among_runs(ctx):
    # 5,300 tasks, items of five: stretches of one task's sources between runs of several (every 50th task of one target
    # has every particle in its direct list, the others their own neighbourhood)
    w = W.build_grav(W.uniform_cube(5300, 98), bucket=1, theta=0.9)
    assert w.n_tasks >= 5 * 4 * 256
    w.ranges = np.concatenate([w.ranges, [[0, w.n]]]).astype(np.int32)
    w.j_first, w.j_nr = w.j_first.copy(), w.j_nr.copy()
    w.j_first[::50] = w.ranges.shape[0] - 1
    w.j_nr[::50] = 1
    _check(ctx, w, 2)


@pytest.mark.parametrize("tasks", [5 * 1024 - 1, 5 * 1024])
@pytest.mark.parametrize("mode", [gc.REORG_NONE, gc.REORG_PACK])
def test_either_side_of_the_line(ctx, tasks, mode):
    # an item a task, whose records the device writes, and items of five tasks, whose records come from the host (256 CUs)
    w = W.build_grav(W.plummer(tasks, 102), bucket=1, theta=0.9)
    assert w.n_tasks == tasks
    _check(ctx, w, 2, mode)


@pytest.mark.parametrize("lists", ["reversed", "repeated", "no_nodes", "no_direct", "some_empty"])
def test_lists_of_any_form(ctx, lists):
    w = W.build_grav(W.plummer(3000, 95), bucket=16, theta=0.8)
    rng = np.random.default_rng(96)
    per = _node_lists(w)
    if lists == "reversed":
        per = [p[::-1] for p in per]
    elif lists == "repeated":
        per = [np.concatenate([p, p[: rng.integers(0, p.size + 1)], p[:3]]) for p in per]
    elif lists == "no_nodes":
        per = [p[:0] for p in per]
    elif lists == "some_empty":
        per = [p if rng.random() < 0.5 else p[:0] for p in per]
    w = _with_lists(w, per)
    if lists == "no_direct":
        w.j_nr = np.zeros_like(w.j_nr)
    if lists == "some_empty":
        w.j_nr = np.where(rng.random(w.n_tasks) < 0.5, w.j_nr, 0).astype(np.int32)
    _check(ctx, w, 2)


def test_indices_after_a_failed_rebuild():
    # A call with another n_nodes builds the indices again.  Where an allocation of that build fails, the call reports it
    # and the next one, with the first n_nodes, builds its own; before, it would have taken the buffers for its own.
    import torch
    refuse = []

    def alloc(nbytes, _user):
        return None if refuse and refuse.pop() else torch.cuda.caching_allocator_alloc(int(nbytes), 0)

    def free(ptr, _user):
        torch.cuda.caching_allocator_delete(ptr)

    c = gc.Context(0, allocator=(alloc, free))
    w = W.build_grav(W.plummer(3000, 99), bucket=16, theta=0.8)
    g = np.random.default_rng(100).normal(size=(w.n, 3)).astype(np.float32).astype(np.float64)
    rig = GravRig(c, w)
    b = rig.batch(whole(w))
    rig.run(b, gc.REORG_PACK, order=2)
    cot = torch.zeros((w.n, 4), dtype=torch.float32, device="cuda")
    cot[:, :3] = torch.from_numpy(g.astype(np.float32)).cuda()
    n = w.nodes.shape[0]
    # the same nodes and 200,000 more that no list names: larger indices, so their buffer is allocated again
    more = 200_000
    nr = torch.from_numpy(np.concatenate([w.node_range, np.zeros((more, 2), np.int32)]).astype(np.int32)).cuda()
    nodes = torch.cat([rig.nodes.reshape(n, -1), torch.zeros((more, rig.nodes.numel() // n), device="cuda")]).contiguous()
    rp, rm = O.vjp_grav(w, g, order=2)

    def backward(n_nodes):
        gpos = torch.zeros((w.n, 4), dtype=torch.float32, device="cuda")
        gmass = torch.zeros(w.n, dtype=torch.float32, device="cuda")
        b.backward(gc.grav_params(order=2), nodes, nr, n_nodes, cot, gpos, gmass)
        torch.cuda.synchronize()
        for name, x, y in (("positions", gpos.cpu().numpy()[:, :3], rp), ("masses", gmass.cpu().numpy(), rm)):
            ok, e = close(x, y)
            assert ok, (n_nodes, name, e)

    print("[gpu] adjoint indices, a refused allocation between two builds", flush=True)
    backward(n)
    refuse.append(True)
    with pytest.raises(gc.GcError) as err:
        backward(n + more)
    assert err.value.status == gc.GC_E_NOMEM and not refuse
    backward(n)
    backward(n + more)
    backward(n)
    b.destroy()
    rig.close()
    c.close()


def test_a_long_run_of_tasks_without_sources(ctx):
    # an item holds at most 16 tasks, those without nodes or direct ranges among them
    w = W.build_grav(W.plummer(60000, 94), bucket=8, theta=1.0)
    n = w.n_tasks
    assert n > 16 * 256
    bare = (np.arange(n) >= n // 8) & (np.arange(n) < n // 2)
    w = _with_lists(w, [p[:0] if bare[t] else p for t, p in enumerate(_node_lists(w))])
    w.j_nr = np.where(bare, 0, w.j_nr).astype(np.int32)
    _check(ctx, w, 2, gc.REORG_PACK)


@pytest.mark.parametrize("mode", [gc.REORG_NONE, gc.REORG_PACK])
def test_softening_whose_square_underflows(ctx, mode):
    # soft_eps 1e-24: its square is zero in 32 bits, and the skipped pair of a particle with itself must stay skipped.
    # Particles on a lattice, so that no other two lie close together; direct lists alone.
    import torch
    k = np.arange(8, dtype=np.float64)
    xyz = np.stack(np.meshgrid(k, k, k, indexing="ij"), -1).reshape(-1, 3) + 0.25
    rec = np.concatenate([xyz, np.full((512, 1), 1.0 / 512)], 1).astype(np.float32)
    w = W.build_grav(rec, bucket=16, theta=0.0)
    g = np.random.default_rng(101).normal(size=(w.n, 3)).astype(np.float32).astype(np.float64)
    rig = GravRig(ctx, w)
    b = rig.batch(whole(w))
    b.reorganize(rig.pool, mode)
    cot = torch.zeros((w.n, 4), dtype=torch.float32, device="cuda")
    cot[:, :3] = torch.from_numpy(g.astype(np.float32)).cuda()
    gpos = torch.zeros((w.n, 4), dtype=torch.float32, device="cuda")
    gmass = torch.zeros(w.n, dtype=torch.float32, device="cuda")
    nr = torch.from_numpy(np.ascontiguousarray(w.node_range)).cuda()
    b.backward(gc.grav_params(order=1, eps=1e-24), rig.nodes, nr, w.nodes.shape[0], cot, gpos, gmass)
    torch.cuda.synchronize()
    rp, rm = O.vjp_grav(w, g, eps=1e-24, order=1)
    for name, x, y in (("positions", gpos.cpu().numpy()[:, :3], rp), ("masses", gmass.cpu().numpy(), rm)):
        ok, e = close(x, y)
        assert ok, (name, e)
    b.destroy()
    rig.close()
