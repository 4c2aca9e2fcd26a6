"""Device commit at the edges of its kernels: task counts around the launch-order sort's sizes (every task
must be launched once: forces bitwise equal to the host submission's, whose union and positions are the
same), and requests whose ranges start at the same id with different lengths, touch and nest across tasks
(the union and every position against the oracle's insertion)."""
import numpy as np
import pytest

import oracle as O
import paper_2008_05712_amd as gc
import workloads as W
from gpu_helpers import GravRig, grav_tasks, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gc.Context(0)
    yield c
    c.close()


def _device_batch(ctx, tasks, n, n_nodes):
    torch = torch_cuda()
    b = gc.Batch(ctx, gc.KIND_GRAV, n)
    b.submit_device(torch.from_numpy(grav_tasks(tasks).view(np.uint8).copy()).cuda(),
                    torch.from_numpy(np.ascontiguousarray(tasks["ranges"], np.int32)).cuda(),
                    torch.from_numpy(np.ascontiguousarray(tasks["node_idx"], np.int32)).cuda(), n_nodes)
    b.commit()
    return b


@pytest.mark.parametrize("n_tasks", [1, 1023, 1024, 1025, 2049, 4097, 8192, 8193])
def test_every_task_launched_once(ctx, n_tasks):
    torch = torch_cuda()
    w = W.build_grav(W.uniform_cube(8300, 81), bucket=1, theta=1.0)
    t = W.task_subset(w, np.arange(n_tasks))
    rig = GravRig(ctx, w)
    acc = []
    maps = []
    for b in (_device_batch(ctx, t, w.n, w.nodes.shape[0]), rig.batch(t)):
        out = torch.full((w.n, 4), float("nan"), device="cuda")
        b.reorganize(rig.pool, gc.REORG_PACK)
        b.launch(gc.grav_params(order=2), rig.nodes, out)
        torch.cuda.synchronize()
        maps.append(b.maps())
        acc.append(out.cpu().numpy())
        rig.pool.reset()
        b.destroy()
    assert np.isfinite(acc[0][t["i_begin"][0]:t["i_begin"][-1] + t["i_count"][-1]]).all()
    assert np.array_equal(acc[0], acc[1], equal_nan=True)
    for k in ("U", "pos", "pranges", "pi_begin"):
        assert np.array_equal(maps[0][k], maps[1][k]), k
    rig.close()


@pytest.mark.parametrize("n", [40, 4096, 9001])
def test_union_of_overlapping_ranges(ctx, n):
    rng = np.random.default_rng(n)
    rows, ranges, jf = [], [], 0
    targets = np.sort(rng.choice(n // 4, size=min(60, n // 4), replace=False)) * 4
    for i in targets:
        starts = np.unique(rng.choice([0, 4, 5, n // 3, n // 2, n - 7], size=3))
        mine = [(int(s), int(min(rng.integers(1, 40), (starts[k + 1] if k + 1 < len(starts) else n) - s)))
                for k, s in enumerate(starts)]
        rows.append((int(i), int(rng.integers(1, 5)), jf, len(mine)))
        ranges += mine
        jf += len(mine)
    rows = np.array(rows, np.int32)
    z = np.zeros(len(rows), np.int32)
    t = dict(i_begin=rows[:, 0], i_count=np.minimum(rows[:, 1], n - rows[:, 0]).astype(np.int32), j_first=rows[:, 2],
             j_nr=rows[:, 3], n_first=z, n_count=z, ranges=np.array(ranges, np.int32).reshape(-1, 2),
             node_idx=np.zeros(0, np.int32))
    b = _device_batch(ctx, t, n, 1)
    w = W.build_grav(W.uniform_cube(n, 3), bucket=16, theta=0.7)
    rig = GravRig(ctx, w)
    b.reorganize(rig.pool, gc.REORG_PACK)
    got = b.maps()
    U = O.union_insert(t, n)
    pos = np.full(n, -1, np.int32)
    pos[U] = np.arange(U.size)
    assert np.array_equal(got["U"], U)
    assert np.array_equal(got["pos"], pos)
    b.destroy()
    rig.close()


@pytest.mark.parametrize("n_tasks,refused", [(511, False), (512, True), (1024, True), (1025, True)])
def test_direct_entries_beyond_32_bits(ctx, n_tasks, refused):
    # every task lists all 2^22 particles: 512 tasks hold 2^31 direct entries, and 1,024 (one tile of the
    # offsets' scan) exactly 2^32, a total of zero in 32 bits
    torch = torch_cuda()
    n = 1 << 22
    t = np.zeros(n_tasks, gc.TASK_DTYPE)
    t["i_begin"] = np.arange(n_tasks, dtype=np.int32)
    t["i_count"] = 1
    t["j_nranges"] = 1
    b = gc.Batch(ctx, gc.KIND_GRAV, n)
    b.submit_device(torch.from_numpy(t.view(np.uint8).copy()).cuda(), torch.tensor([[0, n]], dtype=torch.int32).cuda(),
                    torch.zeros(0, dtype=torch.int32).cuda(), 1)
    print(f"[gpu] device commit of {n_tasks} tasks of 2^22 direct entries", flush=True)
    if refused:
        with pytest.raises(gc.GcError, match="2.31 entries") as e:
            b.commit()
        assert e.value.status == gc.GC_E_INVAL
    else:
        b.commit()
    b.destroy()
