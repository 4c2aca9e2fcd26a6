"""The combined gravity kernel at the edges of its tiles, against the FP64 oracle: node lists around the node
tiles of a wavefront, direct ranges cut into many short and empty ones (more than one group of 64, starts that
fall on every place of a 64-record window), target counts on either side of 64, and the potential's own-term check.

Bars: per-task relative L2 <= 1e-5 for accelerations and potentials, as for the kernel elsewhere."""
import numpy as np
import pytest

import oracle as O
import paper_2008_05712_amd as gc
import workloads as W
from gpu_helpers import GravRig, rel_l2_per_task, whole

pytestmark = pytest.mark.gpu
TOL = 1e-5
LENGTHS = [0, 1, 2, 63, 64, 65, 191, 192, 193, 255, 256, 257, 383, 385, 767, 768, 769, 1030]


@pytest.fixture(scope="module")
def ctx():
    c = gc.Context(0)
    yield c
    c.close()


def _edges(bucket, seed):
    """A Plummer problem whose node lists have the lengths above (a task's own nodes over and over) and whose
    ranges are cut into pieces of 0 to 5 records."""
    w = W.build_grav(W.plummer(1400, seed), bucket=bucket, theta=0.7)
    rng = np.random.default_rng(seed)
    bt = whole(w)
    node_idx, n_first, n_count, ranges, j_first, j_nr = [], [], [], [], [], []
    for t in range(w.n_tasks):
        own = w.node_idx[w.n_first[t]:w.n_first[t] + w.n_count[t]]
        L = LENGTHS[t % len(LENGTHS)] if own.size else 0
        n_first.append(sum(map(len, node_idx)))
        n_count.append(L)
        node_idx.append(np.resize(own, L) if L else own[:0])
        j_first.append(len(ranges))
        for b, n in bt["ranges"].reshape(-1, 2)[bt["j_first"][t]:bt["j_first"][t] + bt["j_nr"][t]]:
            while n > 0:
                k = min(int(rng.integers(0, 6)), int(n))
                ranges.append((b, k))
                b, n = b + k, n - k
        j_nr.append(len(ranges) - j_first[-1])
    bt = dict(bt, node_idx=np.concatenate(node_idx).astype(np.int32), ranges=np.array(ranges, np.int32),
              n_first=np.array(n_first, np.int32), n_count=np.array(n_count, np.int32),
              j_first=np.array(j_first, np.int32), j_nr=np.array(j_nr, np.int32))
    return w, bt


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("bucket", [3, 24, 33, 90])
@pytest.mark.parametrize("shape", [dict(), dict(targets_per_lane=2, waves_per_block=1), dict(waves_per_block=3, tile=64),
                                   dict(schedule=1, targets_per_lane=3, waves_per_block=8), dict(want_potential=1),
                                   dict(want_potential=1, waves_per_block=1, tile=128)])
def test_tile_edges(ctx, order, bucket, shape):
    print(f"[gpu] grav tile edges order={order} bucket={bucket} {shape}", flush=True)
    w, bt = _edges(bucket, 301)
    rig = GravRig(ctx, w)
    b = rig.batch(bt)
    for mode in (gc.REORG_NONE, gc.REORG_PACK):
        rig.pool.reset()
        acc = rig.run(b, mode, order=order, **shape)
        ref, pot = O.grav_workload(w, order=order, tasks=bt, potential=True)
        err = rel_l2_per_task(acc, ref, bt)
        assert err.max() <= TOL, (mode, err.max(), int(err.argmax()))
        if shape.get("want_potential"):
            perr = O.per_task_rel_l2(acc[:, 3:4].astype(np.float64), pot[:, None], bt["i_begin"], bt["i_count"])
            assert perr.max() <= TOL, (mode, perr.max(), int(perr.argmax()))
        else:
            assert np.all(acc[:, 3].view(np.int32) == 0)
    b.destroy()
    rig.close()


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("mode", [gc.REORG_INDIRECT, gc.REORG_SORTED])
@pytest.mark.parametrize("shape", [dict(), dict(targets_per_lane=2, waves_per_block=1),
                                   dict(schedule=1, targets_per_lane=3, waves_per_block=8)])
def test_tile_edges_of_address_lists(ctx, order, mode, shape):
    # (with address lists a monopole node tile holds 64 nodes, else 128)
    for bucket in (3, 24, 90):
        print(f"[gpu] grav tile edges, address lists, order={order} bucket={bucket} mode={mode} {shape}", flush=True)
        w, bt = _edges(bucket, 302)
        rig = GravRig(ctx, w)
        b = rig.batch(bt)
        acc = rig.run(b, mode, order=order, **shape)
        err = rel_l2_per_task(acc, O.grav_workload(w, order=order, tasks=bt), bt)
        assert err.max() <= TOL, (err.max(), int(err.argmax()))
        b.destroy()
        rig.close()


@pytest.mark.parametrize("order", [1, 2])
def test_node_list_longer_than_a_raw_buffer(ctx, order):
    # one wavefront's list of 2^25 + 1,000 entries is read in two stretches (its own nodes over and over)
    w = W.build_grav(W.plummer(300, 303), bucket=4, theta=1.0)
    t = int(np.argmax(w.n_count))
    own = w.node_idx[w.n_first[t]:w.n_first[t] + w.n_count[t]]
    L = (1 << 25) + 1000
    one = lambda v: np.array([v], np.int32)  # noqa: E731
    bt = dict(i_begin=one(w.i_begin[t]), i_count=one(w.i_count[t]), j_first=one(0), j_nr=one(0),
              ranges=np.zeros((0, 2), np.int32), n_first=one(0), n_count=one(L), node_idx=np.resize(own, L).astype(np.int32))
    print(f"[gpu] grav node list of {L} entries order={order}", flush=True)
    rig = GravRig(ctx, w)
    b = rig.batch(bt)
    acc = rig.run(b, gc.REORG_NONE, order=order, waves_per_block=1)
    err = rel_l2_per_task(acc, O.grav_workload(w, order=order, tasks=bt), bt)
    assert err.max() <= TOL, err.max()
    b.destroy()
    rig.close()
