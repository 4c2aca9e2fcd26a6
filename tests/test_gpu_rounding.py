"""Errors against 64 bits at rounding level: the relative L2 error of whole outputs, root mean square over some seeds,
against that of the kernels that summed every pair term or every visit apart (measured with the same inputs; one part in
200 is allowed for the order of the sums)."""
import numpy as np
import pytest

import oracle as O
import paper_2008_05712_amd as gc
import workloads as W
from gpu_helpers import GravRig, whole
from test_gpu_adjoint import _lj_vjp_gpu, grav_vjp_gpu
from test_gpu_lj import LJRig

pytestmark = pytest.mark.gpu

TYPES = {1: ([1.0], [1.0], [1.0]), 2: ([1.0, 0.5], [1.0, 0.88], [1.0, 1.0])}


def _atoms(side, types, seed):
    xyz, _v, L = W.fcc_modulated(side, side, side, 0.8442, int(3.6 * side ** 3), seed=seed)
    t = np.random.default_rng(seed + 1).integers(0, types, xyz.shape[0])
    return W.build_lj(xyz, t, L, 2.5, *TYPES[types])


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b))


def lj(ctx, side, types, seed):
    w = _atoms(side, types, seed)
    rig = LJRig(ctx, w)
    acc = rig.run(gc.REORG_NONE)[:, :3]
    rig.close()
    return _rel(acc, O.lj_tasks(w))


def lj_gradient(ctx, side, types, seed):
    w = _atoms(side, types, seed)
    g = np.random.default_rng(seed + 2).normal(size=(w.n, 3)).astype(np.float32).astype(np.float64)
    return _rel(_lj_vjp_gpu(ctx, w, g)[0][0], O.vjp_lj(w, g)[0])


def gravity_gradient(ctx, plummer, order, seed):
    w = W.build_grav(W.plummer(80000, seed) if plummer else W.uniform_cube(80000, seed), bucket=16, theta=0.7)
    g = np.random.default_rng(seed + 2).normal(size=(w.n, 3)).astype(np.float32).astype(np.float64)
    got, want = grav_vjp_gpu(ctx, w, g, order=order), O.vjp_grav(w, g, order=order)
    return _rel(got[1], want[1])  # (of the masses: larger than the positions' by far)


def ewald(ctx, n, quad, seed):
    w = W.build_grav(W.uniform_cube(n, seed), bucket=32, theta=0.7)
    rng = np.random.default_rng(seed + 2)
    com = rng.uniform(0.4, 0.6, 3).astype(np.float32)
    S = (np.array([0.083, 0.083, 0.083, 0.0, 0.0, 0.0]) + rng.normal(size=6) * 1e-3).astype(np.float32) if quad else None
    ids = np.sort(rng.choice(n, 20000, replace=False))
    rig = GravRig(ctx, w)
    b = rig.batch(whole(w))
    b.reorganize(rig.pool, gc.REORG_NONE)
    rig.acc.zero_()
    b.ewald(gc.ewald_params(1.0, 1.0, com, S=S), rig.acc)
    rig.torch.cuda.synchronize()
    acc = rig.acc.cpu().numpy()[ids, :3]
    b.destroy()
    rig.close()
    return _rel(acc, O.ewald(w.rec[ids, :3], 1.0, 1.0, 1.0, com.astype(np.float64), 2.0, 1, 10,
                             S=None if S is None else S.astype(np.float64)))


BEFORE = [
    (lj, 28, 1, 4.1579e-7), (lj, 28, 2, 4.4243e-7), (lj, 12, 1, 4.1364e-7),
    (lj_gradient, 28, 1, 4.2296e-7), (lj_gradient, 28, 2, 4.3595e-7), (lj_gradient, 12, 1, 4.2743e-7),
    (lj_gradient, 12, 2, 4.5830e-7),
    (gravity_gradient, True, 2, 1.5339e-7), (gravity_gradient, False, 1, 1.4928e-7),
    (ewald, 40000, True, 3.2664e-7), (ewald, 80000, True, 3.2824e-7), (ewald, 80000, False, 2.5482e-7),
]


def error(ctx, f, a, b):
    seeds = 20 if a == 12 else 3  # (the smallest box: the sums of a few close pairs)
    return float(np.sqrt(np.mean([f(ctx, a, b, 700 + 10 * s) ** 2 for s in range(seeds)])))


@pytest.mark.parametrize("f,a,b,before", BEFORE)
def test_no_further_from_64_bits(f, a, b, before):
    ctx = gc.Context(0)
    e = error(ctx, f, a, b)
    print(f"[gpu] {f.__name__} {a} {b}: {e:.4g} (before {before:.4g})", flush=True)
    ctx.close()
    assert e <= 1.005 * before
