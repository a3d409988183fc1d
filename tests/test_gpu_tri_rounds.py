"""The triangle forward around its one-block limit (4096 vertices): grids and fans (one
vertex with as many neighbours as the mesh has others) on both sides of it, a part no
root reaches, a single triangle and no roots, against the triangle oracle (bar 1e-4
relative as for the other meshes: float32 times to the eps_rel 2^-20 fixed point)."""
import numpy as np
import pytest

import gbp_inputs as gi
from conftest import random_spd, rng
from oracle import tri as O2
from test_gpu_parity import B, _dev, i32, rel_max, t32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def fan(n):
    a = 2 * np.pi * np.arange(n) / n
    k = np.arange(n)
    xy = np.concatenate([[[0.0, 0.0]], np.stack([np.cos(a), np.sin(a)], 1)]).astype(np.float32)
    return xy, np.stack([np.zeros(n, int), 1 + k, 1 + (k + 1) % n], 1).astype(np.int32)


@pytest.mark.parametrize("mesh,size", [("grid", 1), ("grid", 62), ("grid", 63), ("grid", 64), ("fan", 3), ("fan", 300),
                                       ("fan", 4092), ("fan", 4093), ("fan", 4200)])
def test_tri_rounds(mesh, size):
    dev = _dev()
    r = rng(size)
    xy, tris = gi.square_tri(size) if mesh == "grid" else fan(size)
    n = len(xy)
    xy = np.concatenate([xy, [[5, 5], [6, 5], [5, 6]]]).astype(np.float32)     # a part no root reaches
    tris = np.concatenate([tris, [[n, n + 1, n + 2]]]).astype(np.int32)
    D = np.stack([O2.pack2(random_spd(r, 2, 4.0)) for _ in range(len(tris))]).astype(np.float32)
    vs = r.uniform(0.6, 1.4, size=len(xy)).astype(np.float32)
    rn = np.array([n - 1, 1, 1], np.int32)
    rt = np.array([0.2, 0.1, 0.3], np.float32)
    plan = B().TriPlan(xy, tris)
    To, _ = O2.solve2(xy, tris, D, vs, rn, rt)
    for _ in range(2):
        T, st = B().tri_forward(plan, t32(D, dev), t32(vs, dev), i32(rn, dev), t32(rt, dev))
        T = T.cpu().numpy()
        assert st["converged"] and st["unreached"] == 3 and np.all(np.isinf(T[n:]))
        assert st["rounds"] > 0 and st["face_solves"] > 0 and st["node_updates"] > 0
        assert rel_max(T[:n], To[:n]) <= 1e-4
    T, st = B().tri_forward(plan, t32(D, dev), t32(vs, dev), i32(rn[:0], dev), t32(rt[:0], dev))
    assert st["converged"] and st["rounds"] == 0 and st["unreached"] == n + 3
    with pytest.raises(B().GbpError):
        B().tri_forward(plan, t32(-D, dev), t32(vs, dev), i32(rn, dev), t32(rt, dev))
    T2, _ = B().tri_forward(plan, t32(D, dev), t32(vs, dev), i32(rn, dev), t32(rt, dev))
    assert rel_max(T2.cpu().numpy()[:n], To[:n]) <= 1e-4
