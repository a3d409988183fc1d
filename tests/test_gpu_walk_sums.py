"""The adjoint's sums: lambda_i = g_i + sum alpha_c lambda_c over i's children, replayed
on the host along the same parents with exact products, sums in FP64 and each lambda
rounded to FP32 once, for isotropic media on non-obtuse meshes (no cycles).

The gradients of the active roots' onsets are lambdas.  FP64 sums in another order differ
by 1e-16 of their terms, so the replay gives the same FP32 number but for a sum at a
rounding boundary, or where an oracle's weight rounds the other way: the same number on
nine roots of ten, two spacings (2^-22) on the others.  FP32 products, or sums, leave a
few spacings on most of the larger sums.  Gradients >= 0: nothing cancels."""
import numpy as np
import pytest

import gbp_inputs as gi
from conftest import rng
from oracle import tri as O2
from test_gpu_parity import B, _dev, i32, t32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def replay(par_node, par_alpha, T, g):
    lam = g.astype(np.float32)
    n_par = (par_node >= 0) & (par_alpha > 0)
    acc = g.astype(np.float64)
    for i in np.argsort(-T, kind="stable"):        # children are later than their parents
        lam[i] = np.float32(acc[i])
        for p, a, on in zip(par_node[i], par_alpha[i], n_par[i]):
            if on:
                acc[p] += np.float64(np.float32(a)) * np.float64(lam[i])
    return lam


def compare(got, want, active):
    assert active.sum() >= 20
    got, want = got[active].astype(np.float64), want[active].astype(np.float64)
    rel = np.abs(got - want) / np.abs(want)
    assert rel.max() <= 2.0**-22 and np.mean(got == want) >= 0.9, (rel.max(), np.mean(got == want))


def roots(r, n):
    return r.choice(n, 60, replace=False).astype(np.int32), r.uniform(0, 0.1, 60).astype(np.float32)


@pytest.mark.parametrize("cells", [12, 24])      # one block, a team
def test_tet_sums(cells):
    dev, r = _dev(), rng(cells)
    xyz, tets = gi.kuhn_cube(cells)
    D = np.tile(np.array([1, 1, 1, 0, 0, 0], np.float32), (len(tets), 1))
    vs = r.uniform(0.9, 1.1, len(xyz)).astype(np.float32)
    rn, rt = roots(r, len(xyz))
    g = r.uniform(0, 1, len(xyz)).astype(np.float32)
    plan = B().Plan(xyz.astype(np.float32), tets.astype(np.int32))
    a = (plan, t32(D, dev), t32(vs, dev), i32(rn, dev), t32(rt, dev))
    T, _ = B().eikonal_forward(*a)
    _, pn, pa, _ = B().parent_map(*a, T)
    _, _, drt = B().eikonal_backward(*a, T, t32(g, dev), want_D=False)
    assert B().backward_info(plan)["cyclic"] == 0
    lam = replay(pn.cpu().numpy(), pa.cpu().numpy(), T.cpu().numpy(), g)
    drt = drt.cpu().numpy()
    compare(drt, lam[rn], drt != 0)


@pytest.mark.parametrize("cells", [50, 90])
def test_triangle_sums(cells):
    dev, r = _dev(), rng(cells)
    xy, tris = gi.square_tri(cells)
    D = np.tile(np.array([1, 1, 0], np.float32), (len(tris), 1))
    vs = r.uniform(0.9, 1.1, len(xy)).astype(np.float32)
    rn, rt = roots(r, len(xy))
    g = r.uniform(0, 1, len(xy)).astype(np.float32)
    plan = B().TriPlan(xy.astype(np.float32), tris.astype(np.int32))
    a = (plan, t32(D, dev), t32(vs, dev), i32(rn, dev), t32(rt, dev))
    T, _ = B().tri_forward(*a)
    Tn = T.cpu().numpy()
    par = O2.parent_map2(xy.astype(np.float32), tris, O2.metric_inverse2(D, vs, tris), rn, rt, Tn)
    _, _, drt = B().tri_backward(*a, T, t32(g, dev), want_D=False)
    assert B().tri_backward_info(plan)["cyclic"] == 0
    lam = replay(par["par_node"], par["par_alpha"], Tn, g)
    drt = drt.cpu().numpy()
    compare(drt, lam[rn], drt != 0)
