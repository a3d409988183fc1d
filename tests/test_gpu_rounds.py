"""The cold forward whose rounds run in one launch: wheels (two vertices with as many
neighbours as the mesh has others), boxes on both sides of a change of the team's
size, a part no root reaches, budgets below and above the rounds it takes, and input
errors, against the oracle (bar 1e-4 relative, as for the other meshes) and against
rounds as launches (a bucket width beyond all times holds nothing back)."""
import numpy as np
import pytest

import gbp_inputs as gi
import oracle as O
from conftest import random_spd, rng
from test_gpu_leadfield_windows import wheel
from test_gpu_parity import B, _dev, i32, rel_max, t32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def problem(mesh, size):
    r = rng(size)
    if mesh == "wheel":
        xyz, tets = wheel(size, size)
    else:
        xyz, tets = gi.kuhn_cube(size)
    n = len(xyz)
    xyz = np.concatenate([xyz, [[5, 5, 5], [6, 5, 5], [5, 6, 5], [5, 5, 6]]]).astype(np.float32)
    tets = np.concatenate([tets, [[n, n + 1, n + 2, n + 3]]]).astype(np.int32)
    A = np.stack([random_spd(r, 3, 3.0) for _ in range(64)])[r.integers(0, 64, len(tets))]
    D = np.stack([A[:, 0, 0], A[:, 1, 1], A[:, 2, 2], A[:, 0, 1], A[:, 0, 2], A[:, 1, 2]], 1).astype(np.float32)
    vs = r.uniform(0.6, 1.4, size=len(xyz)).astype(np.float32)
    return n, xyz, tets, D, vs, np.array([n - 1, 1, 1], np.int32), np.array([0.2, 0.1, 0.3], np.float32)


@pytest.mark.parametrize("mesh,size", [("wheel", 3), ("wheel", 40), ("wheel", 120), ("box", 3), ("box", 22), ("box", 23)])
def test_rounds_in_one_launch(mesh, size):
    dev = _dev()
    n, xyz, tets, D, vs, rn, rt = problem(mesh, size)
    plan = B().Plan(xyz, tets)
    a = (t32(D, dev), t32(vs, dev), i32(rn, dev), t32(rt, dev))
    T, st = B().eikonal_forward(plan, *a)
    assert st["converged"] and st["unreached"] == 4
    again, st2 = B().eikonal_forward(plan, *a)
    assert torch.equal(T, again) and {**st, "updates": 0} == {**st2, "updates": 0}
    Tn = T.cpu().numpy()
    assert np.all(np.isinf(Tn[n:]))
    if n < 4000:
        To = O.solve(xyz, tets, D, vs, rn, rt)[0]
        assert rel_max(Tn[:n], To[:n]) <= 1e-4
    B().set_hold(plan, 1e6)
    launches, _ = B().eikonal_forward(plan, *a)
    B().set_hold(plan, 0.0)
    assert rel_max(Tn[:n], launches.cpu().numpy()[:n]) <= 1e-4
    Ta = B().eikonal_forward_async(plan, *a, st["rounds"])
    assert B().plan_status(plan)["forward_converged"] and torch.equal(T, Ta)
    assert B().forward_work(plan)["face_solves"] == st["face_solves"]
    if st["rounds"] > 1:
        B().eikonal_forward_async(plan, *a, st["rounds"] - 1)
        assert not B().plan_status(plan)["forward_converged"]
    T0, st0 = B().eikonal_forward(plan, a[0], a[1], a[2][:0], a[3][:0])
    assert st0["converged"] and st0["rounds"] == 0 and st0["unreached"] == n + 4
    with pytest.raises(B().GbpError):
        B().eikonal_forward(plan, -a[0], *a[1:])
    assert torch.equal(T, B().eikonal_forward(plan, *a)[0])
