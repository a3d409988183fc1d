"""Cold rounds as launches without hold-back (meshes past 2^18 vertices): every lane count
and both queue layouts against the oracle (bar 1e-4 relative, as for the other meshes) and
against one another (both end within eps_rel of one fixed point: 1e-5)."""
import numpy as np
import pytest

import gbp_inputs as gi
import oracle as O
from conftest import rng
from test_gpu_parity import B, _dev, i32, rel_max, t32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_plain_rounds_past_one_launch():
    dev, r, cells = _dev(), rng(65), 64
    xyz, tets = gi.kuhn_cube(cells, length=30.0)
    xyz = gi.jitter_nodes(xyz, 30.0 / cells, 0.1, 3)
    assert len(xyz) > 1 << 18
    z = xyz[tets].mean(axis=1)[:, 2] / 30.0
    a = np.pi * (z - 0.5)
    D = gi.fibre_tensor(np.stack([np.cos(a), np.sin(a), np.zeros_like(a)], 1))
    vs = r.uniform(0.7, 1.3, len(xyz)).astype(np.float32)
    rn, rt = r.choice(len(xyz), 40, replace=False).astype(np.int32), r.uniform(0, 5, 40).astype(np.float32)
    To = O.solve(xyz, tets, D, vs, rn, rt)[0]
    plan = B().Plan(xyz, tets)
    args = (t32(D, dev), t32(vs, dev), i32(rn, dev), t32(rt, dev))
    first = None
    for lanes in (8, 16, 32):
        for split in (True, False):
            B().set_launch(plan, lanes, 1024, 128)
            B().set_queue_split(plan, split)
            T, st = B().eikonal_forward(plan, *args)
            T = T.cpu().numpy()
            assert st["converged"] and st["unreached"] == 0
            assert rel_max(T, To) <= 1e-4, (lanes, split)
            first = T if first is None else first
            assert rel_max(T, first) <= 1e-5, (lanes, split)
            Ta = B().eikonal_forward_async(plan, *args, st["rounds"] + 8)
            assert B().plan_status(plan)["forward_converged"] and rel_max(Ta.cpu().numpy(), To) <= 1e-4
