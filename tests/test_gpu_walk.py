"""The adjoint's walk at the sizes where its launch changes: one block, a team on one
XCD (few or many blocks), a team on every XCD, Gauss-Seidel sweeps by a team or as
launches.

Oracle: weights of a vertex's parents sum to 1, so whatever the (valid) parents are, the
gradients of the active roots' onsets sum to the incoming gradient's sum.  With
non-negative gradients nothing cancels, and the FP32 sums along at most a few hundred
levels of up to a few dozen children keep the relative error below 1e-4.
"""
import numpy as np
import pytest

import gbp_inputs as gi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [1, 19, 20, 57, 58, 63, 64, 102])
def test_walk_launches(cells):
    import torch
    from paper_2308_08410_amd import binding as B

    dev = torch.device("cuda", 0)
    xyz, tets = gi.kuhn_cube(cells, length=30.0)
    xyz = gi.jitter_nodes(xyz, 30.0 / cells, 0.1, 3)
    # fibres that turn with z: an anisotropic medium, with cycles in its parent graph
    z = xyz[tets].mean(axis=1)[:, 2] / 30.0
    a = np.pi * (z - 0.5) * 1.3
    D = gi.fibre_tensor(np.stack([np.cos(a), np.sin(a), np.zeros_like(a)], 1))
    rng = np.random.Generator(np.random.PCG64(7))
    n_v, R = len(xyz), min(5, len(xyz))
    f32 = lambda x: torch.as_tensor(np.ascontiguousarray(x, np.float32), device=dev)
    rn = torch.as_tensor(rng.choice(n_v, R, replace=False).astype(np.int32), device=dev)
    Dd, vs, rt, g = f32(D), f32(rng.uniform(0.7, 1.3, n_v)), f32(rng.uniform(0, 5, R)), f32(rng.uniform(0, 1, n_v))
    plan = B.Plan(xyz, tets)
    T, _ = B.eikonal_forward(plan, Dd, vs, rn, rt)
    _, dvs, drt = B.eikonal_backward(plan, Dd, vs, rn, rt, T, g, want_D=False)
    info = B.backward_info(plan)
    want = float(g.double().sum())
    assert abs(float(drt.double().sum()) - want) <= 1e-4 * want, info
    assert info["levels"] >= 1 and (info["gs_sweeps"] > 0) == (info["cyclic"] > 0)
    # the enqueue-only walk with just the levels it needs, and with fewer
    gs = max(1, 2 * info["gs_sweeps"])
    _, dvs2, drt2 = B.eikonal_backward_async(plan, Dd, vs, rn, rt, T, g, info["levels"], gs, want_D=False)
    st = B.plan_status(plan)
    assert st["backward_settled"] and st["levels"] == info["levels"]
    assert float((drt2 - drt).abs().max()) <= 1e-5 * float(drt.abs().max())
    assert float((dvs2 - dvs).norm()) <= 1e-5 * float(dvs.norm())
    if info["levels"] > 2:
        B.eikonal_backward_async(plan, Dd, vs, rn, rt, T, g, info["levels"] // 2, 0, want_D=False)
        st = B.plan_status(plan)
        assert not st["backward_settled"] and st["levels"] == info["levels"] // 2
    plan.close()


@pytest.mark.parametrize("target", [9, 2700, 40000, (1 << 20) + 60000])
def test_triangle_walk_launches(target):
    import torch
    from paper_2308_08410_amd import binding as B

    dev = torch.device("cuda", 0)
    xy, tris, inner, fib, _ = gi.annulus_mesh(target)
    rng = np.random.Generator(np.random.PCG64(9))
    f32 = lambda x: torch.as_tensor(np.ascontiguousarray(x, np.float32), device=dev)
    rn = torch.as_tensor(rng.choice(inner, min(8, len(inner)), replace=False).astype(np.int32), device=dev)
    D, vs, rt = f32(gi.fibre_tensor2(fib)), f32(rng.uniform(0.7, 1.3, len(xy))), f32(rng.uniform(0, 20, len(rn)))
    g = f32(rng.uniform(0, 1, len(xy)))
    plan = B.TriPlan(xy, tris)
    T, _ = B.tri_forward(plan, D, vs, rn, rt)
    _, _, drt = B.tri_backward(plan, D, vs, rn, rt, T, g, want_D=False)
    info = B.tri_backward_info(plan)
    want = float(g.double().sum())
    assert abs(float(drt.double().sum()) - want) <= 1e-4 * want, info
    assert info["levels"] >= 1 and (info["sweeps"] > 0) == (info["cyclic"] > 0)
    plan.close()


def test_long_list_of_cycles():
    """Uniform scales on a fine slice: a cycle near a root leaves most vertices to the
    sweeps, a list that launches sweep (the sweeps end at 1e-7 of the largest lambda and
    contract in some 560, 35 times that in the sum)."""
    import torch
    from paper_2308_08410_amd import binding as B

    dev = torch.device("cuda", 0)
    p = gi.annulus_problem(250_000)
    f32 = lambda x: torch.as_tensor(np.ascontiguousarray(x, np.float32), device=dev)
    rn = torch.as_tensor(p.root_node, device=dev)
    D, vs, rt = f32(p.D), f32(np.ones(p.n_v)), f32(p.root_t + 2.0)
    g = f32(np.random.Generator(np.random.PCG64(4)).uniform(0, 1, p.n_v))
    plan = B.TriPlan(p.xyz, p.tets)
    T, _ = B.tri_forward(plan, D, vs, rn, rt)
    _, _, drt = B.tri_backward(plan, D, vs, rn, rt, T, g, want_D=False)
    info = B.tri_backward_info(plan)
    print(f"[sweeps] {info}", flush=True)
    want = float(g.double().sum())
    assert abs(float(drt.double().sum()) - want) <= 1e-4 * want, info
    assert info["cyclic"] > 32768 and info["sweeps"] % 32 == 0
    plan.close()
