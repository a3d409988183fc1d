"""Teams of fewer blocks than their launch has, and teams that blocks join in the middle
of a solve: what one, two or three blocks compute, and what a team founded by one or two
ends with, is what the whole launch computes.  Times (rounds are Jacobi steps) and the
walk's lambdas (fixed sums) are the same to the bit; sweeps in place end within their
tolerance of one another.  Two plans on two streams, and a plan beside a stream that
fills the device, end with the same numbers too."""
import numpy as np
import pytest

import gbp_inputs as gi
from conftest import rng
from test_gpu_parity import B, _dev, i32, t32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LIMITS = [(0, 1), (0, 2), (0, 3), (1, 0), (1, 3), (2, 9), (3, 0)]


def check_sizes(plan, founders, most, full):
    n0, n1 = B().team(plan)
    assert n0 <= n1 and (not founders or n0 <= founders) and (not most or n1 <= most), (n0, n1, founders, most)
    if not full:
        return
    assert n1 > n0 if founders and (not most or most > founders) else n1 >= 1, (n0, n1, founders, most)


def cube(cells, uniform):
    r = rng(cells)
    xyz, tets = gi.kuhn_cube(cells, length=30.0)
    xyz = gi.jitter_nodes(xyz, 30.0 / cells, 0.1, 3)
    z = xyz[tets].mean(axis=1)[:, 2] / 30.0
    a = np.pi * (z - 0.5) * 1.3
    D = gi.fibre_tensor(np.stack([np.cos(a), np.sin(a), np.zeros_like(a)], 1))
    vs = np.ones(len(xyz)) if uniform else r.uniform(0.7, 1.3, len(xyz))
    dev = _dev()
    rn = r.choice(len(xyz), 5, replace=False)
    return (B().Plan(xyz, tets), t32(D, dev), t32(vs, dev), i32(rn, dev), t32(r.uniform(0, 5, 5), dev),
            t32(r.uniform(0, 1, len(xyz)), dev))


@pytest.mark.parametrize("cells,uniform", [(24, False), (40, False), (60, True)])
def test_tet_teams(cells, uniform):
    plan, D, vs, rn, rt, g = cube(cells, uniform)
    a = (plan, D, vs, rn, rt)
    T0, st0 = B().eikonal_forward(*a)
    n0, n1 = B().team(plan)
    assert n0 == n1 >= 64
    G0 = B().eikonal_backward(*a, T0, g)
    info0 = B().backward_info(plan)
    for founders, most in LIMITS:
        B().set_team(plan, founders, most)
        T, st = B().eikonal_forward(*a)
        check_sizes(plan, founders, most, True)
        assert torch.equal(T, T0) and {**st, "updates": 0} == {**st0, "updates": 0}, (founders, most)
        G = B().eikonal_backward(*a, T, g)
        info = B().backward_info(plan)
        check_sizes(plan, founders, most, info["cyclic"] > 0)   # the sweeps' team, if there was one
        assert (info["levels"], info["cyclic"]) == (info0["levels"], info0["cyclic"])
        for x, y in zip(G, G0):
            assert torch.equal(x, y) if info["cyclic"] == 0 else float((x - y).norm()) <= 1e-5 * float(y.norm())
    # an enqueue-only backward that leaves most of the mesh to the sweeps
    lv, gs = max(2, info0["levels"] // 2), 400
    for founders, most in [(0, 0), (1, 0), (0, 2)]:
        B().set_team(plan, founders, most)
        G = B().eikonal_backward_async(*a, T0, g, lv, gs)
        check_sizes(plan, founders, most, True)
        assert B().plan_status(plan)["backward_settled"], (founders, most)
        for x, y in zip(G, G0):
            assert float((x - y).norm()) <= 1e-4 * float(y.norm()), (founders, most)
    with pytest.raises(B().GbpError):
        B().set_team(plan, -1, 0)


@pytest.mark.parametrize("target", [6000, 40000])
def test_triangle_teams(target):
    dev, r = _dev(), rng(target)
    xy, tris, inner, fib, _ = gi.annulus_mesh(target)
    plan = B().TriPlan(xy, tris)
    a = (plan, t32(gi.fibre_tensor2(fib), dev), t32(r.uniform(0.7, 1.3, len(xy)), dev),
         i32(r.choice(inner, 8, replace=False), dev), t32(r.uniform(0, 20, 8), dev))
    T0, st0 = B().tri_forward(*a)
    assert B().team(plan)[0] == B().team(plan)[1] >= 32
    for founders, most in LIMITS:
        B().set_team(plan, founders, most)
        T, st = B().tri_forward(*a)
        check_sizes(plan, founders, most, True)
        assert torch.equal(T, T0) and {**st, "updates": 0} == {**st0, "updates": 0}, (founders, most)
    with pytest.raises(B().GbpError):
        B().set_team(plan, 0, -1)


def test_triangle_walk_team():
    """Past 2^20 vertices a team walks the triangles' levels too."""
    dev, r = _dev(), rng(1)
    xy, tris, inner, fib, _ = gi.annulus_mesh((1 << 20) + 60000)
    plan = B().TriPlan(xy, tris)
    a = (plan, t32(gi.fibre_tensor2(fib), dev), t32(r.uniform(0.7, 1.3, len(xy)), dev),
         i32(r.choice(inner, 8, replace=False), dev), t32(r.uniform(0, 20, 8), dev))
    g = t32(r.uniform(0, 1, len(xy)), dev)
    T, _ = B().tri_forward(*a)
    _, _, drt0 = B().tri_backward(*a, T, g, want_D=False)
    levels = B().tri_backward_info(plan)["levels"]
    for founders, most in [(0, 3), (1, 0)]:
        B().set_team(plan, founders, most)
        _, _, drt = B().tri_backward(*a, T, g, want_D=False)
        assert B().tri_backward_info(plan)["levels"] == levels
        assert float((drt - drt0).abs().max()) <= 1e-5 * float(drt0.abs().max())


def test_two_streams():
    plans = [cube(30, False), cube(34, False)]
    want = []
    for p in plans:
        T, _ = B().eikonal_forward(*p[:5])
        G = B().eikonal_backward(*p[:5], T, p[5])
        want.append((T, *G))
    streams = [torch.cuda.Stream() for _ in plans]
    big = torch.zeros(1 << 28, device=_dev())
    torch.cuda.synchronize()
    for busy in (False, True):
        for _ in range(3):
            got = []
            if busy:
                for _ in range(20):
                    big.add_(1.0)
            for p, s in zip(plans, streams):
                with torch.cuda.stream(s):
                    T = B().eikonal_forward_async(*p[:5], 200)
                    G = B().eikonal_backward_async(*p[:5], T, p[5], 400, 0)
                    got.append((T, *G))
            torch.cuda.synchronize()
            for p, w, g in zip(plans, want, got):
                st = B().plan_status(p[0])
                assert st["forward_converged"] and st["backward_settled"]
                for x, y in zip(g, w):
                    assert torch.equal(x, y)


@pytest.mark.parametrize("cells", [45, 63, 64])   # a team's list on both sides of 65,536; launches
def test_long_lists(cells):
    """An enqueue-only backward whose levels end early leaves long lists to the sweeps,
    which end where the walk does: each is exact once its children are, so as many sweeps
    as there are levels suffice."""
    plan, D, vs, rn, rt, g = cube(cells, False)
    a = (plan, D, vs, rn, rt)
    T, _ = B().eikonal_forward(*a)
    G0 = B().eikonal_backward(*a, T, g)
    info = B().backward_info(plan)
    for levels in (info["levels"] // 3, 2):
        G = B().eikonal_backward_async(*a, T, g, levels, 2 * info["levels"] + 64)
        assert B().plan_status(plan)["backward_settled"]
        for x, y in zip(G, G0):
            assert float((x - y).norm()) <= 1e-5 * float(y.norm()), levels


@pytest.mark.parametrize("cells", [66, 102])     # one XCD's blocks, all
def test_walk_takes_its_blocks(cells):
    """Past 2^18 vertices (sweeps are launches, so the walk's team is the last): the least
    level_blocks leaves the walk as it is."""
    plan, D, vs, rn, rt, g = cube(cells, False)
    a = (plan, D, vs, rn, rt)
    T, _ = B().eikonal_forward(*a)
    want = []
    for level_blocks in (2048, 16):
        B().set_launch(plan, 16, 2048, level_blocks)
        _, dvs, drt = B().eikonal_backward(*a, T, g, want_D=False)
        want.append((B().team(plan), dvs, drt))
    assert want[0][0] == want[1][0] and want[0][0][1] >= 32, want
    if B().backward_info(plan)["cyclic"] == 0:
        assert torch.equal(want[0][1], want[1][1]) and torch.equal(want[0][2], want[1][2])
