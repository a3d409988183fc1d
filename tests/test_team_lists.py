"""Sizes of the lists that a team of blocks pushes into (csrc/plan.cpp): on the host, for
every team size, room for the most pushes of a share; on the GPU, a plan with one vertex
of 300 neighbours beside a slice of 250,000 takes hardly more memory than without it, and
the slice's times are the same."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import gbp_inputs as gi

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_lists_hold_every_share(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path / "lists")
    src = [os.path.join(ROOT, "paper_2308_08410_amd", "csrc", "plan.cpp"),
           os.path.join(HERE, "host_sanitize", "hip_stub.cpp"), os.path.join(HERE, "host_sanitize", "lists_driver.cpp")]
    b = subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2308_08410_amd", "csrc"),
                        *src, "-o", exe], capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "OK (0 failures)" in r.stdout, r.stdout


@pytest.mark.gpu
def test_hub_beside_a_slice():
    import torch
    from oracle import tri as O2
    from paper_2308_08410_amd import binding as B

    dev = torch.device("cuda", 0)
    t = lambda x, k=np.float32: torch.as_tensor(np.ascontiguousarray(x, k), device=dev)
    p = gi.annulus_problem(250_000)
    n, m, k = p.n_v, len(p.tets), 300
    a = 2 * np.pi * np.arange(k) / k
    hub_xy = np.concatenate([[[0.0, 0.0]], np.stack([np.cos(a), np.sin(a)], 1)]).astype(np.float32)
    hub_tri = np.stack([np.zeros(k, int), 1 + np.arange(k), 1 + (np.arange(k) + 1) % k], 1).astype(np.int32)
    xy = np.concatenate([np.asarray(p.xyz, np.float32), hub_xy + np.float32(1000)])
    tri = np.concatenate([np.asarray(p.tets, np.int32), hub_tri + n])
    D = np.concatenate([p.D, np.tile([1.0, 1.0, 0.0], (k, 1))]).astype(np.float32)
    rn, rt = np.append(p.root_node, n + 5).astype(np.int32), np.append(p.root_t, 0.25).astype(np.float32)

    def create(xy, tri):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        plan = B.TriPlan(xy, tri)
        torch.cuda.synchronize()
        return plan, free - torch.cuda.mem_get_info()[0]

    create(xy, tri)[0].close()      # the allocator's first pools
    plain, used = create(np.asarray(p.xyz, np.float32), np.asarray(p.tets, np.int32))
    with_hub, used_hub = create(xy, tri)
    assert used_hub <= used + (16 << 20), (used, used_hub)
    T0, _ = B.tri_forward(plain, t(p.D), None, t(p.root_node, np.int32), t(p.root_t))
    T1, _ = B.tri_forward(with_hub, t(D), None, t(rn, np.int32), t(rt))
    assert torch.equal(T1[:n], T0)
    To, _ = O2.solve2(hub_xy, hub_tri, D[m:], np.ones(k + 1), np.array([5]), np.array([0.25]))
    assert np.abs(T1[n:].cpu().numpy() - To).max() <= 1e-4 * To.max()
