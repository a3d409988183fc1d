"""Lead weights of vertices around the 32 neighbours that are assembled at a time, and
chunks of 8 leads around their ends, against the FP64 oracle (one float32 rounding of
the result: rtol 1e-6, plus 1e-7 of the largest weight where a row nearly cancels)."""
import numpy as np
import pytest

import oracle as O
from test_gpu_parity import B, _dev, t32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def wheel(n, seed):
    """n elements around one edge: its two ends have n + 1 neighbours."""
    r = np.random.Generator(np.random.PCG64(seed))
    a = (np.arange(n) + r.uniform(-0.2, 0.2, n)) * 2 * np.pi / n
    ring = np.stack([np.cos(a), np.sin(a), r.uniform(-0.2, 0.2, n)], 1)
    xyz = np.concatenate([[[0, 0, 0.9], [0.05, 0, -1.0]], ring]).astype(np.float32)
    k = np.arange(n)
    tets = np.stack([np.zeros_like(k), np.ones_like(k), 2 + k, 2 + (k + 1) % n], 1).astype(np.int32)
    return xyz, tets[:, r.permutation(4)]


@pytest.mark.parametrize("n,leads", [(3, 1), (30, 7), (31, 8), (32, 9), (63, 16), (64, 17), (200, 12)])
def test_lead_field_windows(n, leads):
    dev = _dev()
    xyz, tets = wheel(n, n)
    r = np.random.Generator(np.random.PCG64(leads))
    e = r.normal(size=(leads, 3))
    e = (3.0 * e / np.linalg.norm(e, axis=1, keepdims=True)).astype(np.float32)
    W = B().lead_field(B().Plan(xyz, tets), t32(e, dev)).cpu().numpy().astype(np.float64)
    Wo = O.lead_field(xyz, tets, e)
    np.testing.assert_allclose(W, Wo, rtol=1e-6, atol=1e-7 * np.abs(Wo).max())
