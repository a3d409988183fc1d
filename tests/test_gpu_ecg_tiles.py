"""The ECG and its backward pass around the tiles of the kernels: blocks of 64 to 512
vertices in steps of 16, one or two tiles of 16 leads, tiles of 16 time steps and
launches of at most 8032 (32 leads) or 16096 steps, with windows that begin before the
first step, end behind the last or lie past it, and vertices that are never reached.

Tolerances: each term carries two bf16 hi/lo splits (2^-17 each, and 2^-17 for the
product left out) and the rounding of t - T at up to 100 ms, 2^-23 * 100 * slope 1/tau:
together below 2^-14 of the terms' absolute sum, for the derivative (whose slope is up to
4/tau of its size) below 2^-12."""
import numpy as np
import pytest

import oracle as O
from test_gpu_parity import B, _dev, t32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leads,steps,dt", [
    (1, 16, 16, 0.5), (15, 17, 17, 0.5), (63, 32, 33, 1.0), (65, 33, 250, 0.3), (32769, 3, 40, 2.0),
    (65600, 20, 30, 3.0), (262145, 2, 25, 4.0), (130, 32, 8032, 0.01), (70, 31, 8033, 0.01),
    (40, 2, 16097, 0.005), (129, 5, 1, 1.0), (300, 12, 20, 20.0)])
def test_ecg_tiles(n, leads, steps, dt):
    dev = _dev()
    r = np.random.Generator(np.random.PCG64(n))
    T = (r.uniform(-5, 95) + 20 * np.sort(r.random(n)) + 3 * r.random(n)).astype(np.float32)
    T[r.random(n) < 0.1] = np.inf
    if n > 200:
        T[64:160] = np.inf
        T[160:192] = 4000.0
    W = r.normal(size=(n, leads)).astype(np.float32)
    ap = dict(K0=-85.0, K1=30.0, tau=1.0, t0=-2.0, dt=dt, n_steps=steps)
    e = B().ecg_forward(t32(T, dev), t32(W, dev), B().make_ap(**ap)).cpu().numpy()
    assert np.all(np.abs(e - O.ecg_forward(T, W, ap)) <= 2.0**-14 * 200 * np.abs(W).sum(0))
    G = r.normal(size=(steps, leads)).astype(np.float32)
    d = B().ecg_backward(t32(T, dev), t32(W, dev), B().make_ap(**ap), t32(G, dev)).cpu().numpy()
    t = ap["t0"] + np.arange(steps) * dt
    size = np.array([(np.abs(W[k]) * np.abs(G)[np.abs(t - T[k]) < 7].sum(0)).sum() for k in range(min(n, 4096))])
    assert np.all(np.abs(d - O.ecg_backward(T, W, ap, G))[:4096] <= 2.0**-12 * 115 * size + 1e-6 * np.abs(W).sum(1)[:4096])
