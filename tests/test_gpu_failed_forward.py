"""A synchronous forward that ends with an input error leaves the caller's output as it
was, whether its rounds are one launch or many, also where the output is the guess that
orders a cold solve."""
import numpy as np
import pytest

import gbp_inputs as gi
from test_gpu_parity import B, _dev, i32, t32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hold", [0.0, 1.0])
@pytest.mark.parametrize("fault", ["root", "onset", "tensor", "spd", "scale"])
def test_output_is_kept(fault, hold):
    dev = _dev()
    p = gi.cube_problem(8)
    D, vs = p.D.astype(np.float32).copy(), np.ones(p.n_v, np.float32)
    rn, rt = p.root_node.copy(), p.root_t.astype(np.float32).copy()
    if fault == "root":
        rn[-1] = p.n_v
    elif fault == "onset":
        rt[-1] = np.nan
    elif fault == "tensor":
        D[5, 1] = np.inf
    elif fault == "spd":
        D[7] *= -1
    else:
        vs[3] = 0.0
    plan = B().Plan(p.xyz, p.tets)
    B().set_hold(plan, hold)
    B().set_warm_order(plan, True)
    kept = torch.linspace(1, 2, p.n_v, device=dev)
    for T_init in (None, True):
        out = kept.clone()
        with pytest.raises(B().GbpError):
            B().eikonal_forward(plan, t32(D, dev), t32(vs, dev), i32(rn, dev), t32(rt, dev),
                                T_init=out if T_init else None, out=out)
        assert torch.equal(out, kept), (fault, hold, T_init)
    T, st = B().eikonal_forward(plan, t32(p.D, dev), None, i32(p.root_node, dev), t32(p.root_t, dev))
    assert st["converged"] and st["unreached"] == 0 and bool(torch.isfinite(T).all())
