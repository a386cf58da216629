"""Border choice among three 2D elements whose squared distances form a chain of
ties (neighbours within 1e-14, the ends not): the rule is applied in ascending
element order, also where the oriented box of the first element drops it from the
first round, whatever the size of the call."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _cup(gap):
    """Order 2, top edge y = 0.3 x^2 - gap on [-2, 2]: (0, 1) lies outside it at
    distance 1 + gap, inside its boxes."""
    x = np.array([-2.0, 0.0, 2.0])
    top = 0.3 * x * x - gap
    bot = np.full(3, -4.0)
    return np.tile(x, (3, 1)), np.stack([bot, 0.5 * (bot + top), top])


def _turned_square(gap):
    """Side 4, turned: (0, 1) lies off the middle of an edge at distance 1 + gap,
    inside the axis-aligned box and outside the oriented one."""
    n, t = np.array([0.6, 0.8]), np.array([-0.8, 0.6])
    c = np.array([0.0, 1.0]) - (3.0 + gap) * n
    u = np.array([-2.0, 0.0, 2.0])
    P = c + u[None, :, None] * t + u[:, None, None] * n  # row: along n
    return P[..., 0], P[..., 1]


@pytest.mark.parametrize("order,own", [((0, 1, 2), 2), ((0, 2, 1), 1), ((1, 0, 2), 0),
                                       ((2, 0, 1), 0)])
def test_chain_of_ties(order, own):
    from paper_1811_04891_amd import findpts as fp
    print(f"case: chain of ties, elements {order}", flush=True)
    dev = torch.device("cuda:0")
    # squared distances 1 + 1.5e-14 (turned), 1 + 0.75e-14, 1
    parts = [_turned_square(7.5e-15), _cup(3.75e-15), _cup(0.0)]
    x = np.stack([parts[k][0] for k in order])
    y = np.stack([parts[k][1] for k in order])
    om = oracle.OracleMesh2(x.ravel(), y.ravel(), 2, TOL)
    p = np.array([[0.0, 1.0]])
    oc, oe, _, od = om.findpts(p)
    assert oc[0] == 1 and oe[0] == own
    n = 65537
    h = fp.findpts2_setup(torch.as_tensor(x.ravel().copy()).to(dev),
                          torch.as_tensor(y.ravel().copy()).to(dev), 2, tol=TOL, max_points=n)
    for k in (1, 5, n):
        code, el, _, d2 = fp.findpts2(h, torch.as_tensor(np.tile(p, (k, 1))).to(dev))
        torch.cuda.synchronize()
        assert torch.all(code == 1)
        assert torch.all(el == own), (k, el[0].item())
        assert np.max(np.abs(d2.cpu().numpy() - od[0])) <= 2e-15
    h.free()
