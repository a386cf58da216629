"""Infinite and not-a-number nodal values: interpolation and the owner rule
give what the sum over the nodes gives (a node's infinity with the sign of its
weight, NaN only where a NaN node is), whatever the size of the call, against
the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads as w

pytestmark = pytest.mark.gpu

TOL = 1e-12
GROUPED = 16385  # one point more than the largest small call


def _inner_points(m, n, seed):
    """n points strictly inside elements of a box mesh (no weight is zero)."""
    rng = np.random.default_rng(seed)
    e = rng.integers(0, m.E, n)
    X = np.stack([m.x.numpy(), m.y.numpy(), m.z.numpy()], 1).reshape(m.E, 3, -1)
    lo, hi = X.min(2)[e], X.max(2)[e]
    return lo + (hi - lo) * rng.uniform(0.02, 0.98, (n, 3))


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("N", [1, 3, 7, 9, 12, 15])
def test_interpolation(N, value):
    from paper_1811_04891_amd import findpts as fp
    print(f"case: nodal value {value}, order {N}", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(4, 2, 1, N=N)
    V = (N + 1) ** 3
    f = (m.x + 2.0 * m.y - m.z).reshape(m.E, V).clone()
    # elements 0 to 4: one such node each (first row of nodes, its end, the last
    # row, the middle); the others stay finite
    for e, node in enumerate((0, N, V - 1, V - N - 1, V // 2)):
        f[e, node] = value
    f = f.contiguous()
    pts = _inner_points(m, GROUPED, N)
    md = m.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, tol=TOL, max_points=GROUPED)
    dp, df = torch.as_tensor(pts).to(dev), [f.to(dev), md.x]
    code, el, rst, _ = fp.findpts(h, dp)
    grouped = fp.findpts_eval(h, code, el, rst, df)
    small = torch.cat([fp.findpts_eval(h, code[a:b].contiguous(), el[a:b].contiguous(),
                                       rst[a:b].contiguous(), df)
                       for a, b in ((0, 1), (1, 4000), (4000, 8000), (8000, 12000),
                                    (12000, GROUPED))], dim=1)
    torch.cuda.synchronize()
    assert torch.all(code == 0)
    om = oracle.OracleMesh.from_mesh(m, TOL)
    ref = om.eval(code.cpu().numpy(), el.cpu().numpy(), rst.cpu().numpy(), [f.numpy(), m.x.numpy()])
    special = el.cpu().numpy() < 5
    assert 0 < special.sum() < GROUPED
    assert np.all(~np.isfinite(ref[0][special])) and np.all(np.isfinite(ref[0][~special]))
    for out in (grouped.cpu().numpy(), small.cpu().numpy()):
        assert np.array_equal(out[0][special], ref[0][special], equal_nan=True)
        assert np.max(np.abs(out[0][~special] - ref[0][~special])) <= 1e-13 * 5.0
        assert np.max(np.abs(out[1] - ref[1])) <= 1e-13
    h.free()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("N", [1, 3, 9, 12])
def test_distance_field(N, value):
    """Two meshes of the same box: every point is inside both.  Session 0 has
    the value at all nodes of some elements (order 1: a mesh without a
    boundary), at their first node above (where its weight's sign decides)."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: distance field with {value}, order {N}", flush=True)
    dev = torch.device("cuda:0")
    a = w.box_mesh(3, 2, 2, N=N)
    V = (N + 1) ** 3
    d0 = torch.full((a.E, V), 1.0, dtype=torch.float64)
    d0[::2, : (V if N == 1 else 1)] = value
    d0[1::2] = 3.0
    d1 = torch.full((a.E, V), 2.0, dtype=torch.float64)
    x, y, z = (torch.cat([getattr(a, c), getattr(a, c)]) for c in "xyz")
    sess = torch.cat([torch.zeros(a.E, dtype=torch.int32), torch.ones(a.E, dtype=torch.int32)])
    mesh = w.Mesh("two", N, x, y, z, sess, torch.cat([d0, d1]).reshape(x.shape).contiguous())
    pts = _inner_points(a, GROUPED, N + 20)
    md = mesh.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, tol=TOL, elem_session=md.session, delta=md.delta,
                         max_points=GROUPED)
    dp = torch.as_tensor(pts).to(dev)
    big = fp.findpts(h, dp)
    parts = [fp.findpts(h, dp[p:q].contiguous()) for p, q in ((0, 1), (1, 6000), (6000, 11000),
                                                              (11000, GROUPED))]
    torch.cuda.synchronize()
    om = oracle.OracleMesh.from_mesh(mesh, TOL)
    oc, oe, _, _ = om.findpts(pts)
    assert np.all(oc == 0)
    for code, el in ((big[0], big[1]), (torch.cat([p[0] for p in parts]),
                                        torch.cat([p[1] for p in parts]))):
        assert torch.all(code == 0)
        assert np.array_equal(el.cpu().numpy(), oe)
    h.free()
