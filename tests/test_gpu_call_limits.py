"""Calls at the limits between the small kernels and the grouped ones, and one
point past them: the same points on both sides of each limit, against the oracle
and each other."""
import numpy as np
import pytest
import torch

import oracle
import workloads as w
from parity import compare_eval, compare_locate

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _ring_points(n, seed, dim):
    rng = np.random.default_rng(seed)
    rho = np.sqrt(rng.uniform(0.24, 1.02, n))
    th = rng.uniform(0.0, 2.0 * np.pi, n)
    p = [rho * np.cos(th), rho * np.sin(th), rng.uniform(-0.005, 1.005, n)]
    return np.stack(p[:dim], 1)


# orders 1 to 12 locate up to 16,384 points, above 6,144; interpolation up to 16,384,
# 8,192 (orders 10 to 12) and 4,096
@pytest.mark.parametrize("N,limit", [(2, 16384), (7, 16384), (9, 16384), (10, 8192), (12, 16384),
                                     (12, 8192), (13, 6144), (13, 4096), (15, 6144), (15, 4096)])
def test_locate_and_interpolate(N, limit):
    from paper_1811_04891_amd import findpts as fp
    print(f"case: order {N}, {limit} points and one more", flush=True)
    dev = torch.device("cuda:0")
    mesh = w.annulus_mesh(2, 10, 2, N=N)
    fields, _ = w.poly_fields(mesh, 2, degree=3, seed=N)
    pts = _ring_points(limit + 1, N, 3)
    md = mesh.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, tol=TOL, max_points=limit + 1)
    dp, df = torch.as_tensor(pts).to(dev), [f.to(dev) for f in fields]
    om = oracle.OracleMesh.from_mesh(mesh, TOL)
    _, hs = om.bbox()
    sub = np.arange(0, limit, 19)
    ref = om.findpts(pts[sub])
    hf = [f.numpy() for f in fields]
    outs = []
    for n in (limit, limit + 1):
        loc = fp.findpts(h, dp[:n].contiguous())
        out = fp.findpts_eval(h, *loc[:3], df).cpu().numpy()
        res = [t.cpu().numpy() for t in loc]
        compare_locate(om, pts[sub], [a[sub] for a in res], ref, hs, TOL)
        compare_eval(out[:, sub], om.eval(*(a[sub] for a in res[:3]), hf), hf)
        outs.append(res)
    assert np.array_equal(outs[0][0], outs[1][0][:limit])
    h.free()


@pytest.mark.parametrize("N,shape,n,nf", [
    (7, (8, 8, 8), 7325, 8),    # 512 elements: 3e7 node values lie between n and n - 1
    (7, (8, 8, 8), 3663, 16),
    (5, (9, 8, 8), 9921, 14),   # 576 elements
    (9, (9, 8, 8), 3334, 9),
    (7, (1, 1, 1), 16384, 8),   # too few elements to share
])
def test_many_fields(N, shape, n, nf):
    """A call that reads just under and over the node values from which it is
    grouped by element."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: order {N}, {shape}, {n} points, {nf} fields", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(*shape, N=N)
    fields, _ = w.poly_fields(m, nf, degree=3, seed=1)
    rng = np.random.default_rng(n)
    el = rng.integers(0, m.E, n).astype(np.int32)
    code = np.zeros(n, np.int32)
    code[::37], el[::37] = 2, -1
    rst = rng.uniform(-1, 1, (n, 3))
    md = m.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, tol=TOL, max_points=n)
    df = [f.to(dev) for f in fields]
    om = oracle.OracleMesh.from_mesh(m, TOL)
    hf = [f.numpy() for f in fields]
    ref = om.eval(code, el, rst, hf)
    args = [torch.as_tensor(a).to(dev) for a in (code, el, rst)]
    for k in (n - 1, n):
        cut = [a[:k].contiguous() for a in args]
        out = fp.findpts_eval(h, *cut, df)
        compare_eval(out.cpu().numpy(), ref[:, :k], hf)
        out2 = torch.empty_like(out)
        fp.findpts_eval_noalloc(h, *cut, df, out2)
        assert torch.equal(torch.nan_to_num(out, nan=7.0), torch.nan_to_num(out2, nan=7.0))
    h.free()


@pytest.mark.parametrize("N", [1, 3, 7, 12, 15])
@pytest.mark.parametrize("mesh,limit", [((2, 10), 40000), ((2, 10), 65536), ((50, 82), 65536)])
def test_two_dimensions(N, mesh, limit):
    """Few elements change at 40,000 points, more than 4,096 at 65,536."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: 2D order {N}, {mesh}, {limit} points and one more", flush=True)
    dev = torch.device("cuda:0")
    m = w.annulus2d_mesh(*mesh, N=N)
    fields = [m.x.clone(), m.x * m.y]
    pts = _ring_points(limit + 1, N, 2)
    md = m.to(dev)
    h = fp.findpts2_setup(md.x, md.y, N, tol=TOL, max_points=limit + 1)
    dp, df = torch.as_tensor(pts).to(dev), [f.to(dev) for f in fields]
    om = oracle.OracleMesh2.from_mesh(m, TOL)
    _, hs = om.bbox()
    sub = np.arange(0, limit, 61)
    ref = om.findpts(pts[sub])
    hf = [f.numpy() for f in fields]
    outs = []
    for n in (limit, limit + 1):
        loc = fp.findpts2(h, dp[:n].contiguous())
        out = fp.findpts2_eval(h, *loc[:3], df).cpu().numpy()
        res = [t.cpu().numpy() for t in loc]
        compare_locate(om, pts[sub], [a[sub] for a in res], ref, hs, TOL)
        compare_eval(out[:, sub], om.eval(*(a[sub] for a in res[:3]), hf), hf)
        outs.append(res)
    assert np.array_equal(outs[0][0], outs[1][0][:limit])
    h.free()
