"""Small two-dimensional calls (16 lanes per point) and calls just past their
limit (the element-grouped path): the same points through both paths against
the CPU oracle, under the parity rules of the other GPU tests."""
import numpy as np
import pytest
import torch

import oracle
import workloads as w
from parity import compare_eval, compare_locate

pytestmark = pytest.mark.gpu

TOL = 1e-12
LIMIT = 65536  # the largest call that takes 16 lanes per point


def _points(n, seed):
    """Around a ring 0.5 <= rho <= 1: inside, off its walls, outside."""
    rng = np.random.default_rng(seed)
    rho = np.sqrt(rng.uniform(0.24, 1.02, n))
    th = rng.uniform(0.0, 2.0 * np.pi, n)
    p = np.stack([rho * np.cos(th), rho * np.sin(th)], 1)
    p[0] = np.nan
    return p


def _call(fp, h, pts, tags, fields):
    code, el, rs, d2 = fp.findpts2(h, pts, tags)
    out = fp.findpts2_eval(h, code, el, rs, fields)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (code, el, rs, d2)], out.cpu().numpy()


@pytest.mark.parametrize("N", list(range(1, 16)))
def test_both_paths_match_oracle(N):
    from paper_1811_04891_amd import findpts as fp
    print(f"case: 2D small calls and a grouped call, order {N}", flush=True)
    dev = torch.device("cuda:0")
    mesh = w.annulus2d_mesh(2, 10, N=N)
    fields = [mesh.x.clone(), mesh.x * mesh.y, mesh.y.clone()]
    n = LIMIT + 1
    pts = _points(n, N)
    md = mesh.to(dev)
    h = fp.findpts2_setup(md.x, md.y, N, tol=TOL, max_points=n)
    dp, df = torch.as_tensor(pts).to(dev), [f.to(dev) for f in fields]
    fp.findpts2_stats(h, reset=True)
    big, big_out = _call(fp, h, dp, None, df)
    cands = fp.findpts2_stats(h, reset=True)[2]
    cuts = [0, 1, 4, 9, 1000, 20000, n]
    parts = [_call(fp, h, dp[a:b].contiguous(), None, df)
             for a, b in zip(cuts[:-1], cuts[1:])]
    assert fp.findpts2_stats(h)[2] == cands
    small = [np.concatenate([p[0][k] for p in parts]) for k in range(4)]
    small_out = np.concatenate([p[1] for p in parts], axis=1)
    om = oracle.OracleMesh2.from_mesh(mesh, TOL)
    _, hs = om.bbox()
    sub = np.arange(0, n, 32)
    ref = om.findpts(pts[sub])
    hf = [f.numpy() for f in fields]
    assert np.array_equal(big[0], small[0])
    assert np.mean(big[1] != small[1]) <= 1e-3  # ties between border elements only
    for res, out in ((big, big_out), (small, small_out)):
        compare_locate(om, pts[sub], [a[sub] for a in res], ref, hs, TOL)
        compare_eval(out[:, sub], om.eval(res[0][sub], res[1][sub], res[2][sub], hf), hf)
    h.free()


@pytest.mark.parametrize("shape", [(1, 8), (16, 64), (41, 100)])
def test_crowded_and_many_elements(shape):
    """A grouped call on few elements (ranks in LDS) and just past their limit."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: 2D grouped call on {shape}", flush=True)
    dev = torch.device("cuda:0")
    m = w.annulus2d_mesh(*shape, N=3)
    n = LIMIT + 2049
    pts = _points(n, 11)
    md = m.to(dev)
    h = fp.findpts2_setup(md.x, md.y, 3, tol=TOL, max_points=n)
    fields = [m.x * m.y, m.y]
    res, out = _call(fp, h, torch.as_tensor(pts).to(dev), None, [f.to(dev) for f in fields])
    om = oracle.OracleMesh2.from_mesh(m, TOL)
    _, hs = om.bbox()
    sub = np.arange(0, n, 16)
    compare_locate(om, pts[sub], [a[sub] for a in res], om.findpts(pts[sub]), hs, TOL)
    hf = [f.numpy() for f in fields]
    compare_eval(out, om.eval(res[0], res[1], res[2], hf), hf)
    h.free()


@pytest.mark.parametrize("N", [1, 4, 7, 11])
@pytest.mark.parametrize("nf", [1, 9])
def test_small_call_sessions_and_field_counts(N, nf):
    """Three overlapping rings with the distance field, tagged and untagged
    points, passes shorter than the call, one and two field launches."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: 2D small call, sessions, order {N}, {nf} fields", flush=True)
    dev = torch.device("cuda:0")
    ms = [w.annulus2d_mesh(2, 10, 0.5, 0.8, N=N), w.annulus2d_mesh(2, 12, 0.7, 1.0, N=N),
          w.annulus2d_mesh(1, 11, 0.6, 0.9, N=N)]
    x, y = (torch.cat([getattr(m, c) for m in ms]) for c in "xy")
    sess = torch.cat([torch.full((m.E,), i, dtype=torch.int32) for i, m in enumerate(ms)])
    rho = torch.sqrt(x * x + y * y)
    s3 = sess[:, None, None]
    delta = torch.where(s3 == 0, 0.8 - rho, torch.where(s3 == 1, rho - 0.7, 0.1 * rho)).contiguous()
    mesh = w.Mesh2("three", N, x, y, sess, delta)
    fields = [x * (0.5 + k) + y * y for k in range(nf)]
    n = 1501
    pts = _points(n, 5)
    tags = (np.arange(n) % 4 - 1).astype(np.int32)
    md = mesh.to(dev)
    h = fp.findpts2_setup(md.x, md.y, N, tol=TOL, elem_session=md.session, delta=md.delta,
                          max_points=700)
    res, out = _call(fp, h, torch.as_tensor(pts).to(dev), torch.as_tensor(tags).to(dev),
                     [f.to(dev) for f in fields])
    om = oracle.OracleMesh2.from_mesh(mesh, TOL)
    _, hs = om.bbox()
    st = compare_locate(om, pts, res, om.findpts(pts, tags), hs, TOL)
    assert st["inside"] > 500
    hf = [f.numpy() for f in fields]
    compare_eval(out, om.eval(res[0], res[1], res[2], hf), hf)
    h.free()
