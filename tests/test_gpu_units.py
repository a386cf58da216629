"""Work units: one crowded element, meshes whose element count is around a scan
tile (1024), elements just below and above the unit sizes, empty runs; points in
random order, both entry points, against the oracle and the field's polynomial."""
import numpy as np
import pytest
import torch

import oracle
import workloads as w
from parity import compare_eval, compare_locate

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _mesh_points(m, counts, seed):
    """counts[e] points strictly inside element e of a box mesh, shuffled; also
    their elements."""
    rng = np.random.default_rng(seed)
    e = np.repeat(np.arange(m.E), counts)
    X = np.stack([m.x.numpy(), m.y.numpy(), m.z.numpy()], 1).reshape(m.E, 3, -1)
    lo, hi = X.min(2)[e], X.max(2)[e]
    p = lo + (hi - lo) * rng.uniform(0.05, 0.95, (len(e), 3))
    q = rng.permutation(len(e))
    return p[q], e[q]


def _counts(E, seed):
    rng = np.random.default_rng(seed)
    c = rng.integers(0, 80, E)
    c[rng.random(E) < 0.5] = 0
    for k, v in enumerate((63, 64, 65, 127, 128, 129, 144, 255, 256, 257, 700, 5000)):
        c[(k * 83 + 1) % E] = v
    return c


@pytest.mark.parametrize("N", [3, 7, 9])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 3, 3), (11, 31, 3), (16, 16, 4), (41, 5, 5),
                                   (32, 32, 3)])
def test_units_of_all_sizes(N, shape):
    from paper_1811_04891_amd import findpts as fp
    E = shape[0] * shape[1] * shape[2]
    print(f"case: units, order {N}, {E} elements", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(*shape, N=N)
    counts = np.array([30011]) if E == 1 else _counts(E, E)
    pts, own = _mesh_points(m, counts, N)
    if E == 27:
        pts, own = np.tile(pts, (3, 1)), np.tile(own, 3)
    n = len(pts)
    assert n > 16384  # past the small calls
    fields, _ = w.poly_fields(m, 3, degree=min(N, 3), seed=1)
    md = m.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, tol=TOL, max_points=n)
    code, el, rst, d2 = fp.findpts(h, torch.as_tensor(pts).to(dev))
    out = fp.findpts_eval(h, code, el, rst, [f.to(dev) for f in fields])
    torch.cuda.synchronize()
    res = [t.cpu().numpy() for t in (code, el, rst, d2)]
    assert np.all(res[0] == 0) and np.array_equal(res[1], own)
    sub = np.arange(0, n, max(1, n // 1500))
    om = oracle.OracleMesh.from_mesh(m, TOL)
    _, hs = om.bbox()
    compare_locate(om, pts[sub], [a[sub] for a in res], om.findpts(pts[sub]), hs, TOL)
    hf = [f.numpy() for f in fields]
    exp = om.eval(res[0], res[1], res[2], hf)
    compare_eval(out.cpu().numpy(), exp, hf)
    # interpolation without the handle's workspace
    out2 = torch.empty_like(out)
    fp.findpts_eval_noalloc(h, code, el, rst, [f.to(dev) for f in fields], out2)
    torch.cuda.synchronize()
    compare_eval(out2.cpu().numpy(), exp, hf)
    h.free()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,n", [((4, 4, 4), (1 << 21) + 37), ((17, 16, 16), (1 << 20) + 37)])
def test_staged_and_direct_interpolation_agree(shape, n, prec):
    """A pass just past the staged path's smallest (few and many elements) and
    the same points in two direct calls: identical bytes, not-found included."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: staged and direct interpolation, {shape}, {n} points, {prec}", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(*shape, N=3).to(dev)
    fields = [m.x * m.y, m.z - 0.5 * m.x]
    g = torch.Generator(device=dev).manual_seed(3)
    code = torch.zeros(n, dtype=torch.int32, device=dev)
    code[::7] = 2
    el = torch.randint(0, m.E, (n,), generator=g, device=dev, dtype=torch.int32)
    rst = 2.0 * torch.rand((n, 3), generator=g, device=dev, dtype=torch.float64) - 1.0
    h = fp.findpts_setup(m.x, m.y, m.z, 3, tol=TOL, max_points=n,
                         precision=fp.FP_PREC_MIXED if prec == "mixed" else fp.FP_PREC_FP64)
    whole = fp.findpts_eval(h, code, el, rst, fields)
    cut = n // 2
    parts = [fp.findpts_eval(h, code[a:b].contiguous(), el[a:b].contiguous(),
                             rst[a:b].contiguous(), fields) for a, b in ((0, cut), (cut, n))]
    torch.cuda.synchronize()
    both = torch.cat(parts, dim=1)
    assert torch.equal(whole.view(torch.int64)[:, code == 0], both.view(torch.int64)[:, code == 0])
    assert torch.isnan(whole[:, code == 2]).all() and torch.isnan(both[:, code == 2]).all()
    h.free()


def test_more_elements_than_a_large_scan_tile_switch():
    """Over 2^20 elements (the scans then take larger tiles): known owners and a
    linear field, through both interpolation entry points."""
    from paper_1811_04891_amd import findpts as fp
    print("case: 1,100,000 elements of order 1", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(110, 100, 100, N=1)
    rng = np.random.default_rng(2)
    own = np.concatenate([rng.integers(0, m.E, 30000), np.full(700, m.E - 1), np.full(300, 0)])
    X = np.stack([m.x.numpy(), m.y.numpy(), m.z.numpy()], 1).reshape(m.E, 3, -1)[own]
    pts = X.min(2) + (X.max(2) - X.min(2)) * rng.uniform(0.05, 0.95, (len(own), 3))
    md = m.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, 1, tol=TOL, max_points=len(own))
    dp = torch.as_tensor(pts).to(dev)
    code, el, rst, _ = fp.findpts(h, dp)
    f = [(md.x + 2.0 * md.y - md.z).contiguous()]
    out = fp.findpts_eval(h, code, el, rst, f)
    out2 = torch.empty_like(out)
    fp.findpts_eval_noalloc(h, code, el, rst, f, out2)
    torch.cuda.synchronize()
    assert torch.all(code == 0) and np.array_equal(el.cpu().numpy(), own)
    exact = dp[:, 0] + 2.0 * dp[:, 1] - dp[:, 2]
    # r is found to 1e-12 of an element of at most 0.01; sums of a few terms of at most 3
    assert torch.max(torch.abs(out[0] - exact)) <= 1e-13
    assert torch.equal(out, out2)
    h.free()
