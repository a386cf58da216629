"""The matrix-core closest-node scan and the chunked Newton kernels past the small
calls, at the orders where a smaller call takes another kernel: points about
equally far from two turns of a spiral element (near ties of the start node), and
elements with more pairs than one chunk holds in mixed precision."""
import numpy as np
import pytest
import torch

import oracle
import workloads as w
from parity import compare_locate
from test_gpu_parity_more import _spiral_turn_midpoints

pytestmark = pytest.mark.gpu

TOL = 1e-12
GROUPED = 16385  # one point more than the largest small call


@pytest.mark.parametrize("N", [7, 8, 9, 10, 11, 12, 13, 14, 15])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_near_ties_between_turns(N, prec):
    """Order 11 reads the gap between its staged coordinates, orders 8 to 10 and
    12 to 14 the zeros after the element."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: spiral midway points, grouped, order {N}, {prec}", flush=True)
    dev = torch.device("cuda:0")
    mesh = w.spiral_element(N=N)
    mid = _spiral_turn_midpoints(mesh, 2000, 24)
    k = len(mid)
    assert k > 100
    pts = np.tile(mid, (GROUPED // k + 1, 1))
    md = mesh.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, tol=TOL, max_points=len(pts),
                         precision=fp.FP_PREC_MIXED if prec == "mixed" else fp.FP_PREC_FP64)
    res = [t.cpu().numpy() for t in fp.findpts(h, torch.as_tensor(pts).to(dev))]
    om = oracle.OracleMesh.from_mesh(mesh, TOL)
    _, hs = om.bbox()
    o = om.findpts(mid)
    g = [a[:k] for a in res]
    compare_locate(om, mid, g, o, hs, TOL)
    bor = (o[0] == 1) & (g[0] == 1)
    assert bor.sum() > 100
    # a start at the other turn's node would end at another distance
    assert np.all(np.abs(g[3][bor] - o[3][bor]) <= 1e-9 * o[3][bor])
    # every copy of a point gets the same answer, whatever slot it took
    for a in res:
        for c in range(1, len(pts) // k):
            assert np.array_equal(a[:k], a[c * k:(c + 1) * k])
    h.free()


@pytest.mark.parametrize("N", [5, 7, 8, 9])
def test_mixed_many_pairs_per_element(N):
    """20,003 points in two elements: many units and chunks of each."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: mixed, two crowded elements, order {N}", flush=True)
    dev = torch.device("cuda:0")
    mesh = w.annulus_mesh(1, 6, 1, N=N)
    rng = np.random.default_rng(N)
    n = 20003
    rho, th = rng.uniform(0.51, 0.99, n), rng.uniform(0.02, 2.0, n)
    pts = np.stack([rho * np.cos(th), rho * np.sin(th), rng.uniform(0.01, 0.99, n)], 1)
    md = mesh.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, tol=TOL, max_points=n,
                         precision=fp.FP_PREC_MIXED)
    res = [t.cpu().numpy() for t in fp.findpts(h, torch.as_tensor(pts).to(dev))]
    om = oracle.OracleMesh.from_mesh(mesh, TOL)
    _, hs = om.bbox()
    sub = np.arange(0, n, 7)
    st = compare_locate(om, pts[sub], [a[sub] for a in res], om.findpts(pts[sub]), hs, TOL)
    assert st["inside"] == len(sub)
    h.free()


@pytest.mark.parametrize("nf", [9, 17])
@pytest.mark.parametrize("shape", [(4, 4, 4), (17, 16, 16)])
def test_staged_interpolation_of_many_fields(shape, nf):
    """A staged pass whose fields take several launches (each reuses the staging
    room): the bytes of the direct path's halves, for every field."""
    from paper_1811_04891_amd import findpts as fp
    n = ((1 << 21) if shape == (4, 4, 4) else (1 << 20)) + 37
    print(f"case: staged interpolation, {shape}, {n} points, {nf} fields", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(*shape, N=3).to(dev)
    fields = [(m.x * (1.0 + f) + m.y * m.z - 0.1 * f).contiguous() for f in range(nf)]
    g = torch.Generator(device=dev).manual_seed(5)
    code = torch.zeros(n, dtype=torch.int32, device=dev)
    code[::11] = 2
    el = torch.randint(0, m.E, (n,), generator=g, device=dev, dtype=torch.int32)
    rst = 2.0 * torch.rand((n, 3), generator=g, device=dev, dtype=torch.float64) - 1.0
    h = fp.findpts_setup(m.x, m.y, m.z, 3, tol=TOL, max_points=n)
    whole = fp.findpts_eval(h, code, el, rst, fields)
    cut = n // 2
    both = torch.cat([fp.findpts_eval(h, code[a:b].contiguous(), el[a:b].contiguous(),
                                      rst[a:b].contiguous(), fields)
                      for a, b in ((0, cut), (cut, n))], dim=1)
    torch.cuda.synchronize()
    found = code == 0
    assert torch.equal(whole.view(torch.int64)[:, found], both.view(torch.int64)[:, found])
    assert torch.isnan(whole[:, ~found]).all() and torch.isnan(both[:, ~found]).all()
    h.free()
