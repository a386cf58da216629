"""Closest-node scan at very large and very small elements: coordinates scaled by
a power of two give the same elements and reference coordinates bit for bit (each
step of the method scales exactly), also where squares of distances leave
binary32's range.  Points about equally far from two turns of a spiral element,
in calls past the small ones, so that a wrong start node ends elsewhere."""
import numpy as np
import pytest
import torch

import workloads as w
from test_gpu_parity_more import _spiral_turn_midpoints

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [7, 8, 9, 10, 11, 12, 14, 15])
def test_power_of_two_scales(N):
    from paper_1811_04891_amd import findpts as fp
    print(f"case: scaled spiral, order {N}", flush=True)
    dev = torch.device("cuda:0")
    mesh = w.spiral_element(N=N)
    mid = _spiral_turn_midpoints(mesh, 2000, 24)
    n = 16384 + 333
    pts = np.tile(mid, (n // len(mid) + 1, 1))[:n]
    # a few thousand others, in and around the element
    rng = np.random.default_rng(N)
    X = np.stack([mesh.x.numpy().ravel(), mesh.y.numpy().ravel(), mesh.z.numpy().ravel()], 1)
    pts[:4000] = X[rng.integers(0, len(X), 4000)] + rng.normal(0.0, 0.03, (4000, 3))
    # inside binary32's range when squared, about its ends and far past them
    # (multiples of 3: the cells per axis come from a cube root)
    got = {}
    for k in (0, 15, -30, -51, -57, -60, -63, -66, -69, -72, -75, -78, 57, 60, 63, 66, 72):
        s = 2.0 ** k
        md = [(c * s).contiguous().to(dev) for c in (mesh.x, mesh.y, mesh.z)]
        h = fp.findpts_setup(*md, N, tol=1e-12, max_points=n)
        code, el, rst, d2 = fp.findpts(h, torch.as_tensor(pts * s).to(dev))
        torch.cuda.synchronize()
        got[k] = [code.cpu().numpy(), el.cpu().numpy(), rst.cpu().numpy(),
                  d2.cpu().numpy() / (s * s)]
        h.free()
    code = got[0][0]
    assert np.sum(code == 1) > 4000 and np.sum(code == 0) > 500
    for k, g in got.items():
        for a, b in zip(got[0], g):
            assert np.array_equal(a, b), k
