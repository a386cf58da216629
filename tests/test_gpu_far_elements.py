"""Elements far from the origin relative to their size: their boxes are as exact as
near it, and a point that several elements hold goes to the smallest of them."""
from math import comb

import numpy as np
import pytest
import torch

import oracle
import workloads as w

pytestmark = pytest.mark.gpu


def _inverse(N):
    """Nodal values to Bernstein coefficients, in long double (the oracle's
    binary64 matrix, refined)."""
    z = np.asarray(w.gll_points(N)).astype(np.longdouble)
    u = (1 + z) / 2
    B = np.array([[comb(N, k) * u[i] ** k * (1 - u[i]) ** (N - k) for k in range(N + 1)]
                  for i in range(N + 1)])
    Y = np.asarray(oracle.bernstein_inverse(N)).reshape(N + 1, N + 1).astype(np.longdouble)
    for _ in range(4):
        Y = Y @ (2 * np.eye(N + 1, dtype=np.longdouble) - B @ Y)
    return Y


def _hulls(m, N, Y):
    """Smallest and largest Bernstein coefficient per element and axis."""
    out = []
    for c in (m.x, m.y, m.z):
        X = c.numpy().reshape(-1, N + 1, N + 1, N + 1).astype(np.longdouble)
        o = X[:, :1, :1, :1]
        b = np.einsum("ia,jb,kc,eabc->eijk", Y, Y, Y, X - o).reshape(len(X), -1)
        out += [o.ravel() + b.min(1), o.ravel() + b.max(1)]
    return np.stack(out, 1)


@pytest.mark.parametrize("far", [0.0, 1e4, 1e7])
@pytest.mark.parametrize("N", [1, 2, 4, 5, 6, 7, 8])
def test_boxes(N, far):
    from paper_1811_04891_amd import findpts as fp
    print(f"case: boxes, order {N}, {far} away", flush=True)
    dev = torch.device("cuda:0")
    m = w.annulus_mesh(2, 10, 2, 1.0, 3.0, 0.0, 2.0, N=N)
    m = w.Mesh("far", N, m.x + 0.6 * far, m.y - 0.7 * far, m.z + 0.5 * far)
    md = m.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, max_points=64)
    box, size = fp.findpts_get_bbox(h)
    h.free()
    Y = _inverse(N)
    X = np.stack([c.numpy().reshape(m.E, -1) for c in (m.x, m.y, m.z)], 1)
    assert np.array_equal(size, np.max(X.max(2) - X.min(2), 1))
    amax = np.max(np.abs(X), (1, 2))
    margin = 1e-8 * size + 1e-14 * amax
    got = box + margin[:, None] * np.array([1, -1, 1, -1, 1, -1])
    # three transforms of n1 products each, the matrix rounded, and the shift and
    # margin added at the coordinates' magnitude
    kappa = float(np.abs(Y).sum(1).max())
    tol = 3 * (N + 2) * 2.0 ** -53 * kappa ** 3 * size + 2.0 ** -51 * amax
    assert np.all(np.abs(got - _hulls(m, N, Y)) <= tol[:, None])


@pytest.mark.parametrize("N,far", [(3, 1e7), (7, 1e7), (9, 1e6), (11, 1e6), (12, 1e7), (14, 1e5),
                                   (15, 1e5)])
def test_shared_nodes_go_to_the_smallest_element(N, far):
    """Points at the mesh nodes of a turned box: every one lies in each element
    that has the node."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: order {N}, {far} element sizes away", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(3, 3, 2, (0.0, 0.0, 0.0), (3.0, 3.0, 2.0), N=N)
    X = np.stack([m.x.numpy().ravel(), m.y.numpy().ravel(), m.z.numpy().ravel()], 1)
    # distinct nodes (by position before the turn) and their smallest element
    key = np.round(X * 1e6).astype(np.int64)
    _, first, back = np.unique(key, axis=0, return_index=True, return_inverse=True)
    elem = np.arange(len(X)) // (N + 1) ** 3
    own = np.full(len(first), m.E)
    np.minimum.at(own, back.ravel(), elem)
    Q, _ = np.linalg.qr(np.random.default_rng(4).normal(size=(3, 3)))
    # every element gets the same turned and moved node
    Y = (X[first] @ Q.T + far * np.array([0.6, -0.7, 0.5]))[back.ravel()]
    md = [torch.as_tensor(np.ascontiguousarray(Y[:, c])).to(dev) for c in range(3)]
    pts = Y[first]
    n = len(pts)
    big = np.tile(pts, (16385 // n + 1, 1))
    h = fp.findpts_setup(*md, N, tol=1e-12, max_points=len(big))
    for p, o in ((pts, own), (big, np.tile(own, len(big) // n))):
        for q0 in range(0, len(p), len(p) if len(p) > 16384 else 4000):
            q = slice(q0, len(p) if len(p) > 16384 else q0 + 4000)
            code, el, _, _ = fp.findpts(h, torch.as_tensor(p[q].copy()).to(dev))
            torch.cuda.synchronize()
            assert torch.all(code == 0)
            assert np.array_equal(el.cpu().numpy(), o[q])
    h.free()
