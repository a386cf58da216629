"""Setup products at every order: element boxes and sizes against the oracle,
and the hash cells' lists (ascending, exactly the elements whose box meets the
cell, the longest one reported), after setup and after an update that needs
more list entries than the setup had room for."""
import numpy as np
import pytest
import torch

import oracle
import workloads as w

pytestmark = pytest.mark.gpu


def _check(fp, h, mesh):
    om = oracle.OracleMesh.from_mesh(mesh, 1e-12)
    ob, os_ = om.bbox()
    gb, gs = fp.findpts_get_bbox(h)
    # sizes are differences of nodes; the boxes differ by the rounding of the
    # Bernstein transform (condition up to about 1e6 at order 15, so at most
    # about 1e-9 of the coordinates), a tenth of their margin 1e-8 h_e
    assert np.allclose(gs, os_, rtol=1e-15, atol=0)
    assert np.max(np.abs(gb - ob.reshape(gb.shape)) / gs[:, None]) <= 1e-9
    nc, lo, dx, (ncell, nnz, longest) = fp.findpts_get_hash(h)
    off, cel = fp.findpts_get_cells(h)
    assert off[0] == 0 and off[-1] == nnz == len(cel) and ncell == np.prod(nc)
    assert longest == np.max(np.diff(off))
    inner = np.ones(nnz, bool)
    inner[off[:-1][np.diff(off) > 0]] = False  # the first entry of each list
    assert np.all(np.diff(cel)[inner[1:]] > 0)
    # every element is in the cells of its box's corners and centre
    b = gb.reshape(-1, 3, 2)
    for pick in range(9):
        p = np.stack([b[:, a, (pick >> a) & 1] if pick < 8 else b[:, a].mean(1)
                      for a in range(3)], 1)
        c = np.clip(np.floor((p - lo) / dx).astype(int), 0, np.array(nc) - 1)
        # (a corner within rounding of a cell border may sit in the next cell)
        frac = (p - lo) / dx - np.floor((p - lo) / dx)
        sure = np.all((frac > 1e-9) & (frac < 1 - 1e-9), axis=1)
        cell = c[:, 0] + nc[0] * (c[:, 1] + nc[1] * c[:, 2])
        for e in np.nonzero(sure)[0]:
            assert e in cel[off[cell[e]]:off[cell[e] + 1]]


@pytest.mark.parametrize("N", list(range(1, 16)))
def test_boxes_and_cells(N):
    from paper_1811_04891_amd import findpts as fp
    print(f"case: setup products, order {N}", flush=True)
    dev = torch.device("cuda:0")
    mesh = w.box_mesh(5, 4, 3, N=N)
    md = mesh.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, max_points=64)
    _check(fp, h, mesh)
    # a ring's rotated elements meet more cells than the box's
    ring = w.annulus_mesh(2, 10, 3, N=N)
    rd = ring.to(dev)
    fp.findpts_update(h, rd.x, rd.y, rd.z)
    _check(fp, h, ring)
    h.free()
