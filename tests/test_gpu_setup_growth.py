"""Updates whose hash lists outgrow the room that the setup made for them: the
lists hold exactly the elements whose box meets the cell, and the handle answers
as one set up on the new coordinates."""
import numpy as np
import pytest
import torch

import workloads as w

pytestmark = pytest.mark.gpu


def _cells(fp, h):
    """Every list entry by the boxes and the grid, on the host; returns the count.

    A cell index is decided where it is further than 1e-10 from a border (the
    product that the device rounds is at most 1024, so it is off by 1e-13)."""
    b = fp.findpts_get_bbox(h)[0].reshape(-1, 3, 2)
    nc, lo, dx, (ncell, nnz, longest) = fp.findpts_get_hash(h)
    off, cel = fp.findpts_get_cells(h)
    assert ncell == np.prod(nc) and len(off) == ncell + 1
    assert off[0] == 0 and off[-1] == nnz == len(cel)
    assert np.all(np.diff(off) >= 0) and longest == np.max(np.diff(off))
    top = np.array(nc) - 1

    def box(shift):
        u = (b - lo[:, None]) / dx[:, None] + np.array([-shift, shift])
        return np.clip(np.floor(u).astype(int), 0, top[:, None])

    def lists(r):
        out = [set() for _ in range(ncell)]
        for e, ((i0, i1), (j0, j1), (k0, k1)) in enumerate(r):
            for k in range(k0, k1 + 1):
                for j in range(j0, j1 + 1):
                    for i in range(i0, i1 + 1):
                        out[i + nc[0] * (j + nc[1] * k)].add(e)
        return out

    must, may = lists(box(-1e-10)), lists(box(1e-10))
    for c in range(ncell):
        got = cel[off[c]:off[c + 1]]
        assert np.all(np.diff(got) > 0)
        assert must[c] <= set(got.tolist()) <= may[c], (c, got, must[c], may[c])
    assert sum(map(len, must)) >= 0.9 * nnz  # (few entries are undecided)
    return nnz


def _sheared(m, by):
    out = w.box_mesh(5, 4, 3, N=m.N)
    out.x = m.x + by * m.y
    out.y = m.y + by * m.z
    return out


@pytest.mark.parametrize("N", [1, 4, 7, 12, 15])
def test_lists_outgrow_their_room(N):
    from paper_1811_04891_amd import findpts as fp
    print(f"case: updates with growing cell lists, order {N}", flush=True)
    dev = torch.device("cuda:0")
    box = w.box_mesh(5, 4, 3, N=N)
    steps = [w.annulus_mesh(2, 10, 3, N=N), box, _sheared(box, 0.7), _sheared(box, 1.9), box]
    first = steps[0].to(dev)
    h = fp.findpts_setup(first.x, first.y, first.z, N, max_points=512)
    room = _cells(fp, h)
    grown = 0
    for m in steps[1:]:
        d = m.to(dev)
        fp.findpts_update(h, d.x, d.y, d.z)
        nnz = _cells(fp, h)
        grown += nnz > room
        room = max(room, nnz)
        rng = np.random.default_rng(5)
        ext = [(float(c.min()), float(c.max())) for c in (m.x, m.y, m.z)]
        p = torch.tensor(np.stack([rng.uniform(a, b, 500) for a, b in ext], 1), device=dev)
        f = fp.findpts_setup(d.x, d.y, d.z, N, max_points=512)
        assert _cells(fp, f) == nnz
        for got, want in zip(fp.findpts(h, p), fp.findpts(f, p)):
            np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
        f.free()
    assert grown >= 2
    h.free()
