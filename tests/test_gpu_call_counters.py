"""Counters of small calls against those of grouped calls on the same points: the
method's candidates where a cell lists more elements than one round of box tests
takes, and the pairs of first and second passes where no point is inside."""
import numpy as np
import pytest
import torch

import workloads as w

pytestmark = pytest.mark.gpu

GROUPED3, GROUPED2 = 16385, 65537  # one point past the small calls


def _copies(m, k):
    return [c.reshape(1, -1).repeat(k, 1).reshape(-1).contiguous()
            for c in ((m.x, m.y, m.z) if hasattr(m, "z") else (m.x, m.y))]


@pytest.mark.parametrize("delta", [False, True])
@pytest.mark.parametrize("copies", [31, 33, 100])
def test_long_cell_lists(copies, delta):
    """Copies of a box of two elements: each cell lists 2 k or k of them."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: {copies} copies, distance field {delta}", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(2, 1, 1, N=3)
    md = [c.to(dev) for c in _copies(m, copies)]
    sess = torch.arange(copies, dtype=torch.int32).repeat_interleave(2).to(dev)
    h = fp.findpts_setup(*md, 3, max_points=GROUPED3, elem_session=sess,
                         delta=torch.ones_like(md[0]) if delta else None)
    pts = torch.as_tensor(np.random.default_rng(copies).uniform(0.01, 0.99, (GROUPED3, 3))).to(dev)
    fp.findpts_stats(h, reset=True)
    big = fp.findpts(h, pts)
    want = fp.findpts_stats(h, reset=True)
    small = [fp.findpts(h, pts[a:b].contiguous()) for a, b in ((0, 1), (1, 9000), (9000, GROUPED3))]
    got = fp.findpts_stats(h, reset=True)
    assert want[2] == got[2] == GROUPED3
    assert want[3] >= copies * GROUPED3 and got[3] == want[3]
    assert torch.equal(torch.cat([s[1] for s in small]), big[1])
    assert torch.all(big[1] < 2)  # the first copy holds every point
    h.free()


@pytest.mark.parametrize("delta", [False, True])
@pytest.mark.parametrize("copies", [7, 9, 40])
def test_long_cell_lists_2d(copies, delta):
    from paper_1811_04891_amd import findpts as fp
    print(f"case: 2D, {copies} copies, distance field {delta}", flush=True)
    dev = torch.device("cuda:0")
    m = w.box2d_mesh(2, 1, N=3)
    md = [c.to(dev) for c in _copies(m, copies)]
    sess = torch.arange(copies, dtype=torch.int32).repeat_interleave(2).to(dev)
    h = fp.findpts2_setup(*md, 3, max_points=GROUPED2, elem_session=sess,
                          delta=torch.ones_like(md[0]) if delta else None)
    pts = torch.as_tensor(np.random.default_rng(copies).uniform(0.01, 0.99, (GROUPED2, 2))).to(dev)
    fp.findpts2_stats(h, reset=True)
    big = fp.findpts2(h, pts)
    want = fp.findpts2_stats(h, reset=True)
    small = [fp.findpts2(h, pts[a:b].contiguous())
             for a, b in ((0, 1), (1, 40000), (40000, GROUPED2))]
    got = fp.findpts2_stats(h, reset=True)
    assert want[2] >= copies * GROUPED2 and got[2] == want[2]
    assert torch.equal(torch.cat([s[1] for s in small]), big[1])
    h.free()


@pytest.mark.parametrize("N", [2, 7, 9, 12])
def test_first_and_second_pass_pairs(N):
    """Points beside a ring, inside its elements' axis-aligned boxes: some lie in
    oriented boxes too, some in none (their whole set is then solved in the
    first pass)."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: pairs of both passes, order {N}", flush=True)
    dev = torch.device("cuda:0")
    m = w.annulus_mesh(2, 6, 1, N=N)
    md = m.to(dev)
    h = fp.findpts_setup(md.x, md.y, md.z, N, max_points=GROUPED3)
    rng = np.random.default_rng(N)
    rho = np.where(rng.random(GROUPED3) < 0.5, rng.uniform(0.3, 0.49, GROUPED3),
                   rng.uniform(1.01, 1.1, GROUPED3))
    th = rng.uniform(0.0, 2.0 * np.pi, GROUPED3)
    pts = torch.as_tensor(np.stack([rho * np.cos(th), rho * np.sin(th),
                                    rng.uniform(0.1, 0.9, GROUPED3)], 1)).to(dev)
    fp.findpts_stats(h, reset=True)
    code = fp.findpts(h, pts)[0]
    want = fp.findpts_stats(h, reset=True, first_pass=True)
    for a, b in ((0, 3000), (3000, 6000), (6000, 9000), (9000, 12000), (12000, GROUPED3)):
        fp.findpts(h, pts[a:b].contiguous())
    got = fp.findpts_stats(h, reset=True, first_pass=True)
    assert torch.all(code != 0) and torch.any(code == 1)
    assert 0 < want[4] < want[0]  # both passes have pairs
    assert (got[0], got[2], got[3], got[4]) == (want[0], want[2], want[3], want[4])
    h.free()
