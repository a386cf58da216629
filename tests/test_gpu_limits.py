"""Limits that callers size against: the smallest serving budget that admits a
request, and the largest mesh the allocation-free interpolation takes."""
import numpy as np
import pytest
import torch

import workloads as w

pytestmark = pytest.mark.gpu


def _pass_bytes(E, MC, M, delta):
    """Workspace of a pass of M points with MC candidate slots each: pair arrays,
    element counters of both calls, per-block counts; 256-byte pieces."""
    def a(n, size=4):
        return (max(n, 1) * size + 255) // 256 * 256
    spare = min(4096, 2 * ((M + 63) // 64))
    return (a(M) + 4 * a(M * MC) + a(4 * M * MC, 8) + (a(M * MC, 8) if delta else 0) + 4 * a(E + 1)
            + a(M) + a(1) + a((E + 1 + 4095) // 4096 + 1) + a((M + 255) // 256) + a(E + spare)
            + 3 * a(M) + a(512, 8))


@pytest.mark.parametrize("delta", [False, True])
@pytest.mark.parametrize("shape", [(2, 2, 2), (11, 10, 10), (40, 30, 30)])
def test_smallest_budget_of_a_request(shape, delta):
    """The workspace of a 256-point pass admits any request, and 256 bytes less
    refuse it."""
    from paper_1811_04891_amd import findpts as fp
    print(f"case: serving budget, {shape}, distance field {delta}", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(*shape, N=2).to(dev)
    h = fp.findpts_setup(m.x, m.y, m.z, 2, max_points=1000,
                         delta=torch.ones_like(m.x) if delta else None)
    need = _pass_bytes(m.E, max(1, fp.findpts_get_hash(h)[3][2]), 256, delta)
    pts = torch.as_tensor(np.random.default_rng(1).uniform(0, 1, (5000, 3))).to(dev)
    alone = fp.findpts(h, pts)
    out = fp.findpts_eval(h, alone[0], alone[1], alone[2], [m.x])
    torch.cuda.synchronize()
    srv = fp.Server(need, slots=2)
    q = srv.submit(srv.add_mesh(h, [m.x]), pts, [0])
    assert srv.wait(q, 60.0) == fp.FP_OK
    for a, b in zip((q.code, q.el, q.rst, q.dist2, q.out), (*alone, out)):
        assert torch.equal(a, b)
    assert srv.latency()["peak_arena_bytes"] <= need
    srv.destroy()
    srv = fp.Server(need - 256, slots=2)
    mid = srv.add_mesh(h, [m.x])
    with pytest.raises(fp.FindptsError) as ei:
        srv.submit(mid, pts, [0])
    assert ei.value.code == fp.FP_ENOMEM
    srv.destroy()
    h.free()


def test_elements_of_the_allocation_free_interpolation():
    """4,192,191 elements are the most; one more is refused.  The pass is then 256
    points, and these go in 67."""
    from paper_1811_04891_amd import findpts as fp
    print("case: 4,192,191 and 4,192,192 elements", flush=True)
    dev = torch.device("cuda:0")
    m = w.box_mesh(64, 65503, 1, (0.0, 0.0, 0.0), (64.0, 65503.0, 1.0), N=1, device=dev)
    n = 17000
    g = torch.Generator(device=dev).manual_seed(2)
    for E in (4192192, 4192191):
        x, y, z = (c.reshape(-1, 8)[:E].contiguous() for c in (m.x, m.y, m.z))
        h = fp.findpts_setup(x, y, z, 1, max_points=64)
        el = torch.randint(0, E, (n,), generator=g, device=dev, dtype=torch.int32)
        el[0] = E - 1
        code = torch.zeros(n, dtype=torch.int32, device=dev)
        rst = 2.0 * torch.rand((n, 3), generator=g, device=dev, dtype=torch.float64) - 1.0
        out = torch.empty((1, n), dtype=torch.float64, device=dev)
        if E > 4192191:
            with pytest.raises(fp.FindptsError) as ei:
                fp.findpts_eval_noalloc(h, code, el, rst, [y], out)
            assert ei.value.code == fp.FP_ERANGE
        else:
            fp.findpts_eval_noalloc(h, code, el, rst, [y], out)
            lo = y[el.long(), 0]
            hi = y[el.long(), 7]
            want = lo + (hi - lo) * 0.5 * (1.0 + rst[:, 1])
            # sums of eight terms at the coordinate's magnitude
            assert torch.max(torch.abs(out[0] - want)) <= 16 * 2.0 ** -53 * 65503.0
        h.free()
