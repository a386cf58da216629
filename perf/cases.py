"""Performance cases of the point-location and interpolation path.

Each case is one unit of work that a user of this library has it do: locate a
set of points and interpolate fields there, exchange interface data between
overlapping meshes, follow a moving mesh, or serve a batch of requests.  All
inputs are synthetic, made on the GPU from the seed.

Every mesh and field here is a sum of a few products of one-dimensional
functions of the parameter axes (u, v, w), sampled at the GLL nodes.  The
nodal interpolant of such a product is the product of the one-dimensional
interpolants, so the position and the field values at a chosen (element, r)
are known without any search: points are chosen as (element, r), mapped to
space, and `exact` returns what locating and interpolating them must give.
Most points lie inside an element; a small part lies just off a curved wall
(the nearest point of the mesh is then the foot of the wall's normal), and
some lie outside the domain.
"""
import math

import numpy as np
import torch

from paper_1811_04891_amd import findpts as fp

DEV = "cuda"


# --------------------------------------------------------------------------
# Case lists
# --------------------------------------------------------------------------
def listed():
    return [
        # a small interface or a handful of probes: few launches' worth of work
        dict(name="cube_1e4", kind="locate", mesh="box", n=4, m=4, l=4, N=5, points=10_000,
             fields=1, mixed=False, spread="uniform"),
        # one mid-size mesh with points everywhere: particles or grid-to-grid transfer
        dict(name="annulus_1e6", kind="locate", mesh="ring", n=16, m=64, l=16, N=7,
             points=1_010_000, fields=4, mixed=False, spread="uniform"),
        # a large mesh, many points near surfaces inside it, in random order
        dict(name="large_box_2e7", kind="locate", mesh="box", n=100, m=50, l=40, N=7,
             points=20_000_000, fields=5, mixed=False, spread="spheres"),
        # two overlapping meshes: interface points with session tags, and
        # points of the overlap that the distance field assigns
        dict(name="two_sessions_1e6", kind="sessions", n=8, m=121, l=20, m1=50, N=7,
             points=1_200_000, fields=4, mixed=False),
        # a higher order with many points per element
        dict(name="order9_2e6", kind="locate", mesh="box", n=40, m=25, l=20, N=9,
             points=2_000_000, fields=4, mixed=False, spread="uniform"),
        # a request on a large resident mesh: a few points per element
        dict(name="order9_sparse", kind="locate", mesh="box", n=36, m=36, l=36, N=9,
             points=150_001, fields=3, mixed=False, spread="uniform"),
        # high-order elements
        dict(name="order12_2e5", kind="locate", mesh="ring", n=8, m=32, l=8, N=12,
             points=200_003, fields=2, mixed=False, spread="uniform"),
        # one strongly curved element at a tight tolerance
        dict(name="spiral_1000", kind="spiral", N=15, points=1000, fields=1),
        # a timestep of the overlapping-mesh exchange at known locations:
        # extrapolation, then subiterations of interpolation and flux correction
        dict(name="exchange_step", kind="exchange", n=8, m=121, l=20, m1=50, N=7,
             points=120_320, subiterations=4),
        # a two-dimensional mesh
        dict(name="ring2d_1e6", kind="locate2d", mesh="ring", n=64, m=256, N=7,
             points=1_010_000, fields=4, spread="uniform"),
        # a mesh that moved: new coordinates, then its interface points again
        dict(name="moving_mesh", kind="moving", n=16, m=64, l=16, N=7, points=120_320, fields=4),
        # a batch of requests of mixed sizes on resident meshes, in the mixed precision
        dict(name="serving_batch", kind="serving", e_min=729, e_max=20_000, p_min=1_000,
             p_max=1_000_000, requests=12, slots=4, mixed=True),
    ]


def _log_int(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["locate"] * 7 + ["sessions", "spiral", "exchange", "locate2d", "locate2d",
                                        "moving", "serving"])
    if kind in ("locate", "moving"):
        N = rng.choice([3, 4, 5, 5, 6, 7, 7, 7, 7, 8, 9, 9, 10, 11, 12, 13, 15])
        e_max = min(50_000, int(3e7 / (N + 1) ** 3))
        E = _log_int(rng, 64, e_max)
        mesh = rng.choice(["box", "ring"])
        if mesh == "box":
            n = max(4, round(E ** (1 / 3)))
            m = max(4, n + rng.randint(-1, 2))
            l = max(4, round(E / (n * m)))
        else:
            n = max(2, round((E / 4) ** (1 / 3)))
            m = max(12, 4 * n + rng.randint(-2, 3))
            l = max(2, round(E / (n * m)))
        case = dict(kind=kind, n=n, m=m, l=l, N=N, points=_log_int(rng, 1_000, 3_000_000 // (N + 1) * 4),
                    fields=rng.randint(1, 6))
        if kind == "locate":
            case.update(mesh=mesh, mixed=rng.random() < 0.3,
                        spread=rng.choice(["uniform", "uniform", "spheres"]))
        else:
            case.update(n=max(2, n // 2), m=max(12, m), l=max(2, l // 2),
                        points=_log_int(rng, 1_000, 300_000))
        return case
    if kind in ("sessions", "exchange"):
        case = dict(kind=kind, n=rng.choice([4, 5, 7, 8]), m=rng.randint(24, 130),
                    l=rng.randint(4, 20), m1=rng.randint(20, 60), N=rng.choice([5, 6, 7, 7, 8, 9]))
        if kind == "sessions":
            case.update(points=_log_int(rng, 5_000, 1_200_000), fields=rng.randint(1, 5),
                        mixed=rng.random() < 0.3)
        else:
            case.update(points=_log_int(rng, 5_000, 300_000), subiterations=rng.randint(1, 4))
        return case
    if kind == "spiral":
        return dict(kind=kind, N=rng.choice([13, 14, 15, 15]), points=_log_int(rng, 100, 300_000),
                    fields=rng.randint(1, 3))
    if kind == "locate2d":
        mesh = rng.choice(["ring", "box"])
        n = _log_int(rng, 4, 100)
        return dict(kind=kind, mesh=mesh, n=n, m=max(16, 4 * n) if mesh == "ring" else max(4, n),
                    N=rng.choice([3, 5, 7, 7, 9, 11]), points=_log_int(rng, 1_000, 2_000_000),
                    fields=rng.randint(1, 5), spread="uniform")
    return dict(kind=kind, e_min=500, e_max=_log_int(rng, 2_000, 20_000), p_min=1_000,
                p_max=_log_int(rng, 20_000, 1_000_000), requests=rng.randint(4, 12),
                slots=rng.randint(1, 4), mixed=rng.random() < 0.7)


# --------------------------------------------------------------------------
# One-dimensional node tables
# --------------------------------------------------------------------------
def _gll(N):
    c = np.zeros(N + 1)
    c[N] = 1.0
    inner = np.polynomial.legendre.legroots(np.polynomial.legendre.legder(c)) if N > 1 else []
    z = np.concatenate([[-1.0], np.real(np.sort(inner)), [1.0]])
    return 0.5 * (z - z[::-1])


class _Basis:
    """Lagrange basis on the GLL nodes: values at r, and the matrix that takes
    nodal values to the nodal values of the derivative."""

    def __init__(self, N):
        z = _gll(N)
        self.n1 = N + 1
        self.z = z
        diff = z[:, None] - z[None, :] + np.eye(N + 1)
        self.wb = 1.0 / diff.prod(1)
        D = (self.wb[None, :] / self.wb[:, None]) / diff
        np.fill_diagonal(D, 0.0)
        np.fill_diagonal(D, -D.sum(1))
        self.D = torch.tensor(D, dtype=torch.float64, device=DEV)
        self.nodes = torch.tensor(z, dtype=torch.float64, device=DEV)

    def at(self, r):
        t = [r - float(z) for z in self.z]
        pre = [torch.ones_like(r)]
        for i in range(self.n1 - 1):
            pre.append(pre[-1] * t[i])
        suf = torch.ones_like(r)
        h = [None] * self.n1
        for i in reversed(range(self.n1)):
            h[i] = float(self.wb[i]) * pre[i] * suf
            suf = suf * t[i]
        return torch.stack(h, -1)


class _Part:
    """A structured block of elements: per axis the element count and the
    parameter interval, per coordinate a list of terms (one function per
    axis, None for 1)."""

    def __init__(self, dims, lo, hi, N, coords):
        self.dims, self.lo, self.hi, self.N, self.coords = dims, lo, hi, N, coords
        self.B = _Basis(N)
        self.E = math.prod(dims)
        self.pos = []
        for a, nel in enumerate(dims):
            q = torch.arange(nel, dtype=torch.float64, device=DEV)[:, None]
            q = q + (self.B.nodes[None, :] + 1.0) * 0.5
            self.pos.append(lo[a] + (hi[a] - lo[a]) * (q / nel))

    def _table(self, f, a):
        return f(self.pos[a])

    def nodal(self, terms):
        """Nodal values, shape (E, n1, ...), the first axis' nodes fastest."""
        d, n1 = len(self.dims), self.B.n1
        total = 0.0
        for term in terms:
            prod = torch.ones([1] * (2 * d), dtype=torch.float64, device=DEV)
            for a, f in enumerate(term):
                if f is None:
                    continue
                shape = [1] * (2 * d)
                shape[d - 1 - a], shape[2 * d - 1 - a] = self.dims[a], n1
                prod = prod * self._table(f, a).reshape(shape)
            total = total + prod
        full = list(reversed(self.dims)) + [n1] * d
        return total.expand(full).reshape([self.E] + [n1] * d).contiguous()

    def at(self, sums, cell, ref, along=None):
        """Interpolants of several sums of terms at (cell, ref): (len(sums),
        P); with `along`, their derivatives in that axis."""
        P = ref[0].numel()
        out = torch.empty((len(sums), P), dtype=torch.float64, device=DEV)
        step = 1 << 20
        for b in range(0, P, step):
            s = slice(b, min(P, b + step))
            h = [self.B.at(r[s]) for r in ref]
            seen = {}

            def axis(f, a):
                if (f, a) not in seen:
                    tab = self._table(f, a)
                    if a == along:
                        tab = tab @ self.B.D.T
                    seen[f, a] = (tab[cell[a][s]] * h[a]).sum(-1)
                return seen[f, a]

            for q, terms in enumerate(sums):
                total = 0.0
                for term in terms:
                    if along is not None and term[along] is None:
                        continue
                    prod = 1.0
                    for a, f in enumerate(term):
                        if f is not None:
                            prod = prod * axis(f, a)
                    total = total + prod
                out[q, s] = total
        return out

    def place(self, par):
        """(cell, ref) of parameter positions, kept off the element faces."""
        cell, ref = [], []
        for a, nel in enumerate(self.dims):
            q = (par[a] - self.lo[a]) / (self.hi[a] - self.lo[a]) * nel
            c = q.floor().clamp(0, nel - 1)
            cell.append(c.long())
            ref.append((2.0 * (q - c) - 1.0).clamp(-1 + 1e-7, 1 - 1e-7))
        return cell, ref

    def element(self, cell):
        e, stride = torch.zeros_like(cell[0]), 1
        for a, nel in enumerate(self.dims):
            e = e + stride * cell[a]
            stride *= nel
        return e

    def off_wall(self, axis, side, cell, ref, distance, spots=2):
        """Points at `distance` off the wall (axis, side) above the wall point
        (cell, ref) (ref[axis] = side), and which of them lie in the box of
        the element's corners (and of `spots` - 2 places between them along
        the first axis), so that the element is a candidate for them."""
        d = len(self.dims)
        x = self.at(self.coords, cell, ref)
        J = [self.at(self.coords, cell, ref, along=a) for a in range(d)]
        t = [J[a] for a in range(d) if a != axis]
        if d == 3:
            nrm = torch.linalg.cross(t[0], t[1], dim=0)
        else:
            nrm = torch.stack([t[0][1], -t[0][0]])
        nrm = nrm / nrm.norm(dim=0)
        nrm = nrm * torch.sign((nrm * J[axis]).sum(0) * side)
        y = x + distance * nrm
        lo, hi = torch.full_like(x, math.inf), torch.full_like(x, -math.inf)
        for k in range(spots << (d - 1)):
            c = [torch.full_like(ref[0], 2.0 * (k >> (d - 1)) / (spots - 1) - 1.0)]
            c += [torch.full_like(ref[0], 1.0 if k >> a & 1 else -1.0) for a in range(d - 1)]
            p = self.at(self.coords, cell, c)
            lo, hi = torch.minimum(lo, p), torch.maximum(hi, p)
        return y, ((y > lo) & (y < hi)).all(0)


# --------------------------------------------------------------------------
# Meshes
# --------------------------------------------------------------------------
def _one_dim(f, *args):
    return lambda x: f(x, *args)


def _lin(x, a, b):
    return a + b * x


def _sin(x, k, p):
    return torch.sin(k * x + p)


def _rad_cos(x, a, b):
    return a * torch.cos(x + b)


def _box(n, m, l, N, rng):
    """Box stretched to the element counts, wavy in all coordinates; the
    waves vanish on the side walls but not on the walls w = const."""
    small = max(n, m, l) <= 8
    ext = (1.0, 1.0, 1.0) if small else (0.02 * n, 0.02 * m, 0.02 * l)
    amp = (0.04 if small else 0.02 * min(1.0, min(ext) / 0.8)) * (0.75 + 0.25 * rng.random())
    ku, kv, kw = (2.0, 2.0, 2.0) if small else (1.0, 2.0, 2.5)
    wave = (_one_dim(_sin, ku * math.pi / ext[0] * (2.0 if ku == 1.0 else 1.0), 0.0),
            _one_dim(_sin, kv * math.pi / ext[1], 0.0),
            _one_dim(_sin, kw * math.pi / ext[2], 0.5 + rng.random()))
    ident = _one_dim(_lin, 0.0, 1.0)
    scaled = lambda f: (lambda x: amp * f(x))  # noqa: E731
    first = scaled(wave[0])
    bump = (first, wave[1], wave[2])
    coords = [[(ident, None, None), bump], [(None, ident, None), bump], [(None, None, ident), bump]]
    return _Part((n, m, l), (0.0, 0.0, 0.0), ext, N, coords)


def _ring(n, m, l, N, r0, r1, turn, height=1.0):
    """Annulus, nodes at exact polar positions; axes radius, angle, height."""
    rho = _one_dim(_lin, 0.0, 1.0)
    cos, sin = _one_dim(_rad_cos, 1.0, turn), _one_dim(_rad_cos, 1.0, turn - 0.5 * math.pi)
    coords = [[(rho, cos, None)], [(rho, sin, None)], [(None, None, _one_dim(_lin, 0.0, 1.0))]]
    return _Part((n, m, l), (r0, 0.0, 0.0), (r1, 2.0 * math.pi, height), N, coords)


def _ring2d(n, m, N, turn):
    rho = _one_dim(_lin, 0.0, 1.0)
    coords = [[(rho, _one_dim(_rad_cos, 1.0, turn))],
              [(rho, _one_dim(_rad_cos, 1.0, turn - 0.5 * math.pi))]]
    return _Part((n, m), (0.5, 0.0), (1.0, 2.0 * math.pi), N, coords)


def _box2d(n, m, N, rng):
    ident = _one_dim(_lin, 0.0, 1.0)
    amp = 0.03 * (0.75 + 0.25 * rng.random())
    first = lambda x: amp * torch.sin(2.0 * math.pi * x)  # noqa: E731
    bump = (first, _one_dim(_sin, math.pi, 0.7))
    return _Part((n, m), (0.0, 0.0), (1.0, 1.0), N, [[(ident, None), bump], [(None, ident), bump]])


def _spiral(N, rng):
    """One element: a thick sheet along a spiral of one and a half turns."""
    theta = lambda r: 1.5 * math.pi * (r + 1.0)  # noqa: E731
    turn = rng.random()
    mid_c = lambda r: (1.0 + 0.25 * theta(r)) * torch.cos(theta(r) + turn)  # noqa: E731
    mid_s = lambda r: (1.0 + 0.25 * theta(r)) * torch.sin(theta(r) + turn)  # noqa: E731
    dir_c = lambda r: 0.2 * torch.cos(theta(r) + turn)  # noqa: E731
    dir_s = lambda r: 0.2 * torch.sin(theta(r) + turn)  # noqa: E731
    s = _one_dim(_lin, 0.0, 1.0)
    coords = [[(mid_c, None, None), (dir_c, s, None)], [(mid_s, None, None), (dir_s, s, None)],
              [(None, None, _one_dim(_lin, 0.0, 0.5))]]
    return _Part((1, 1, 1), (-1.0, -1.0, -1.0), (1.0, 1.0, 1.0), N, coords)


def _field_terms(d, count, rng):
    """Smooth fields: each the sum of two products of sines of the axes."""
    fields = []
    for _ in range(count):
        terms = []
        for _ in range(2):
            terms.append(tuple(_one_dim(_sin, rng.uniform(0.5, 3.0), rng.uniform(0.0, 6.0))
                               for _ in range(d)))
        fields.append(terms)
    return fields


# --------------------------------------------------------------------------
# Points with known locations
# --------------------------------------------------------------------------
class _Points:
    """Query points, and where they are: per run of points the part, the cell
    and the reference position (None: not on the mesh), and the squared
    distance."""

    def __init__(self, dim):
        self.dim, self.runs = dim, []

    def add(self, x, part=None, base=0, cell=None, ref=None, distance=0.0, tag=-1):
        self.runs.append((x, part, base, cell, ref, distance, tag))

    def finish(self, gen):
        x = torch.cat([r[0].T for r in self.runs])
        self.perm = torch.randperm(x.shape[0], generator=gen, device=DEV)
        tags = torch.cat([torch.full((r[0].shape[1],), r[6], dtype=torch.int32, device=DEV)
                          for r in self.runs])
        return x[self.perm].contiguous(), tags[self.perm].contiguous()

    def truth(self, fields):
        """(rst, dist2, values of the fields) in the points' order."""
        rst, d2, out = [], [], []
        for x, part, base, cell, ref, distance, _ in self.runs:
            P = x.shape[1]
            if part is None:
                rst.append(torch.zeros((P, self.dim), dtype=torch.float64, device=DEV))
                d2.append(torch.full((P,), math.inf, dtype=torch.float64, device=DEV))
                out.append(torch.full((len(fields), P), math.nan, dtype=torch.float64, device=DEV))
            else:
                rst.append(torch.stack(ref, -1))
                d2.append(torch.full((P,), distance * distance, dtype=torch.float64, device=DEV))
                out.append(part.at(fields, cell, ref))
        p = self.perm
        return torch.cat(rst)[p], torch.cat(d2)[p], torch.cat(out, 1)[:, p]


def _uniform(gen, n):
    return torch.rand(n, generator=gen, dtype=torch.float64, device=DEV)


def _inside(pts, part, gen, n, spread, base=0, tag=-1):
    d = len(part.dims)
    span = [h - l for l, h in zip(part.lo, part.hi)]
    if spread == "spheres":  # near 8 surfaces, half an element off them
        cen = torch.stack([part.lo[a] + span[a] * (0.1 + 0.8 * _uniform(gen, 8)) for a in range(d)])
        rad = (0.15 + 0.2 * _uniform(gen, 8)) * min(span)
        which = torch.randint(0, 8, (n,), generator=gen, device=DEV)
        v = torch.randn((d, n), generator=gen, dtype=torch.float64, device=DEV)
        v = v / v.norm(dim=0)
        off = torch.randn(n, generator=gen, dtype=torch.float64, device=DEV)
        h = min(s / k for s, k in zip(span, part.dims))
        v = cen[:, which] + (rad[which] + 0.5 * h * off) * v
        par = []
        for a in range(d):  # those past a wall are reflected back
            q = (v[a] - part.lo[a]) / span[a]
            par.append(part.lo[a] + span[a] * (1.0 - (1.0 - q.abs()).abs()).clamp(0.0, 1.0))
    else:
        par = [part.lo[a] + span[a] * _uniform(gen, n) for a in range(d)]
    cell, ref = part.place(par)
    pts.add(part.at(part.coords, cell, ref), part, base, cell, ref, tag=tag)


def _off_wall(pts, part, gen, n, axis, side, distance, margin=0.3, base=0, tag=-1, spots=2):
    """Up to n points just off a wall; fewer where the wall's shape leaves no
    room for them in their element's box."""
    cell, ref = [], []
    for a, nel in enumerate(part.dims):
        if a == axis:
            cell.append(torch.full((n,), 0 if side < 0 else nel - 1, dtype=torch.long, device=DEV))
            ref.append(torch.full((n,), float(side), dtype=torch.float64, device=DEV))
        else:
            cell.append(torch.randint(0, nel, (n,), generator=gen, device=DEV))
            ref.append((2.0 * _uniform(gen, n) - 1.0) * margin)
    x, ok = part.off_wall(axis, side, cell, ref, distance, spots)
    pts.add(x[:, ok], part, base, [c[ok] for c in cell], [r[ok] for r in ref], distance, tag)
    return int(ok.sum())


def _outside(pts, part, gen, n, tag=-1):
    d = len(part.dims)
    x = torch.stack([2.5 * max(abs(v) for v in part.hi) + 3.0 + _uniform(gen, n)
                     for _ in range(d)])
    pts.add(x, tag=tag)


def _ring_gap(part):
    """Distance off the inner wall: a ten-thousandth of an element, and less
    than what keeps the point in its element's box."""
    return min(0.03 * part.lo[0] * (2.0 * math.pi / part.dims[1]) ** 2,
               1e-4 * (part.hi[0] - part.lo[0]) / part.dims[0])


def _all_points(case, part, gen, P):
    """99 % inside, up to 0.8 % just off a wall, the rest outside."""
    d = len(part.dims)
    pts = _Points(d)
    n_wall, n_out = max(16, P // 125), max(2, P // 500)
    if case.get("mesh") == "ring" or case["kind"] == "moving":
        n_wall = _off_wall(pts, part, gen, n_wall, 0, -1, _ring_gap(part))
    elif case["kind"] == "spiral":
        n_wall = _off_wall(pts, part, gen, n_wall, 1, 1, 1e-4, margin=0.8, spots=41)
    else:
        h = (part.hi[d - 1] - part.lo[d - 1]) / part.dims[d - 1]
        n_wall = _off_wall(pts, part, gen, n_wall, d - 1, 1, 1e-4 * h, margin=0.8)
    _outside(pts, part, gen, n_out)
    _inside(pts, part, gen, P - n_wall - n_out, case.get("spread", "uniform"))
    return pts


def _generators(seed):
    return torch.Generator(device=DEV).manual_seed(seed), np.random.default_rng(seed)


# --------------------------------------------------------------------------
# One mesh
# --------------------------------------------------------------------------
def _one_mesh(case, seed):
    gen, rng = _generators(seed)
    kind, N = case["kind"], case["N"]
    if kind == "locate2d":
        part = (_ring2d(case["n"], case["m"], N, rng.random()) if case["mesh"] == "ring"
                else _box2d(case["n"], case["m"], N, rng))
    elif kind == "spiral":
        part = _spiral(N, rng)
    elif kind == "moving" or case["mesh"] == "ring":
        part = _ring(case["n"], case["m"], case["l"], N, 0.5, 1.0, rng.random())
    else:
        part = _box(case["n"], case["m"], case["l"], N, rng)
    fields = _field_terms(len(part.dims), case["fields"], rng)
    return part, fields, _all_points(case, part, gen, case["points"]), gen


def _buffers(P, nf, dim):
    return dict(code=torch.empty(P, dtype=torch.int32, device=DEV),
                el=torch.empty(P, dtype=torch.int32, device=DEV),
                rst=torch.empty((P, dim), dtype=torch.float64, device=DEV),
                dist2=torch.empty(P, dtype=torch.float64, device=DEV),
                out=torch.empty((nf, P), dtype=torch.float64, device=DEV))


def _prepare_one(case, seed):
    part, fields, pts, gen = _one_mesh(case, seed)
    x, _ = pts.finish(gen)
    P = x.shape[0]
    X = [part.nodal(c) for c in part.coords]
    s = dict(pts=x, fields=[part.nodal(f) for f in fields], **_buffers(P, len(fields), x.shape[1]))
    if case["kind"] == "locate2d":
        s["h"] = fp.findpts2_setup(X[0], X[1], part.N, tol=1e-12, max_points=P)
    elif case["kind"] == "moving":  # set up before the motion, coordinates after it kept
        before = _ring(case["n"], case["m"], case["l"], part.N, 0.5, 1.0, -0.01)
        s["h"] = fp.findpts_setup(*[before.nodal(c) for c in before.coords], part.N, tol=1e-12,
                                  max_points=P)
        s["X"] = X
    else:
        s["h"] = fp.findpts_setup(*X, part.N, tol=1e-14 if case["kind"] == "spiral" else 1e-12,
                                  max_points=P, precision=fp.FP_PREC_MIXED if case.get("mixed")
                                  else fp.FP_PREC_FP64)
    return s


def _located(s):
    return {k: s[k] for k in ("code", "el", "rst", "dist2", "out")}


def _run_one(case_kind, s):
    if case_kind == "locate2d":
        fp.findpts2(s["h"], s["pts"], None, s["code"], s["el"], s["rst"], s["dist2"])
        fp.findpts2_eval(s["h"], s["code"], s["el"], s["rst"], s["fields"], s["out"])
        return _located(s)
    if case_kind == "moving":
        fp.findpts_update(s["h"], *s["X"])
    fp.findpts(s["h"], s["pts"], s.get("tags"), s["code"], s["el"], s["rst"], s["dist2"])
    fp.findpts_eval(s["h"], s["code"], s["el"], s["rst"], s["fields"], s["out"])
    return _located(s)


def _exact_one(case, seed):
    part, fields, pts, gen = _one_mesh(case, seed)
    pts.finish(gen)
    rst, d2, out = pts.truth(fields)
    return dict(code=None, el=None, rst=rst, dist2=d2, out=out)


# --------------------------------------------------------------------------
# Two overlapping sessions: annuli that share the layer 0.7 <= radius <= 0.8
# --------------------------------------------------------------------------
def _two_parts(case, rng):
    n, l, N = case["n"], case["l"], case["N"]
    return (_ring(n, case["m"], l, N, 0.5, 0.8, rng.random()),
            _ring(n, case["m1"], l, N, 0.7, 1.0, rng.random()))


def _layer(pts, part, gen, n, r_lo, r_hi, base, tag):
    par = [r_lo + (r_hi - r_lo) * _uniform(gen, n), 2.0 * math.pi * _uniform(gen, n),
           _uniform(gen, n)]
    cell, ref = part.place(par)
    pts.add(part.at(part.coords, cell, ref), part, base, cell, ref, tag=tag)


def _sessions(case, seed):
    gen, rng = _generators(seed)
    a, b = _two_parts(case, rng)
    fields = _field_terms(3, case["fields"], rng)
    P, pts = case["points"], _Points(3)
    n_free, n_out = P // 10, max(2, P // 500)
    # points off the inner wall; tagged 1 like that mesh's own interface points
    n_wall = _off_wall(pts, a, gen, max(16, P // 125), 0, -1, _ring_gap(a), tag=1)
    _outside(pts, a, gen, n_out)
    _layer(pts, a, gen, n_free // 2, 0.705, 0.74, 0, -1)  # the distance field picks session 0
    _layer(pts, b, gen, n_free - n_free // 2, 0.76, 0.795, a.E, -1)  # and here session 1
    rest = P - n_wall - n_out - n_free
    _layer(pts, b, gen, rest // 2, 0.8, 0.8, a.E, 0)  # session 0's interface, in session 1
    _layer(pts, a, gen, rest - rest // 2, 0.7, 0.7, 0, 1)  # session 1's interface, in session 0
    return a, b, fields, pts, gen


def _two_handle(case, a, b, P):
    X = [torch.cat([a.nodal(p), b.nodal(q)]) for p, q in zip(a.coords, b.coords)]
    own = torch.cat([torch.zeros(a.E, dtype=torch.int32, device=DEV),
                     torch.ones(b.E, dtype=torch.int32, device=DEV)])
    delta = torch.cat([a.nodal([(_one_dim(_lin, 0.8, -1.0), None, None)]),
                       b.nodal([(_one_dim(_lin, -0.7, 1.0), None, None)])])
    return fp.findpts_setup(*X, case["N"], tol=1e-12, elem_session=own, delta=delta, max_points=P,
                            precision=fp.FP_PREC_MIXED if case.get("mixed") else fp.FP_PREC_FP64)


def _prepare_sessions(case, seed):
    a, b, fields, pts, gen = _sessions(case, seed)
    x, tags = pts.finish(gen)
    F = [torch.cat([a.nodal(f), b.nodal(f)]) for f in fields]
    return dict(pts=x, tags=tags, fields=F, h=_two_handle(case, a, b, x.shape[0]),
                **_buffers(x.shape[0], len(F), 3))


def _exact_sessions(case, seed):
    _, _, fields, pts, gen = _sessions(case, seed)
    pts.finish(gen)
    rst, d2, out = pts.truth(fields)
    return dict(code=None, el=None, rst=rst, dist2=d2, out=out)


# --------------------------------------------------------------------------
# Interface exchange at known locations
# --------------------------------------------------------------------------
def _exchange(case, seed):
    gen, rng = _generators(seed)
    a, b = _two_parts(case, rng)
    sets = [_field_terms(3, 4, rng) for _ in range(case["subiterations"])]
    P = case["points"]
    n0 = P // 2
    pts = _Points(3)
    _layer(pts, b, gen, n0, 0.8, 0.8, a.E, 0)
    _layer(pts, a, gen, P - n0, 0.7, 0.7, 0, 1)
    pts.perm = slice(None)  # points stay grouped by session
    x = torch.cat([r[0].T for r in pts.runs]).contiguous()
    tags = torch.cat([torch.full((r[0].shape[1],), r[6], dtype=torch.int32, device=DEV)
                      for r in pts.runs])
    rho = x[:, :2].norm(dim=1)
    nrm = torch.stack([x[:, 0] / rho, x[:, 1] / rho, torch.zeros_like(rho)])
    nrm[:, n0:] *= -1.0
    wts = torch.empty(P, dtype=torch.float64, device=DEV)
    wts[:n0] = 2.0 * math.pi * 0.8 / max(n0, 1)
    wts[n0:] = 2.0 * math.pi * 0.7 / (P - n0)
    hist = [torch.randn((4, P), generator=gen, dtype=torch.float64, device=DEV) for _ in range(3)]
    return a, b, sets, pts, x, tags, n0, nrm, wts, hist


def _prepare_exchange(case, seed):
    a, b, sets, pts, x, tags, n0, nrm, wts, hist = _exchange(case, seed)
    P = x.shape[0]
    h = _two_handle(case, a, b, P)
    code, el, rst, _ = fp.findpts(h, x, tags)
    return dict(h=h, code=code, el=el, rst=rst, n0=n0, hist=hist,
                sets=[[torch.cat([a.nodal(f), b.nodal(f)]) for f in fs] for fs in sets],
                sides=[(wts[:n0].contiguous(), nrm[:, :n0].contiguous(), slice(0, n0)),
                       (wts[n0:].contiguous(), nrm[:, n0:].contiguous(), slice(n0, P))],
                pred=torch.empty((4, P), dtype=torch.float64, device=DEV),
                outs=[torch.empty((4, P), dtype=torch.float64, device=DEV) for _ in sets],
                work=torch.empty(fp.FP_FLUX_WORK, dtype=torch.float64, device=DEV))


def _run_exchange(s):
    fp.fp_extrapolate(s["hist"], 3, s["pred"])
    for fields, out in zip(s["sets"], s["outs"]):
        fp.findpts_eval(s["h"], s["code"], s["el"], s["rst"], fields, out)
        for wts, nrm, cols in s["sides"]:
            fp.fp_flux_correct(wts, nrm, out[:3, cols], work=s["work"])
    return dict(pred=s["pred"], outs=list(s["outs"]))


def _exact_exchange(case, seed):
    _, _, sets, pts, _, _, n0, nrm, wts, hist = _exchange(case, seed)
    outs = []
    for fields in sets:
        out = pts.truth(fields)[2]
        for cols in (slice(0, n0), slice(n0, None)):
            w, n, u = wts[cols], nrm[:, cols], out[:3, cols]
            out[:3, cols] = u - (w * u * n).sum() / (w * n * n).sum() * n
        outs.append(out)
    return dict(pred=3.0 * hist[0] - 3.0 * hist[1] + hist[2], outs=outs)


# --------------------------------------------------------------------------
# A batch of served requests
# --------------------------------------------------------------------------
_SERVED_ORDERS = (5, 7, 9, 7)


def _served(case, seed):
    gen, rng = _generators(seed)
    meshes = []
    for i, N in enumerate(_SERVED_ORDERS):
        E = case["e_min"] * (case["e_max"] / case["e_min"]) ** (i / (len(_SERVED_ORDERS) - 1))
        if i % 2 == 0:
            n = max(4, round(E ** (1 / 3)))
            part = _box(n, n, n, N, rng)
        else:
            h = (math.pi * 0.75 / E) ** (1 / 3)
            part = _ring(max(1, round(0.5 / h)), max(12, round(2 * math.pi * 0.75 / h)),
                         max(1, round(1.0 / h)), N, 0.5, 1.0, rng.random())
        meshes.append((part, _field_terms(3, 5, rng), "ring" if i % 2 else "box"))
    reqs, n = [], case["requests"]
    for k in range(n):
        P = int(case["p_min"] * (case["p_max"] / case["p_min"]) ** (((5 * k) % n + 0.5) / n)) | 1
        part, fields, mesh = meshes[k % len(meshes)]
        pts = _all_points(dict(kind="locate", mesh=mesh), part, gen, P)
        x, _ = pts.finish(gen)
        ids = sorted(rng.choice(5, 1 + k % 5, replace=False).tolist())
        reqs.append((k % len(meshes), x, pts, ids))
    return meshes, reqs


def _prepare_serving(case, seed):
    meshes, reqs = _served(case, seed)
    srv = fp.Server(8 << 30, slots=case["slots"])
    ids = []
    for part, fields, _ in meshes:
        h = fp.findpts_setup(*[part.nodal(c) for c in part.coords], part.N, tol=1e-12,
                             max_points=4096, precision=fp.FP_PREC_MIXED if case["mixed"]
                             else fp.FP_PREC_FP64)
        ids.append(srv.add_mesh(h, [part.nodal(f) for f in fields]))
    todo = []
    for m, x, _, f in reqs:
        b = _buffers(x.shape[0], len(f), 3)
        todo.append((ids[m], x, f, (b["code"], b["el"], b["rst"], b["dist2"], b["out"])))
    torch.cuda.synchronize()  # requests' inputs have to be ready when they are submitted
    return dict(srv=srv, todo=todo)


def _run_serving(s):
    tickets = [s["srv"].submit(m, x, f, out=out) for m, x, f, out in s["todo"]]
    for t in tickets:
        s["srv"].wait(t)
    return [list(out) for _, _, _, out in s["todo"]]


def _exact_serving(case, seed):
    meshes, reqs = _served(case, seed)
    got = []
    for m, _, pts, ids in reqs:
        rst, d2, out = pts.truth([meshes[m][1][i] for i in ids])
        got.append([None, None, rst, d2, out])
    return got


# --------------------------------------------------------------------------
# The interface
# --------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    s = {"sessions": _prepare_sessions, "exchange": _prepare_exchange,
         "serving": _prepare_serving}.get(kind, _prepare_one)(case, seed)
    s["kind"] = kind
    return s


def run(s):
    if s["kind"] == "exchange":
        return _run_exchange(s)
    if s["kind"] == "serving":
        return _run_serving(s)
    return _run_one(s["kind"], s)


def exact(case, seed):
    return {"sessions": _exact_sessions, "exchange": _exact_exchange,
            "serving": _exact_serving}.get(case["kind"], _exact_one)(case, seed)


def _newton_flops(N, d):
    """One point: the closest node of one element, three steps of the map with
    its derivatives, one value of the map."""
    n1 = N + 1
    V = n1 ** d
    if d == 2:
        return 5 * V + 4 * (8 * V + 32 * n1)
    return 7 * V + 3 * (12 * V + 18 * n1 ** 2 + 24 * n1) + 6 * (V + n1 ** 2 + n1)


def _eval_flops(N, d):
    n1 = N + 1
    return 2 * sum(n1 ** k for k in range(1, d + 1))


def _work_locate(E, N, P, nf, d=3, tags=False, locate=True):
    V = (N + 1) ** d
    used = min(E, P)
    b = P * (8 * d + 8 + 8 * d + 8 + 8 * nf) + used * V * 8 * (nf + (d if locate else 0))
    return b + (4 * P if tags else 0), P * ((_newton_flops(N, d) if locate else 0)
                                            + nf * _eval_flops(N, d))


def work(case):
    kind = case["kind"]
    if kind == "serving":
        b = f = 0.0
        n = case["requests"]
        for k in range(n):
            i = k % len(_SERVED_ORDERS)
            E = case["e_min"] * (case["e_max"] / case["e_min"]) ** (i / (len(_SERVED_ORDERS) - 1))
            P = case["p_min"] * (case["p_max"] / case["p_min"]) ** (((5 * k) % n + 0.5) / n)
            x, y = _work_locate(E, _SERVED_ORDERS[i], P, 1 + k % 5)
            b, f = b + x, f + y
    elif kind in ("sessions", "exchange"):
        E = case["n"] * case["l"] * (case["m"] + case["m1"])
        E = E // case["n"] if kind == "exchange" else E // case["n"] * 2  # the layers that are met
        if kind == "sessions":
            b, f = _work_locate(E, case["N"], case["points"], case["fields"], tags=True)
        else:
            b, f = _work_locate(E, case["N"], case["points"], 4, locate=False)
            k, P = case["subiterations"], case["points"]
            b, f = k * (b + P * 80) + P * 128, k * (f + 12 * P)
    elif kind == "spiral":
        b, f = _work_locate(1, case["N"], case["points"], case["fields"])
    else:
        E = case["n"] * case["m"] * case.get("l", 1)
        d = 2 if kind == "locate2d" else 3
        b, f = _work_locate(E, case["N"], case["points"], case["fields"], d)
        if kind == "moving":
            b += E * (case["N"] + 1) ** 3 * 8 * 6
            f += E * 18 * (case["N"] + 1) ** 4
    return {"bytes": b, "flops": f}
