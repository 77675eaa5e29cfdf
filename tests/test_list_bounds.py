"""Bounds behind the candidate lists, checked by replaying their FP32
arithmetic (fused multiply-adds included) on the CPU.

A seed j leaves the list of a box when a lower bound of C_j - C_o over the box,
o the box's owner, exceeds the two seeds' slacks and the lists' own.  That is
sound when the computed bound is at most the exact one plus the slacks, less
what the double evaluation of the two costs (which decides the label) can be
off: 2^-49 (lambda_G |d|^2 + |w| + lambda_G sum_d Y_d^2) per seed, |d| the
largest distance to the box and Y_d the largest coordinate.  The exact values are
formed in extended precision (2^-64) from the exact box.

Three forms of the bound are replayed: a box's seeds from the caller's arrays, a
tile's from its super-tile's records (their offsets shifted to the tile's centre
in FP32), and a wave's from the tile's staged coefficients; on whole tiles and on
last tiles that the grid's end clips to a column or a single pixel, boxes with
very uneven pixels and away from the origin, seeds near and far, condition
numbers up to 10^12 and a large common offset of the weights.
"""
from __future__ import annotations

import numpy as np
import pytest

f4, ld = np.float32, np.longdouble


def fma(a, b, c):
    """a b + c in FP32 with one rounding (the product is exact in extended
    precision)."""
    return (np.asarray(a, ld) * np.asarray(b, ld) + np.asarray(c, ld)).astype(f4)


def tile_ext(dim, p):
    return (8 * p, 32) if dim == 2 else (16, 16, 8) if p == 8 else (4 * p, 8, 8)


class Case:
    """A tile of a grid, the super-tile that holds it, and m pairs of seeds."""

    def __init__(self, rng, dim, grid, lo, hi, p, sf, tile, m, kappa, reach, offset=0.0, soft=False):
        self.dim, self.m = dim, m
        self.ext = tile_ext(dim, p)
        self.lo, self.grid = lo, grid
        self.s = [(hi[d] - lo[d]) / grid[d] for d in range(dim)]
        self.a = [tile[d] * self.ext[d] for d in range(dim)]
        self.b = [min(self.a[d] + self.ext[d], grid[d]) - 1 for d in range(dim)]
        self.sa = [tile[d] // sf[d] * sf[d] * self.ext[d] for d in range(dim)]
        self.sb = [min(self.sa[d] + sf[d] * self.ext[d], grid[d]) - 1 for d in range(dim)]
        # seeds at distances of `reach` of the smallest pixel side (geometrically
        # spread) or of the tile, about a pixel of the tile
        y = np.stack([lo[d] + (rng.integers(self.a[d], self.b[d] + 1, m) + 0.5) * self.s[d] for d in range(dim)], 1)
        far = np.exp(rng.uniform(np.log(reach[0]), np.log(reach[1]), (m, 2, 1)))
        u = rng.normal(size=(m, 2, dim))
        u /= np.linalg.norm(u, axis=-1, keepdims=True)
        scale = np.where(rng.random((m, 1, 1)) < 0.5, min(self.s), np.asarray(self.s))
        k = np.exp(rng.uniform(0.0, np.log(kappa), (m, 2)))
        ev = np.stack([k ** (t / (dim - 1)) for t in range(dim)], -1) * k[..., None] ** -0.5
        R = np.linalg.qr(rng.normal(size=(m, 2, dim, dim)))[0]
        if soft:  # along the direction of the least eigenvalue
            u, scale = R[..., 0], min(self.s)
        self.x = y[:, None, :] + far * u * scale
        A = (R * ev[..., None, :]) @ np.swapaxes(R, -1, -2)
        self.A = 0.5 * (A + np.swapaxes(A, -1, -2))
        self.w = np.zeros((m, 2))
        # the weights: the two costs nearly tie at that pixel
        c = self.cost(y)
        tie = np.exp(rng.uniform(np.log(1e-12), np.log(1e-2), m)) * c.max(1) * rng.choice([-1.0, 1.0], m)
        self.w[:, 1] = c[:, 1] - c[:, 0] + tie
        self.w += offset
        self.wmax = self.w.max(1)
        lg = np.abs(self.A).sum(-1).max(-1)
        self.lg = lg
        self.lam = lg.max(1).astype(f4) * f4(1.0001)
        det = np.linalg.det(self.A)
        self.kap = (2.0 * lg ** dim / det).max(1).astype(f4) * f4(1.0001)
        self.Y2 = sum((abs(lo[d]) + grid[d] * self.s[d]) ** 2 for d in range(dim))
        self.sab = (2.0 ** -44 * (np.abs(self.wmax) + self.lam.astype(float) * self.Y2)).astype(f4)
        self.lsl = f4(2) * self.sab + f4(2.0 ** -20) * (self.lam.astype(float) * min(self.s) ** 2).astype(f4)

    def cost(self, y):
        """Both costs at y in double, in the definition's order."""
        out = []
        for q in range(2):
            d = [y[:, r] - self.x[:, q, r] for r in range(self.dim)]
            v = 0.0
            for r in range(self.dim):
                row = 0.0
                for c in range(self.dim):
                    t = self.A[:, q, min(r, c), max(r, c)] * d[c]
                    row = t if c == 0 else row + t
                t = d[r] * row
                v = t if r == 0 else v + t
            out.append(v - self.w[:, q])
        return np.stack(out, 1)

    def exact(self, a, b):
        """The exact lower bound of C_0 - C_1 and of C_1 - C_0 over the pixel
        centres a .. b, and what the double costs of the two can be off there."""
        dim = self.dim
        s = [ld(v) for v in self.s]
        ctr = [ld(self.lo[d]) + (ld(a[d] + b[d] + 1) / 2) * s[d] for d in range(dim)]
        h = [ld(b[d] - a[d]) / 2 * s[d] for d in range(dim)]
        e = np.stack([self.x[..., d].astype(ld) - ctr[d] for d in range(dim)], -1)
        A = self.A.astype(ld)
        Ae = (A * e[..., None, :]).sum(-1)
        c = (e * Ae).sum(-1) - (self.w.astype(ld) - self.wmax.astype(ld)[:, None])
        g = -2 * Ae
        out = []
        for q in (0, 1):
            lb = c[:, q] - c[:, 1 - q] - sum(np.abs(g[:, q, d] - g[:, 1 - q, d]) * h[d] for d in range(dim))
            for r in range(dim):
                for k in range(r, dim):
                    v = (A[:, q, r, k] - A[:, 1 - q, r, k]) * (1 if r == k else 2)
                    lb = lb + (np.minimum(v, 0) if r == k else -np.abs(v)) * h[r] * h[k]
            out.append(lb)
        dist = np.sqrt((e ** 2).sum(-1)) + np.sqrt(sum(v * v for v in h))
        off = (ld(2) ** -49 * (self.lg * dist ** 2 + np.abs(self.w) + self.lg * self.Y2)).sum(1)
        return out, off

    def bound(self, Q, h):
        """can_beat's bound and threshold for seed q against the other."""
        out = []
        for q in (0, 1):
            (c, s, g, a), (co, so, go, ao) = Q[q], Q[1 - q]
            lb = c - co
            for d in range(self.dim):
                lb = fma(-np.abs(g[d] - go[d]), h[d], lb)
            for k, (r, t) in enumerate((r, t) for r in range(self.dim) for t in range(r, self.dim)):
                v = a[k] - ao[k]
                lb = fma(np.minimum(v, f4(0)) if r == t else -np.abs(v), f4(h[r]) * f4(h[t]), lb)
            out.append((lb, s + so + self.lsl))
        return out

    def cell_quad(self, e, q, hh):
        """The quadratic of seed q from its FP32 offset e, and its slack."""
        A, wp = self.A[:, q].astype(f4), (self.w[:, q] - self.wmax).astype(f4)
        e2, c, g = np.full(self.m, hh, f4), np.zeros(self.m, f4), []
        for j in range(self.dim):
            ae = np.zeros(self.m, f4)
            for k in range(self.dim):
                ae = fma(A[:, min(j, k), max(j, k)], e[k], ae)
            g.append(f4(-2) * ae)
            c = fma(e[j], ae, c)
            e2 = fma(e[j], e[j], e2)
        a = [A[:, r, t] * f4(1 if r == t else 2) for r in range(self.dim) for t in range(r, self.dim)]
        return c - wp, f4(2.0 ** -15) * fma(self.lam, e2, np.abs(wp)), g, a

    def centre(self, d, a, b):
        return 0.5 * ((self.lo[d] + (a[d] + 0.5) * self.s[d]) + (self.lo[d] + (b[d] + 0.5) * self.s[d]))

    def from_arrays(self):
        """A tile's seeds from the caller's arrays."""
        h, hh = [], f4(0)
        for d in range(self.dim):
            lo, hi = (self.lo[d] + (k[d] + 0.5) * self.s[d] for k in (self.a, self.b))
            h.append(f4(0.5 * (hi - lo)) * f4(1 + 2.0 ** -20))
            hh = fma(h[d], h[d], hh)
        Q = [self.cell_quad([(self.x[:, q, d] - self.centre(d, self.a, self.b)).astype(f4) for d in range(self.dim)],
                            q, hh) for q in (0, 1)]
        return self.bound(Q, h), self.exact(self.a, self.b)

    def from_records(self):
        """A tile's seeds from its super-tile's records."""
        h, shift, hh = [], [], f4(0)
        for d in range(self.dim):
            s = f4(self.s[d])
            h.append(f4(0.5) * f4(self.b[d] - self.a[d]) * s * f4(1 + 2.0 ** -20))
            shift.append(f4(0.5) * f4(self.sa[d] + self.sb[d] - self.a[d] - self.b[d]) * s)
            hh = fma(h[d], h[d], hh)
            hh = fma(f4(2.0 ** -10) * shift[d], shift[d], hh)
        Q = [self.cell_quad([(self.x[:, q, d] - self.centre(d, self.sa, self.sb)).astype(f4) + shift[d]
                             for d in range(self.dim)], q, hh) for q in (0, 1)]
        return self.bound(Q, h), self.exact(self.a, self.b)

    def from_staged(self, wa, wb):
        """A wave's seeds (its box the pixels wa .. wb) from the staged
        coefficients of the tile."""
        dim = self.dim
        anc_k = [self.a[d] + self.ext[d] // 2 for d in range(dim)]
        s = [f4(v) for v in self.s]
        r2t = f4(0)
        for d in reversed(range(dim)):
            half = f4(0.5 * self.ext[d]) * s[d]
            r2t = fma(half, half, r2t)
        r2t = self.lam * r2t * f4(1.01)
        uc = [f4(wa[d] + wb[d] + 1 - 2 * anc_k[d]) * (f4(0.5) * s[d]) for d in range(dim)]
        h = [f4(wb[d] - wa[d]) * (f4(0.5 * (1 + 2.0 ** -20)) * s[d]) for d in range(dim)]
        kslack = f4(2.0 ** -44) * (self.kap + f4(1))
        Q = []
        for q in (0, 1):
            e = [self.x[:, q, d] - (self.lo[d] + anc_k[d] * self.s[d]) for d in range(dim)]
            ee, lin = 0.0, []
            for r in range(dim):
                ae = 0.0
                for k in range(dim):
                    ae = ae + self.A[:, q, min(r, k), max(r, k)] * e[k]
                lin.append((-2.0 * ae).astype(f4))
                ee = ee + e[r] * ae
            c0 = (ee - (self.w[:, q] - self.wmax)).astype(f4)
            a = [((1.0 if r == t else 2.0) * self.A[:, q, r, t]).astype(f4) for r in range(dim) for t in range(r, dim)]
            if dim == 2:
                t0 = fma(a[0], uc[0], fma(a[1], uc[1], lin[0]))
                t1 = fma(a[2], uc[1], lin[1])
                c = fma(t0, uc[0], fma(t1, uc[1], c0))
                g = [fma(a[0], uc[0], t0), fma(a[1], uc[0], fma(a[2], uc[1], t1))]
            else:
                t0 = fma(a[0], uc[0], fma(a[1], uc[1], fma(a[2], uc[2], lin[0])))
                t1 = fma(a[3], uc[1], fma(a[4], uc[2], lin[1]))
                t2 = fma(a[5], uc[2], lin[2])
                c = fma(t0, uc[0], fma(t1, uc[1], fma(t2, uc[2], c0)))
                g = [fma(a[0], uc[0], t0), fma(a[1], uc[0], fma(a[3], uc[1], t1)),
                     fma(a[2], uc[0], fma(a[4], uc[1], fma(a[5], uc[2], t2)))]
            Q.append((c, (f4(2.0 ** -16) + kslack) * (np.abs(c) + f4(2) * r2t), g, a))
        return self.bound(Q, h), self.exact(wa, wb)


def worst(result):
    """Largest (computed bound - exact bound + what the double costs can be
    off) / threshold: above 1, a seed that wins could leave the list."""
    got, (lbs, off) = result
    return max(float(((lb.astype(ld) - e + off) / t.astype(ld)).max()) for (lb, t), e in zip(got, lbs))


BOXES = [
    # dim, grid, lo, hi, rows per lane, tiles of a super-tile, tile
    (2, (1024, 1024), (0, 0), (1, 1), 4, (3, 3), (10, 11)),         # a whole tile
    (2, (65536, 225), (0, 0), (1, 1), 4, (8, 8), (100, 7)),         # one column, sides 1 : 291
    (2, (225, 65536), (0, 0), (1, 1), 8, (4, 8), (3, 100)),         # one row
    (2, (2017, 2017), (0, 0), (1, 1), 4, (8, 8), (63, 63)),         # one pixel
    (2, (1505, 1761), (3, -7), (4, -6), 4, (8, 8), (47, 55)),       # one pixel, away from the origin
    (3, (256, 256, 256), (0, 0, 0), (1, 1, 1), 8, (3, 3, 5), (4, 4, 9)),
    (3, (65, 65, 65), (0, 0, 0), (1, 1, 1), 2, (8, 8, 8), (8, 8, 8)),            # one voxel
    (3, (4097, 65, 65), (-1, 0, 2), (0, 1, 3), 4, (8, 8, 8), (256, 8, 8)),       # one voxel, sides 1 : 63
    (3, (8192, 57, 57), (0, 0, 0), (1, 1, 1), 8, (4, 4, 8), (30, 3, 7)),         # thin, sides 1 : 144
]


@pytest.mark.parametrize("box", range(len(BOXES)))
@pytest.mark.parametrize("kappa,reach,offset", [(9.0, (0.05, 40.0), 0.0), (9.0, (0.5, 400.0), 1e3),
                                                (1e6, (0.05, 400.0), 0.0)])
def test_lists_of_a_tile(box, kappa, reach, offset):
    """A tile's seeds from the caller's arrays and from the records."""
    rng = np.random.default_rng(100 + box)
    case = Case(rng, *BOXES[box], m=60000, kappa=kappa, reach=reach, offset=offset)
    assert worst(case.from_arrays()) <= 1.0
    assert worst(case.from_records()) <= 1.0


@pytest.mark.parametrize("box", range(len(BOXES)))
def test_pairs_beside_a_clipped_tile(box):
    """Pairs of seeds of one matrix on either side of the tile's middle along its
    last axis, where the whole tile sees the same difference of the costs: the
    one of lower double cost at every pixel stays in the list."""
    rng = np.random.default_rng(200 + box)
    case = Case(rng, *BOXES[box], m=60000, kappa=1.0 + 1e-12, reach=(1.0, 2.0))
    t = case.dim - 1
    mid = [case.centre(d, case.a, case.b) for d in range(case.dim)]
    case.x[:] = np.asarray(mid) + rng.uniform(-8, 8, (case.m, 1, case.dim)) * min(case.s)
    case.x[..., t] = mid[t] + rng.choice([-1, 1], (case.m, 2)) * rng.uniform(4, 40, (case.m, 2)) * min(case.s)
    case.A[:] = np.eye(case.dim)
    case.w[:] = 0.0
    y = np.broadcast_to(np.asarray(mid), (case.m, case.dim))
    c = case.cost(y)
    case.w[:, 1] = c[:, 1] - c[:, 0] + np.exp(rng.uniform(np.log(1e-9), np.log(1e-3), case.m)) * c.max(1) * \
        rng.choice([-1.0, 1.0], case.m)
    case.wmax = case.w.max(1)
    assert worst(case.from_records()) <= 1.0
    if all(a == b for a, b in zip(case.a, case.b)):
        c = case.cost(y)
        (lb0, t0), (lb1, t1) = case.from_records()[0]
        assert not np.any((lb0 > t0) & (c[:, 0] <= c[:, 1])) and not np.any((lb1 > t1) & (c[:, 1] <= c[:, 0]))


def waves_of(case, p):
    """The pixels of the tile's waves."""
    dim = case.dim
    we = (4 * p, 16) if dim == 2 else (p, 8, 8)
    for w in range(4):
        if dim == 2 or p == 8:
            off = ((w >> 1) * we[0], (w & 1) * we[1], 0)
        else:
            off = (w * p, 0, 0)
        a = [case.a[d] + off[d] for d in range(dim)]
        yield a, [max(a[d], min(a[d] + we[d], case.grid[d]) - 1) for d in range(dim)]


@pytest.mark.parametrize("box", range(len(BOXES)))
@pytest.mark.parametrize("kappa,reach,offset,soft", [(9.0, (0.05, 40.0), 0.0, False), (9.0, (0.5, 400.0), 1e3, False),
                                                     (1e6, (0.05, 400.0), 0.0, True), (1e12, (1e3, 1e9), 0.0, True)])
def test_lists_of_a_wave(box, kappa, reach, offset, soft):
    """A wave's seeds from the tile's staged coefficients.  Far along the least
    eigenvalue's direction of an ill-conditioned matrix a cost is small against the
    terms of its double evaluation, whose rounding the slack has to cover."""
    rng = np.random.default_rng(300 + box)
    case = Case(rng, *BOXES[box], m=20000, kappa=kappa, reach=reach, offset=offset, soft=soft)
    for wa, wb in waves_of(case, BOXES[box][4]):
        assert worst(case.from_staged(wa, wb)) <= 1.0


# ------------------------------------------------ the bounds of the super-tiles

@pytest.mark.parametrize("box", range(len(BOXES)))
@pytest.mark.parametrize("kappa,reach,offset", [(9.0, (0.05, 400.0), 0.0), (9.0, (0.5, 4000.0), 1e3), (1e6, (0.05, 400.0), 0.0)])
@pytest.mark.parametrize("region", [False, True])
def test_bounds_of_a_super_tile(box, kappa, reach, offset, region):
    """The FP32 bounds of a seed's cost over a super-tile, from the caller's arrays
    or from a region's record (offsets shifted in FP32), lie outside the exact
    lambda_min dist^2 - w' and lambda_max maxdist^2 - w' by at least what the double
    costs can be off."""
    rng = np.random.default_rng(400 + box)
    dim, grid, lo, hi, p, sf, tile = BOXES[box]
    case = Case(rng, dim, grid, lo, hi, p, sf, tile, m=30000, kappa=kappa, reach=reach, offset=offset)
    # the region: four super-tiles per axis around this one
    ext = [case.ext[d] * sf[d] for d in range(dim)]
    ra = [case.sa[d] // (4 * ext[d]) * 4 * ext[d] for d in range(dim)]
    rb = [min(ra[d] + 4 * ext[d], grid[d]) - 1 for d in range(dim)]
    ev = np.linalg.eigvalsh(case.A)
    span = 1e-6 * (np.abs(ev[..., -1]) + np.abs(ev[..., 0]))
    lmin, lmax = ev[..., 0] - span, ev[..., -1] + span
    for q in (0, 1):
        ctr = [case.centre(d, case.sa, case.sb) for d in range(dim)]
        dist2, far2 = np.zeros(case.m, f4), np.zeros(case.m, f4)
        edist, efar = np.zeros(case.m, ld), np.zeros(case.m, ld)
        for d in range(dim):
            b0, b1 = (lo[d] + (k[d] + 0.5) * case.s[d] for k in (case.sa, case.sb))
            h = f4(0.5 * (b1 - b0)) * f4(1 + 2.0 ** -20)
            if region:
                rc = case.centre(d, ra, rb)
                shift = f4(rc - ctr[d])
                e = np.abs((case.x[:, q, d] - rc).astype(f4) + shift)
                h = fma(f4(2.0 ** -22), np.abs(shift), h) * f4(1 + 2.0 ** -20)
            else:
                e = np.abs((case.x[:, q, d] - ctr[d]).astype(f4))
            dd, fd = np.maximum(f4(0), e - h), e + h
            dist2, far2 = fma(dd, dd, dist2), fma(fd, fd, far2)
            x0 = case.x[:, q, d].astype(ld)
            xd = np.maximum(np.maximum(ld(b0) - x0, x0 - ld(b1)), 0)
            edist, efar = edist + xd ** 2, efar + np.maximum(x0 - ld(b0), ld(b1) - x0) ** 2
        wp = (case.w[:, q] - case.wmax).astype(f4)
        u = lmax[:, q].astype(f4) * far2
        slack = fma(f4(2.0 ** -18), u + np.abs(wp), case.lsl)
        lb, ub = fma(lmin[:, q].astype(f4), dist2, -wp) - slack, (u - wp) + slack
        we = case.w[:, q].astype(ld) - case.wmax.astype(ld)
        off = ld(2) ** -49 * (case.lg[:, q] * efar + np.abs(case.w[:, q]) + case.lg[:, q] * case.Y2)
        assert np.all(lb <= ev[:, q, 0] * edist - we - off)
        assert np.all(ub >= ev[:, q, -1] * efar - we + off)


# ---------------------------------------------------------- the settle rules

def test_short_settle_rule_implies_the_full_one():
    """A pixel settled by the rule without square roots at the tile's corner radius
    is settled by the per-pixel certificate, for any radius inside the tile."""
    rng = np.random.default_rng(500)
    m = 400000
    r2t = np.exp(rng.uniform(-12, 6, m)).astype(f4)
    r2 = (r2t * rng.random(m).astype(f4)).astype(f4)
    fb = (np.exp(rng.uniform(-14, 8, m)) * rng.choice([1, 1, 1, -1e-3], m)).astype(f4)
    sab = (np.exp(rng.uniform(-30, -10, m))).astype(f4)
    skb = (f4(2.0 ** -44) * np.exp(rng.uniform(1, 30, m)).astype(f4)).astype(f4)
    for kbits in (f4(0), f4(2.0 ** -18)):
        k1 = (f4(1.5 * 2.0 ** -18) + skb + kbits) * f4(1 + 2.0 ** -7)
        c = f4(1.5 * 2.0 ** -18) + skb
        k2 = ((f4(1.5 * 2.0 ** -17) + skb + f4(2.0 ** -9) * c) * r2t + sab) * f4(1 + 2.0 ** -7)
        need = fma(np.abs(fb), k1, k2)
        # the runner-up just above and well above what the short rule asks for
        for far in (f4(1 + 2.0 ** -20), f4(1.5), f4(40)):
            fs = fb + need * far
            short = (fs - fb) > need
            bb = np.maximum(fb, f4(0))
            B1 = bb + f4(2.0 ** -10) * (bb + r2)
            e1 = f4(2.0 ** -20) * (B1 + f4(4) * np.sqrt(r2) * np.sqrt(B1) + f4(4) * r2)
            thr = f4(2) * e1 + kbits * np.maximum(np.abs(fb), np.abs(fs)) + sab + skb * (B1 + r2)
            assert short.sum() > m // 4
            assert np.all((fs - fb)[short] > thr[short])
