#!/usr/bin/env python3
"""Generate the E8 candidate table used by the GPU neighbour search.

Sec. 2.6 of the paper maps a query by a lattice isometry into the fundamental
region

    F = { z : z_0 >= z_1 >= ... >= z_6 >= |z_7|,  z_0 + z_1 <= 2,  sum z <= 4 }

(Lambda = 2*E8 scale) and scans a fixed list of lattice points: those whose
distance to F is below sqrt(8).  This script finds that list by convex
quadratic programming, done exactly: the projection of a point p onto F is the
projection onto the affine span of some active set S of F's ten facets with
non-negative multipliers; all 2^10 active sets are tried (vectorised fp64),
and every classification near r^2 = 8 is re-derived in exact rational
arithmetic.

Output (``e8_candidates.inc``):
  * the STRICT list  -- dist(p, F)^2 < 8 (the paper's 232 points), in
    ascending order of that distance, and E8_FAST / E8_FAST_BOUND: the first
    E8_FAST of them and the exact distance^2 from F of every later one, at
    least E8_FAST_BOUND (a query in F whose k-th closest point among the
    first E8_FAST lies below that bound takes its closest k from them), and
    the same for the first E8_FAST2 (E8_FAST2_BOUND), a smaller first tier;
  * the BOUNDARY list -- dist(p, F)^2 == 8 exactly.  These never lie in the open
    support of a query inside F, but a query whose reduction lands a rounding
    error outside F, or whose fp32 distance rounds below 8, can see them; the
    kernel scans them only on that rare path.
The gap to the next distance level is checked to be large.

Output (``e8_tile.inc``): the strict points in the order of the tile search,
15 blocks of 16 rows (a row of a matrix product each; indices into the strict
list).  How often each point is among the 32 closest is sampled over uniform
queries: ten points always are, 67 others ever.  Blocks 0-3 hold the 64 points
that are next most often, block 4 the ten in its rows 0-9 and six of the
rest, blocks 5-14 the rest (rows repeated to fill the last of either norm).
The search checks its result against every row, so the sample decides only how
often a query takes the general path.
"""
from __future__ import annotations

import os
import sys
from fractions import Fraction

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(HERE, "e8_candidates.inc")
OUT_TILE = os.path.join(HERE, "e8_tile.inc")


FAST = 192  # three candidates per lane of a 64-lane wave
FAST2 = 128  # two per lane: the first tier of the fast set


def lattice_points(max_norm: int) -> np.ndarray:
    """All points of Lambda = {x in (2Z)^8 u (2Z+1)^8 : sum x = 0 mod 4} with |x|^2 <= max_norm."""
    r = int(np.floor(np.sqrt(max_norm)))
    pts = []
    for eps in (0, 1):
        vals = np.array([v for v in range(-r, r + 1) if (v - eps) % 2 == 0], np.int64)
        grid = np.stack(np.meshgrid(*([vals] * 8), indexing="ij"), -1).reshape(-1, 8)
        keep = ((grid * grid).sum(1) <= max_norm) & (grid.sum(1) % 4 == 0)
        pts.append(grid[keep])
    return np.concatenate(pts)


def facets():
    """F as A z <= b (10 rows)."""
    A, b = [], []
    for j in range(6):
        row = np.zeros(8, np.int64)
        row[j + 1], row[j] = 1, -1
        A.append(row), b.append(0)
    row = np.zeros(8, np.int64); row[7], row[6] = 1, -1; A.append(row); b.append(0)
    row = np.zeros(8, np.int64); row[7], row[6] = -1, -1; A.append(row); b.append(0)
    row = np.zeros(8, np.int64); row[0] = row[1] = 1; A.append(row); b.append(2)
    A.append(np.ones(8, np.int64)); b.append(4)
    return np.array(A), np.array(b)


def project_all(P: np.ndarray):
    """fp64 distance^2 from every row of P to F and the active set achieving it."""
    A, b = facets()
    best = np.full(P.shape[0], np.inf)
    best_set = [None] * P.shape[0]
    Pf = P.astype(np.float64)
    for mask in range(1 << 10):
        S = [i for i in range(10) if mask >> i & 1]
        if S:
            As = A[S].astype(np.float64)
            G = As @ As.T
            if np.linalg.matrix_rank(G) < len(S):
                continue
            lam = np.linalg.solve(G, (As @ Pf.T) - b[S][:, None].astype(np.float64))  # [|S|, n]
            Z = Pf - (As.T @ lam).T
            ok = np.all(lam >= -1e-9, axis=0)
        else:
            Z = Pf.copy()
            ok = np.ones(P.shape[0], bool)
        feas = np.all(A @ Z.T <= b[:, None] + 1e-9, axis=0)
        ok &= feas
        d = ((Pf - Z) ** 2).sum(1)
        upd = ok & (d < best - 1e-12)
        best[upd] = d[upd]
        for i in np.nonzero(upd)[0]:
            best_set[i] = S
    return best, best_set


def exact_dist2(p, S) -> Fraction:
    """Exact KKT check of active set S for point p; returns dist^2 as a Fraction."""
    A, b = facets()
    p = [Fraction(int(v)) for v in p]
    if not S:
        z = p
        lam = []
    else:
        As = [[Fraction(int(v)) for v in A[i]] for i in S]
        n = len(S)
        G = [[sum(As[i][k] * As[j][k] for k in range(8)) for j in range(n)] for i in range(n)]
        rhs = [sum(As[i][k] * p[k] for k in range(8)) - b[S[i]] for i in range(n)]
        # Gaussian elimination in rationals
        M = [G[i][:] + [rhs[i]] for i in range(n)]
        for c in range(n):
            piv = next(r for r in range(c, n) if M[r][c] != 0)
            M[c], M[piv] = M[piv], M[c]
            for r in range(n):
                if r != c and M[r][c] != 0:
                    f = M[r][c] / M[c][c]
                    M[r] = [M[r][k] - f * M[c][k] for k in range(n + 1)]
        lam = [M[i][n] / M[i][i] for i in range(n)]
        z = [p[k] - sum(lam[i] * As[i][k] for i in range(n)) for k in range(8)]
    assert all(l >= 0 for l in lam), "negative multiplier"
    for i in range(10):
        assert sum(Fraction(int(A[i][k])) * z[k] for k in range(8)) <= b[i], "infeasible"
    return sum((p[k] - z[k]) ** 2 for k in range(8))


def sample_region(n: int, seed: int = 0) -> np.ndarray:
    """n points of F: uniform queries, reduced by their closest point and the signed permutation."""
    x = np.random.default_rng(seed).random((n, 8)) * 16.0

    def d8(y):
        r = np.rint(y)
        d = y - r
        odd = np.nonzero(r.sum(1).astype(np.int64) & 1)[0]
        j = np.abs(d).argmax(1)[odd]
        r[odd, j] += np.where(d[odd, j] > 0, 1, -1)
        return r

    a, b = 2 * d8(x / 2), 2 * d8((x - 1) / 2) + 1
    y = x - np.where((((x - a) ** 2).sum(1) <= ((x - b) ** 2).sum(1))[:, None], a, b)
    z = -np.sort(-np.abs(y), axis=1)
    z[:, 7] *= np.where((y < 0).sum(1) & 1, -1.0, 1.0)
    return z


def tile_order(strict: np.ndarray, n: int = 200000) -> np.ndarray:
    """Strict-list indices of the tile search's 15 x 16 rows."""
    z = sample_region(n)
    n2 = (strict ** 2).sum(1)
    d = (z ** 2).sum(1)[:, None] + n2[None] - 2.0 * z @ strict.T
    freq = np.bincount(np.argsort(d, axis=1, kind="stable")[:, :32].ravel(), minlength=len(strict))
    order = np.argsort(-freq, kind="stable")
    always, var, rest = order[:10], order[10:74], order[74:]
    assert n2[always].max() <= 8 and always[0] == 0
    small = [i for i in var if n2[i] == 8]
    large = [i for i in var if n2[i] == 16]
    assert len(small) >= 48
    rows = np.zeros((15, 16), np.int64)
    # blocks 0-2 of norm 8 throughout; block 3 the others of norm 8, then norm 16;
    # inside a block neighbours in frequency go to different groups of four
    # rows (a lane of the search holds four rows of a block)
    def deal(block):
        out = np.zeros(16, np.int64)
        for k, i in enumerate(block):
            turn, g = divmod(k, 4)
            out[4 * (g if turn % 2 == 0 else 3 - g) + turn] = i
        return out

    for b in range(3):
        rows[b] = deal(small[b::3][:16])
    used = set(rows[:3].ravel())
    rows[3] = deal([i for i in small if i not in used] + large)
    r8 = [i for i in rest if n2[i] == 8]
    r16 = [i for i in rest if n2[i] == 16]
    rows[4] = np.concatenate([always, r8[:6]])
    r8 = r8[6:]
    r8 += [r8[-1]] * (80 - len(r8))
    r16 += [r16[-1]] * (80 - len(r16))
    rows[5:10] = np.reshape(r8, (5, 16))
    rows[10:15] = np.reshape(r16, (5, 16))
    assert set(rows.ravel()) == set(range(len(strict)))
    return rows


def main(write: bool = True) -> dict:
    # |z| <= 2 on F (covering radius), so a point within sqrt 8 of F has |p|^2 < (2 + sqrt 8)^2 < 24;
    # norm 24 is included to measure the gap above the boundary level.
    P = lattice_points(24)
    d2, sets = project_all(P)
    strict, boundary, above = [], [], []
    for i in range(P.shape[0]):
        if d2[i] > 8 + 1e-6 and d2[i] > 9.0:
            above.append(d2[i])
            continue
        ex = exact_dist2(P[i], sets[i])
        if ex < 8:
            strict.append((ex, P[i]))
        elif ex == 8:
            boundary.append(P[i])
        else:
            above.append(float(ex))
    strict = sorted(strict, key=lambda e: (e[0], int((e[1] * e[1]).sum()), tuple(-e[1])))
    strict_d2 = [e[0] for e in strict]
    strict = [e[1] for e in strict]
    fast_bound = strict_d2[FAST] if FAST < len(strict) else Fraction(8)
    fast2_bound = strict_d2[FAST2]
    boundary = sorted(boundary, key=lambda v: (int((v * v).sum()), tuple(-v)))
    gap = min(above) - 8.0
    norms = {}
    for v in strict:
        norms[int((v * v).sum())] = norms.get(int((v * v).sum()), 0) + 1
    allpts = np.array(strict + boundary)
    info = dict(strict=np.array(strict), boundary=np.array(boundary), gap=gap, norms=norms,
                cmin=int(allpts.min()), cmax=int(allpts.max()), strict_d2=strict_d2, fast_bound=fast_bound,
                fast2_bound=fast2_bound)
    if write:
        with open(OUT, "w") as f:
            f.write("// Generated by gen_e8_candidates.py -- do not edit.\n")
            f.write("// Lattice points of Lambda = 2*E8 by their exact distance to the fundamental\n")
            f.write("// region F (Sec. 2.6): STRICT: dist^2 < 8, BOUNDARY: dist^2 == 8.\n")
            f.write("// Next distance^2 level above 8: 8 + %.6f.\n" % gap)
            f.write("#pragma once\n")
            f.write("#define E8_NSTRICT %d\n#define E8_NBOUNDARY %d\n" % (len(strict), len(boundary)))
            f.write("#define E8_CAND_MIN %d\n#define E8_CAND_MAX %d\n" % (info["cmin"], info["cmax"]))
            f.write("// Strict points FAST.. lie at distance^2 >= %s from F.\n" % fast_bound)
            f.write("#define E8_FAST %d\n#define E8_FAST_BOUND %.9gf\n" % (FAST, float(fast_bound)))
            f.write("// Strict points FAST2.. lie at distance^2 >= %s from F.\n" % fast2_bound)
            f.write("#define E8_FAST2 %d\n#define E8_FAST2_BOUND %.9gf\n" % (FAST2, float(fast2_bound)))
            for name, lst in (("E8_STRICT_INIT", strict), ("E8_BOUNDARY_INIT", boundary)):
                f.write("#define %s { \\\n" % name)
                for v in lst:
                    f.write("  {%s}, \\\n" % ", ".join("%2d" % int(c) for c in v))
                f.write("}\n")
        rows = tile_order(np.array(strict))
        with open(OUT_TILE, "w") as f:
            f.write("// Generated by gen_e8_candidates.py -- do not edit.\n")
            f.write("// Rows of the tile search: 15 blocks of 16 indices into E8_STRICT_INIT.\n")
            f.write("#pragma once\n#define E8_TILE_BLOCKS 15\n#define E8_TILE_INIT { \\\n")
            for r in rows:
                f.write("  {%s}, \\\n" % ", ".join("%3d" % i for i in r))
            f.write("}\n")
    return info


if __name__ == "__main__":
    info = main(write="--check" not in sys.argv)
    print("strict", len(info["strict"]), "by norm", info["norms"], "boundary", len(info["boundary"]),
          "gap", info["gap"], "coord range", info["cmin"], info["cmax"])
