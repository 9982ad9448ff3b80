"""CPU model of the tile search's rule for the closest 32, checked against the oracle.

The tile search forms the candidates' distances to the query in F as |p|^2/4 -
z.p/2 with exact products and fp32 sums (z in three bf16 parts; quarter units), finds a threshold T with 22 of 64 chosen
candidates below it, and accepts those and ten more as the closest 32 when no
candidate of the strict list lies within TILE_EPS of T on either side, the ten
are below, every other one is above, and 4 T + |z|^2 is below the support's
edge.  Whatever it accepts must be the oracle's 32 (decided by the fp32
distance recipe in the original coordinates); what it does not accept takes the
general search.
"""
import os
import re

import numpy as np
import pytest

import oracle
from test_symmetry_search_model import BOUNDARY, ROOT, STRICT, _reduce

CSRC = os.path.join(ROOT, "paper_2107_03474_amd", "csrc")
SEARCH = open(os.path.join(CSRC, "lram_search.h")).read()


def _constant(name):
    return np.float32(re.search(r"constexpr float %s = ([\d.e+-]+)f;" % name, SEARCH).group(1))


EPS, STEP, EDGE = _constant("TILE_EPS"), _constant("TILE_STEP"), _constant("TILE_EDGE")
ROWS = np.array([[int(v) for v in r.split(",")] for r in
                 re.findall(r"\{([\d,\s]+)\}", open(os.path.join(CSRC, "e8_tile.inc")).read())])
VAR, ALWAYS = ROWS[:4].ravel(), ROWS[4, :10]
OTHERS = np.array(sorted(set(range(len(STRICT))) - set(VAR) - set(ALWAYS)))


def test_tile_rows():
    """64 + 10 + the others are the whole strict list; the norms that the kernel takes as constants of a block."""
    assert ROWS.shape == (15, 16) and len(set(VAR)) == 64 and len(set(VAR) & set(ALWAYS)) == 0
    assert set(ROWS.ravel()) == set(range(len(STRICT)))
    n2 = (STRICT ** 2).sum(1)
    assert (n2[ROWS[:3]] == 8).all() and (n2[ROWS[5:10]] == 8).all() and (n2[ROWS[10:]] == 16).all()


def _parts(z):
    """-z/2 as three bf16 numbers (8 bits of the mantissa each): exact."""
    y, out = (-0.5 * z).astype(np.float32), []
    for _ in range(3):
        top = (y.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
        out.append(top)
        y = y - top
    assert not y.any()
    return out


def _toward_zero(d):
    """fp64 -> fp32, truncated."""
    f = d.astype(np.float32)
    return np.where(np.abs(f.astype(np.float64)) > np.abs(d), np.nextafter(f, np.float32(0)), f)


def _quarter_distances(z, rounding=lambda d: d.astype(np.float32)):
    """|p|^2/4 - z.p/2 of every strict candidate as a matrix product forms it: exact products of bf16 numbers, an fp32
    rounding after every addition (the order inside the matrix cores and their rounding are theirs)."""
    d = np.broadcast_to(((STRICT ** 2).sum(1) / 4).astype(np.float32), (z.shape[0], len(STRICT))).copy()
    for part in _parts(z):
        for r in range(8):
            d = rounding(d.astype(np.float64) + part[:, r:r + 1].astype(np.float64) * STRICT[None, :, r])
    return d


def near_ties(gap, n, seed, K=(8,) * 8):
    """Queries moved until their 32nd and 33rd distances differ by about `gap`."""
    rng = np.random.default_rng(seed)
    q = rng.random((n, 8)) * np.asarray(K)
    for _ in range(3):
        nb = oracle.neighbors(q.astype(np.float32), K, k=64)
        x = 2.0 * q
        a = nb["lift"][:, 31].astype(np.float64)
        b = nb["lift"][:, 32].astype(np.float64)
        # |x - b|^2 - |x - a|^2 is linear in x: step along its gradient 2 (a - b) to the wanted gap
        g = 2.0 * (a - b)
        diff = ((x - b) ** 2).sum(1) - ((x - a) ** 2).sum(1)
        q = (x + ((gap - diff) / (g * g).sum(1))[:, None] * g) / 2.0
    return np.mod(q, np.asarray(K)).astype(np.float32)


def _accepted(z, step, q):
    """Accepted lookups; the threshold at the middle of the gap (step None), or STEP past either of its ends (the
    thresholds that the kernel's own steps take).  q: the candidates' distances."""
    v = np.sort(q[:, VAR], axis=1)
    if step is None:
        T = (v[:, 21] + v[:, 22]) * np.float32(0.5)
    else:
        T = v[:, 21] + STEP if step > 0 else v[:, 22] - STEP
    T = T.astype(np.float32)[:, None]
    t = q - T
    below = t < 0
    r2 = (z * z).sum(1, dtype=np.float32)
    ok = (below[:, VAR].sum(1) == 22) & below[:, ALWAYS].all(1) & ~below[:, OTHERS].any(1)
    ok &= (np.abs(t) >= EPS).all(1) & (4 * T[:, 0] + r2 < EDGE)
    return ok, below


def _check(q, K, least):
    K = np.asarray(K)
    x = np.fmod(np.float32(2) * q, (2 * K).astype(np.float32)).astype(np.float32)
    c, r, s = _reduce(x)
    y = x - c.astype(np.float32)
    z = np.zeros_like(y)
    np.put_along_axis(z, r, (y * s).astype(np.float32), 1)
    nb = oracle.neighbors(q, K)
    exact = ((STRICT ** 2).sum(1) / 4.0)[None] - 0.5 * z.astype(np.float64) @ STRICT.T
    for rounding, unit in ((lambda d: d.astype(np.float32), 2.0 ** -22), (_toward_zero, 2.0 ** -21)):
        # against exact arithmetic: 24 additions of sums below 8, half a unit of 2^-21 each, a whole one truncated
        d = _quarter_distances(z, rounding)
        assert np.abs(d - exact).max() < 24 * unit
        for step in (None, 1, -1):
            ok, below = _accepted(z, step, d)
            assert ok.mean() >= least, (step, ok.mean())
            for l in np.nonzero(ok)[0]:
                p = STRICT[below[l]]
                k = c[l] + s[l] * p[:, r[l]]
                assert len(p) == 32
                slots = oracle.locations(k.astype(np.int32), K)
                assert set(slots.tolist()) == set(nb["slot"][l].tolist()), (step, l, q[l])


def test_margin():
    """The margin covers, in quarter units: the product's error whichever way the matrix cores round (24 additions of
    sums below 8, one unit of 2^-21 each at most); z's (differences of norm at most 2, so 2 * 2^-24 in norm, times
    |p| / 2 <= 2); and the recipe's (seven additions below 8, squares and differences each rounded by 2^-24 relative,
    squares summing below 8)."""
    product = 24 * 2.0 ** -21
    z = 2 * 2.0 ** -24 * 2
    recipe = (7 * 2.0 ** -22 + 8 * 2.0 ** -24 + 2 * 8 * 2.0 ** -24) / 4
    assert product + z + recipe < EPS < STEP


@pytest.mark.parametrize("K", [(4,) * 8, (14,) * 8, (4, 6, 8, 10, 4, 4, 6, 4)])
def test_accepted_lists_are_the_oracles(K):
    rng = np.random.default_rng(5)
    q = (rng.random((3000, 8)) * np.asarray(K)).astype(np.float32)
    q[:300] = q[:300] * 5 - 2 * np.asarray(K, np.float32)
    _check(q, K, 0.98)


@pytest.mark.parametrize("gap", [1e-7, 1e-6, 4e-6, 1.6e-5, 3.2e-5, 6.4e-5, 2e-4])
def test_near_ties(gap):
    """Accepted or not, never wrong."""
    _check(near_ties(gap, 300, int(1e9 * gap)), (8,) * 8, 0.0)


def test_special_points():
    """Lattice points, holes, dyadic grids and queries a hair away from a lattice point."""
    K = (8,) * 8
    rng = np.random.default_rng(3)
    q = rng.integers(0, 64, size=(400, 8)) / 8.0
    near = rng.integers(0, 8, size=(300, 8)) + rng.standard_normal((300, 8)) * 10.0 ** rng.uniform(-6, -0.5, (300, 1))
    _check(np.mod(np.concatenate([q, near]), 8).astype(np.float32), K, 0.0)
    assert BOUNDARY.shape[0] == 171
