"""GPU parity of the access statistics and the sparse Adam step against the oracle.

Bars: the weighted access histogram per location relative <= 1e-5 (fp32
atomics against the fp64 sum of the recipe weights), the set of accessed
locations exact, the KL divergence relative <= 1e-6; a lattice-point batch
gives used = 1 and KL = 0.  Adam: moments per row relative <= 1e-6, the step
(new - old value) per row relative <= 1e-4 (fp32 table entries of size 0.02
carry 2e-9 of rounding against steps of size lr), bf16 tables within one bf16
unit of the rounded fp64 result plus the fp32 rounding of the step; untouched
rows bit-identical; used gradient rows cleared.  The touched-row step
(flags from lram_mark_touched) is bit-identical to the full-scan step on
table, moments and gradient, and leaves every flag cleared; the flags mark
exactly the oracle's locations of the lookups.
"""
import itertools

import numpy as np
import pytest
import torch

import oracle
import paper_2107_03474_amd as lram
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _rel_rows(a, b):
    a = np.asarray(a, np.float64).reshape(a.shape[0], -1)
    b = np.asarray(b, np.float64).reshape(b.shape[0], -1)
    num = np.linalg.norm(a - b, axis=1)
    den = np.linalg.norm(b, axis=1)
    return np.where(den > 0, num / np.where(den > 0, den, 1), num)


@pytest.mark.parametrize("K", [(4, 4, 4, 4, 8, 8, 8, 8), (2, 4, 6, 8, 2, 4, 6, 8)])
def test_access_stats(K):
    N = int(np.prod(K))
    w = W.Workload("t", K, 32, "f32", 4096, 4, "zipf_mix", False, gmm_sigma=0.3, zipf_centres=64, zipf_s=1.1)
    q_np = W.queries(w).reshape(-1, 8)
    q = torch.from_numpy(q_np).to(DEV)
    hist = lram.access_histogram(q, K)
    st = lram.access_stats(hist)
    nb = oracle.neighbors(q_np, K)
    href = oracle.access_histogram(nb, N, weights="w32")
    h = hist.cpu().numpy().astype(np.float64)
    assert np.array_equal(h > 0, href > 0)
    np.testing.assert_allclose(h[href > 0], href[href > 0], rtol=1e-5)
    used, kl = oracle.access_stats(oracle.access_histogram(nb, N))
    assert st["count"] == int((href > 0).sum()) and abs(st["used"] - used) < 1e-15
    np.testing.assert_allclose(st["kl"], kl, rtol=1e-6)


@pytest.mark.parametrize("K", [(2, 2, 2, 2, 2, 2, 2, 2), (4, 4, 4, 4, 4, 4, 4, 2), (4, 6, 8, 4, 4, 6, 4, 8)])
@pytest.mark.parametrize("L", [1, 3, 65, 4097, 16383, 16384, 32768 + 5, 70001, 98304 + 1])
def test_histogram_sizes(L, K):
    """Every form of the histogram kernel (pair by pair; merged per workgroup with 4, 8 and 16 lookups to a wave), ragged
    last tiles and waves, non-finite queries, clustered and uniform ones, few locations (dense lines of the hash, which
    wraps) and many, added to what is there.  Bar: the n positive terms of a location and its old value meet in at most
    2 n fp32 additions (in LDS, then in memory), each rounded by at most 2^-24 of the final sum."""
    N = int(np.prod(K))
    rng = np.random.default_rng(L + N)
    n = min(L, 4000)  # the oracle's share; the batch repeats it
    q = rng.random((n, 8)) * np.asarray(K)
    q[: n // 2] = np.asarray(K) / 2.0 + 0.3 * rng.standard_normal((n // 2, 8))
    q = q.astype(np.float32)
    bad = rng.random(n) < 0.02
    q[bad, 3] = rng.choice([np.nan, np.inf, -np.inf], bad.sum())
    times = np.bincount(np.arange(L) % n, minlength=n)
    nb = oracle.neighbors(np.where(bad[:, None], 0.0, q).astype(np.float32), K)
    w = np.where(bad[:, None], 0.0, nb["w32"].astype(np.float64)) * times[:, None]
    real = nb["slot"] >= 0
    ref = np.bincount(nb["slot"][real], weights=w[real], minlength=N)
    old = rng.random(N).astype(np.float32)
    hist = torch.from_numpy(old).to(DEV)
    lram.access_histogram(torch.from_numpy(np.resize(q, (L, 8))).to(DEV), K, hist=hist)
    got = hist.cpu().numpy().astype(np.float64)
    untouched = np.bincount(nb["slot"][real & ~bad[:, None]], minlength=N) == 0
    assert np.array_equal(got[untouched], old[untouched].astype(np.float64))
    pairs = np.bincount(nb["slot"][real], weights=np.broadcast_to(times[:, None], real.shape)[real], minlength=N)
    assert (np.abs(got - old - ref) <= 2 * pairs * 2.0 ** -24 * (old + ref)).all()


@pytest.mark.parametrize("N,offset", [(1, 0), (3, 1), (1023, 0), (1025, 1), (262145, 0), (1048579, 3), (2097152, 0)])
def test_access_stats_sizes(N, offset):
    """One value, remainders of the 16-byte loads, unaligned arrays, one to many workgroups: fp64 sums of at most
    2^21 terms, so 1e-12 relative (2^21 * 2^-53 = 2.3e-10 is the worst case of one serial sum; the partial sums of
    a workgroup are at most 2^13 long)."""
    rng = np.random.default_rng(N)
    h = np.where(rng.random(N) < 0.3, 0.0, rng.exponential(1.0, N)).astype(np.float32)
    h[0] = 0.5
    buf = torch.zeros(N + offset, device=DEV)
    buf[offset:] = torch.from_numpy(h)
    st = lram.access_stats(buf[offset:])
    x = h.astype(np.float64)
    H, pos = x.sum(), x[x > 0]
    kl = np.log(N) + (pos * np.log(pos)).sum() / H - np.log(H)
    assert st["count"] == pos.size and st["used"] == pos.size / N
    np.testing.assert_allclose(st["total"], H, rtol=1e-12)
    np.testing.assert_allclose(st["kl"], kl, rtol=1e-12, atol=1e-11)


def test_access_stats_lattice_points_uniform():
    K = (2, 2, 2, 4, 2, 2, 2, 2)
    pts = []
    for eps in (0, 1):
        for Y in itertools.product(*[range(k) for k in K]):
            if sum(Y) % 2 == 0:
                pts.append((2 * np.asarray(Y) + eps) / 2.0)
    q = torch.from_numpy(np.asarray(pts, np.float32)).to(DEV)
    st = lram.access_stats(lram.access_histogram(q, K))
    assert st["used"] == 1.0 and abs(st["kl"]) < 1e-9 and st["count"] == int(np.prod(K))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m", [32, 64])
def test_sparse_adam(m, dtype):
    rng = np.random.default_rng(5)
    N = 70001
    V0 = (rng.standard_normal((N, m)) * 0.02).astype(np.float32)
    g = rng.standard_normal((N, m)).astype(np.float32) * 1e-2
    g[rng.random(N) < 0.4] = 0.0          # untouched rows
    g[7, :5] = 0.0                         # a touched row with some zero entries
    m1 = (rng.standard_normal((N, m)) * 1e-3).astype(np.float32)
    m2 = (rng.random((N, m)) * 1e-4).astype(np.float32)
    table = torch.from_numpy(V0).to(DEV).to(dtype)
    V0r = table.float().cpu().numpy()       # the table as stored (bf16-rounded)
    grad = torch.from_numpy(g).to(DEV)
    e1 = torch.from_numpy(m1).to(DEV)
    e2 = torch.from_numpy(m2).to(DEV)
    lram.sparse_adam(table, grad, e1, e2, step=3, lr=1e-3)
    torch.cuda.synchronize()
    Vr, r1, r2 = oracle.sparse_adam(V0r, g, m1, m2, 3, lr=1e-3)
    touched = np.any(g != 0, axis=1)
    Vg = table.float().cpu().numpy()
    assert np.array_equal(Vg[~touched], V0r[~touched])
    assert np.array_equal(e1.cpu().numpy()[~touched], m1[~touched])
    assert np.array_equal(e2.cpu().numpy()[~touched], m2[~touched])
    assert _rel_rows(e1.cpu().numpy()[touched], r1[touched]).max() <= 1e-6
    assert _rel_rows(e2.cpu().numpy()[touched], r2[touched]).max() <= 1e-6
    if dtype == torch.float32:
        assert _rel_rows((Vg - V0r)[touched], (Vr - V0r)[touched]).max() <= 1e-4
    else:
        ref = torch.from_numpy(Vr.astype(np.float32)).to(torch.bfloat16).float().numpy()
        # one bf16 unit at either magnitude, plus the fp32 rounding of the step
        # (which dominates where the step cancels the value)
        bound = np.maximum(np.abs(ref), np.abs(Vg)) * 2.0 ** -7 + 4 * 2.0 ** -24 * np.abs(Vr - V0r) + 1e-30
        assert np.all(np.abs(Vg[touched] - ref[touched]) <= bound[touched])
    assert torch.count_nonzero(grad).item() == 0


def test_training_step_roundtrip():
    """forward + backward (merged) + the Adam step leave untouched rows alone
    and move exactly the rows the batch read."""
    K = (4, 4, 4, 4, 8, 8, 8, 8)
    N = int(np.prod(K))
    rng = np.random.default_rng(6)
    q = torch.from_numpy((rng.random((140000, 8)) * np.asarray(K)).astype(np.float32)).to(DEV)
    table = (torch.randn((N, 64), device=DEV) * 0.02)
    before = table.clone()
    opt = lram.SparseAdam(table, lr=1e-3)
    G = torch.randn((140000, 64), device=DEV)
    gt, _ = lram.backward(q, table, K, G, want_grad_q=False, mode="merged")
    read = torch.zeros(N, dtype=torch.bool, device=DEV)
    s = lram.neighbors(q, K, want_d2=False)[0]
    read[s[s >= 0].long()] = True
    opt.step(gt)
    torch.cuda.synchronize()
    moved = (table != before).any(1)
    assert torch.equal(moved, read)
    assert torch.count_nonzero(gt).item() == 0


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m", [32, 64])
def test_sparse_adam_touched_matches_full_scan(m, dtype):
    K = (4, 4, 4, 4, 8, 8, 8, 8)
    N = int(np.prod(K))
    rng = np.random.default_rng(8)
    q_np = (rng.random((3000, 8)) * np.asarray(K)).astype(np.float32)
    q_np[7] = np.nan                       # no neighbours
    q = torch.from_numpy(q_np).to(DEV)
    touched = lram.mark_touched(q, K)
    nb = oracle.neighbors(q_np, K)
    ref = np.zeros(N, bool)
    ref[nb["slot"][nb["slot"] >= 0]] = True
    assert np.array_equal(touched.cpu().numpy() != 0, ref)
    table = (torch.randn((N, m), device=DEV) * 0.02).to(dtype)
    G = torch.randn((3000, m), device=DEV)
    G[11] = 0.0                            # a lookup whose rows get no gradient from it
    gt, _ = lram.backward(q, table.float() if dtype == torch.float32 else table, K, G, want_grad_q=False,
                          mode="merged")
    e1 = (torch.randn((N, m), device=DEV) * 1e-3)
    e2 = torch.rand((N, m), device=DEV) * 1e-4
    t2, g2, a1, a2 = table.clone(), gt.clone(), e1.clone(), e2.clone()
    lram.sparse_adam(table, gt, e1, e2, step=5, lr=1e-3)
    lram.sparse_adam(t2, g2, a1, a2, step=5, lr=1e-3, touched=touched)
    torch.cuda.synchronize()
    assert torch.equal(table, t2) and torch.equal(e1, a1) and torch.equal(e2, a2) and torch.equal(gt, g2)
    assert torch.count_nonzero(touched).item() == 0
