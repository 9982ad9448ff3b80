"""The tile search at its edges: tiles of every size up to two, and tiles that mix lookups which the tile search
decides with ones that take the general search (lattice points, holes, near ties) or have no list (non-finite
queries), in either place of a pair.

Bars as in the parity tests: lists, distances and weights bit-exact against the oracle; forward, dq and the value
gradient per row relative 1e-5 (fp32) / 2e-2 (a bf16 result), zero rows for non-finite queries.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2107_03474_amd as lram
from test_tile_search_model import near_ties
from test_gpu_parity import _rel_rows, _say, check_neighbors, special_queries

pytestmark = pytest.mark.gpu
DEV = "cuda"


def mixed_queries(L, K, seed):
    rng = np.random.default_rng(seed)
    q = (rng.random((L, 8)) * np.asarray(K)).astype(np.float32)
    sp = special_queries(K)
    for l in range(L):
        kind = rng.integers(0, 4)
        if kind == 0:
            q[l] = sp[rng.integers(0, len(sp))]
        elif kind == 1:
            q[l] = (rng.integers(0, 16, 8) / 4.0).astype(np.float32)
    return q


@pytest.mark.parametrize("L", [1, 2, 3, 15, 16, 17, 31, 33, 129])
@pytest.mark.parametrize("K", [(4,) * 8, (2, 4, 6, 8, 10, 2, 4, 6)])
def test_lists(L, K):
    _say("tile lists L=%d K=%s" % (L, K))
    check_neighbors(mixed_queries(L, K, L), K)


@pytest.mark.parametrize("L", [3072, 3073, 4096, 4097, 6143, 6145, 8191, 8192, 8193])
def test_line_between_searches(L):
    """Either side of the sizes at which a second lookup joins a wave and tiles replace the general search (4,096 and
    8,192; 3,072 and 6,144 for m = 64 fp32): lists bit-exact, and the forward, the saved lists and the gradients of
    the same queries in a batch of the other kind."""
    _say("tile line L=%d" % L)
    K = (4, 4, 6, 4, 4, 8, 4, 4)
    q_np = np.resize(mixed_queries(300, K, L), (L, 8))
    check_neighbors(q_np, K)
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    table = torch.randn((int(np.prod(K)), 64), generator=g, device=DEV) * 0.02
    G = torch.randn((L, 64), generator=g, device=DEV)
    q = torch.from_numpy(q_np).to(DEV)
    other = torch.cat([q, q, q]) if L <= 6144 else q[:4096]
    n = min(L, other.shape[0])
    nl, nl2 = lram.new_lists(q), lram.new_lists(other)
    out, out2 = lram.forward(q, table, K, lists=nl), lram.forward(other, table, K, lists=nl2)
    # the same 32 products in the searches' own orders: 32 additions, 32 2^-24 of the terms' sum, far below 1e-5
    assert _rel_rows(out[:n].cpu().numpy(), out2[:n].cpu().numpy()).max() <= 1e-5
    assert torch.equal(nl.slot[:n].sort(1)[0], nl2.slot[:n].sort(1)[0])
    G2 = torch.cat([G, G, G])[:other.shape[0]]
    for kw, kw2 in (({}, {}), ({"lists": nl}, {"lists": nl2})):
        gt, gq = lram.backward(q, table, K, G, mode="atomic", **kw)
        _, gq2 = lram.backward(other, table, K, G2, grad_table=False, mode="atomic", **kw2)
        a, b = gq[:n].cpu().numpy(), gq2[:n].cpu().numpy()
        size = np.linalg.norm(b, axis=1)
        assert (np.linalg.norm(a - b, axis=1) <= np.maximum(1e-5 * size, 1e-6 * size.max())).all()
        nb = oracle.neighbors(q_np, K)
        uniq, acc = oracle.grad_table_rows(nb, G.cpu().numpy())
        assert _rel_rows(gt.cpu().numpy()[uniq], acc).max() <= 2e-5


@pytest.mark.parametrize("m,dtype", [(32, torch.float32), (64, torch.float32), (64, torch.bfloat16)])
@pytest.mark.parametrize("L", [2047, 2048, 2049, 4095, 4097])
def test_line_between_searches_activation_layer(L, m, dtype):
    """theta against the lookup on its own coordinates, scaled (one rounding each: 2^-23, 2^-8 in bf16)."""
    _say("tile line theta L=%d" % L)
    K = (4, 4, 6, 4, 4, 8, 4, 4)
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    table = (torch.randn((int(np.prod(K)), m), generator=g, device=DEV) * 0.02).to(dtype)
    z = torch.randn((L, 16), generator=g, device=DEV)
    z[::101, 3] = float("nan")
    q, s = lram.theta_coords(z, K)
    ref = (lram.forward(q, table.float(), K).double() * s.double()[:, None]).cpu().numpy()
    got = lram.theta_forward(z, table, K).double().cpu().numpy()
    assert _rel_rows(got, ref).max() <= (1e-5 if dtype == torch.float32 else 1e-2)
    G = torch.randn((L, m), generator=g, device=DEV)
    gt, _ = lram.theta_backward(z, table, K, G, mode="atomic")
    gt2, _ = lram.backward(q, table, K, G * s[:, None], mode="atomic")
    a, b = gt.double().cpu().numpy(), gt2.double().cpu().numpy()
    size = np.linalg.norm(b, axis=1)
    assert (np.linalg.norm(a - b, axis=1) <= 2e-5 * size + 1e-6 * size.max()).all()


@pytest.mark.parametrize("m,dtype", [(32, "f32"), (64, "f32"), (32, "bf16"), (64, "bf16")])
@pytest.mark.parametrize("L", [1, 3, 17, 40000])
def test_step(L, m, dtype):
    _say("tile step L=%d m=%d %s" % (L, m, dtype))
    K = (4, 4, 6, 4, 4, 8, 4, 4)
    N = int(np.prod(K))
    q_np = mixed_queries(min(L, 500), K, 7 * L + m)
    q_np = np.resize(q_np, (L, 8))
    if L > 2:
        q_np[L // 2, 3] = np.nan
        q_np[L - 1, 0] = np.inf
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    table = (torch.randn((N, m), generator=g, device=DEV) * 0.02).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    G = torch.randn((L, m), generator=g, device=DEV)
    q = torch.from_numpy(q_np).to(DEV)
    out = lram.forward(q, table, K)
    gt, gq = lram.backward(q, table, K, G, mode="atomic")
    fin = np.isfinite(q_np).all(1)
    assert not out.cpu().float().numpy()[~fin].any() and not gq.cpu().numpy()[~fin].any()
    nb = oracle.neighbors(np.where(fin[:, None], q_np, 0), K)
    rows = oracle.gather_rows(table.float().cpu().numpy(), nb["slot"])
    G_np = np.where(fin[:, None], G.cpu().numpy(), 0)
    assert _rel_rows(out.float().cpu().numpy()[fin], oracle.forward(nb, rows)[fin]).max() <= (1e-5 if dtype == "f32" else 2e-2)
    ref = oracle.grad_query(nb, rows, G_np)
    # at a lattice point dq is the sum of exactly cancelling terms' rounding: absolute bar, 1e-6 of the largest row
    err = np.linalg.norm(gq.cpu().numpy()[fin] - ref[fin], axis=1)
    size = np.linalg.norm(ref[fin], axis=1)
    assert (err <= np.maximum(1e-5 * size, 1e-6 * size.max())).all()
    uniq, acc = oracle.grad_table_rows(nb, G_np)
    got = gt.cpu().numpy()
    assert _rel_rows(got[uniq], acc).max() <= 2e-5
    rest = np.ones(N, bool)
    rest[uniq] = False
    assert not got[rest].any()


@pytest.mark.parametrize("gap", [1e-6, 1e-5, 3e-5, 1e-4])
def test_near_ties(gap):
    """The 32nd and 33rd distances closer than, about as far as and farther apart than the tile search's margin."""
    _say("tile near ties", gap)
    check_neighbors(near_ties(gap, 6000, int(1e7 * gap)), (8,) * 8)
