"""The merged scatter by sorted runs (tables small against the pairs): dV and dq against the atomic scatter.

Both scatters add the same fp32 products w_j G in different orders: a row of n additions of fp32 numbers differs by at
most n 2^-24 of the sum of magnitudes.  Rows here hold up to a few thousand pairs of random sign; the bar is 2e-5 of
the row's norm plus 1e-6 of the largest row (rows whose pairs nearly cancel), and for one row that every lookup hits
(131,072 additions) its own bound.  dq does not depend on the scatter: the same bits.
"""
import numpy as np
import pytest
import torch

import paper_2107_03474_amd as lram

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _say(*a):
    print(*a, flush=True)


def _compare(q, K, m, dtype, seed, merged):
    N = int(np.prod(K))
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    table = (torch.randn((N, m), generator=g, device=DEV) * 0.02).to(dtype)
    G = torch.randn((q.shape[0], m), generator=g, device=DEV)
    a, qa = lram.backward(q, table, K, G, mode="atomic")
    b, qb = merged(q, table, K, G)
    assert torch.equal(qa, qb)
    da, db = a.double(), b.double()
    err, size = (da - db).norm(dim=1), da.norm(dim=1)
    assert (err <= 2e-5 * size + 1e-6 * size.max()).all()
    assert torch.equal((a != 0).any(1), (b != 0).any(1))
    return table, G


def _merged(q, table, K, G):
    return lram.backward(q, table, K, G, mode="merged")


@pytest.mark.parametrize("m,dtype", [(32, torch.float32), (64, torch.float32), (32, torch.bfloat16), (64, torch.bfloat16)])
@pytest.mark.parametrize("L,K", [
    (65535, (4, 4, 4, 4, 4, 4, 4, 4)),     # below RUNS_MIN: the batch merge
    (65536, (4, 4, 4, 4, 4, 4, 4, 4)),
    (65537, (4, 4, 6, 4, 6, 4, 4, 8)),     # ragged, an uneven torus, 294,912 rows
    (131072 + 5, (2, 2, 4, 2, 2, 4, 2, 2)),  # 1,024 rows, both lifts of a side of 2, long runs
    (131072, (8, 8, 8, 8, 4, 4, 8, 4)),    # 2^21 rows, two pairs per row: sorted runs for m = 64, the batch merge for m = 32
])
def test_runs(L, K, m, dtype):
    _say("runs L=%d K=%s m=%d %s" % (L, K, m, dtype))
    g = torch.Generator(device=DEV)
    g.manual_seed(L + m)
    q = torch.rand((L, 8), generator=g, device=DEV) * torch.tensor(K, device=DEV)
    q[::97, 3] = float("nan")                              # padding pairs
    q[1::1013] = torch.round(q[1::1013].nan_to_num())      # lattice points: lists of one
    _compare(q, K, m, dtype, L, _merged)


@pytest.mark.parametrize("m", [32, 64])
def test_one_query(m):
    """Every lookup the same: 32 runs over all spans."""
    _say("one query m=%d" % m)
    K, L = (4,) * 8, 131072
    q = torch.full((L, 8), 1.3, device=DEV) + torch.arange(8, device=DEV) * 0.11
    table = torch.randn((4 ** 8, m), device=DEV)
    G = torch.rand((L, m), device=DEV) + 0.5               # one sign: sums of L terms, relative error below L 2^-24
    gt, _ = lram.backward(q, table, K, G, mode="merged")
    slot, w, _ = lram.neighbors(q[:1], K)
    ref = w[0].double()[:, None] * G.double().sum(0)[None]
    got = gt[slot[0].long()].double()
    assert ((got - ref).norm(dim=1) <= 1e-4 * ref.norm(dim=1)).all()
    rest = torch.ones(4 ** 8, dtype=torch.bool, device=DEV)
    rest[slot[0].long()] = False
    assert not gt[rest].any()


def test_all_lookups_non_finite():
    q = torch.full((70000, 8), float("inf"), device=DEV)
    gt, gq = lram.backward(q, torch.randn((4 ** 8, 32), device=DEV), (4,) * 8, torch.randn((70000, 32), device=DEV),
                           mode="merged")
    assert not gt.any() and not gq.any()


def test_other_callers():
    """An order-sized workspace, an order, the library's own scratch, saved lists and the activation layer."""
    K, L, m = (4, 4, 4, 4, 4, 4, 8, 8), 70001, 64
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    q = torch.rand((L, 8), generator=g, device=DEV) * torch.tensor(K, device=DEV)
    nbytes = lram.order_layout(L, 1)[0]
    assert lram.backward_workspace_bytes(L, 1, m, "merged") > nbytes
    small = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    table, G = _compare(q, K, m, torch.float32, 1, lambda *a: lram.backward(*a, mode="merged", workspace=small))
    _compare(q, K, m, torch.float32, 1, lambda *a: lram.backward(*a, mode="merged", order=lram.order(q, K)))

    # one buffer for both: the order is still there afterwards
    both = torch.empty(lram.backward_workspace_bytes(L, 1, m, "merged"), dtype=torch.uint8, device=DEV)
    both[:nbytes] = lram.order(q, K)[:nbytes]
    before = both.clone()
    _compare(q, K, m, torch.float32, 1, lambda *a: lram.backward(*a, mode="merged", order=both, workspace=both))
    assert torch.equal(both, before)

    def noalloc(q, table, K, G):
        gt = torch.zeros(table.shape, device=DEV)
        gq = torch.empty_like(q)
        lram.backward_noalloc(q, table, K, G, gt, gq, mode="merged")
        return gt, gq

    _compare(q, K, m, torch.float32, 1, noalloc)

    def saved(q, table, K, G):
        nl = lram.new_lists(q)
        lram.forward(q, table, K, lists=nl)
        return lram.backward(q, table, K, G, mode="merged", lists=nl)

    _compare(q, K, m, torch.float32, 1, saved)
    z = torch.randn((L, 16), generator=g, device=DEV)
    ta, za = lram.theta_backward(z, table, K, G, mode="atomic")
    tb, zb = lram.theta_backward(z, table, K, G, mode="merged")
    assert torch.equal(za, zb)
    assert ((ta.double() - tb.double()).norm(dim=1) <= 2e-5 * ta.double().norm(dim=1) + 1e-6 * ta.double().norm(dim=1).max()).all()


def _around(centres, spread, L, K, g):
    Kd = torch.tensor(K, device=DEV, dtype=torch.float64)
    mu = torch.rand((centres, 8), generator=g, device=DEV, dtype=torch.float64) * Kd
    q = mu[torch.randint(0, centres, (L,), generator=g, device=DEV)]
    q = torch.remainder(q + spread * torch.randn((L, 8), generator=g, device=DEV, dtype=torch.float64), Kd).float()
    return torch.where(q >= Kd.float(), torch.zeros_like(q), q).contiguous()


@pytest.mark.parametrize("m,dtype", [(32, torch.float32), (64, torch.bfloat16)])
@pytest.mark.parametrize("L,few", [(65536, True), (131072, True), (262144 + 3, True), (262144 + 3, False), (524288, True)])
def test_few_centres(L, few, m, dtype):
    """Lookups around few centres are merged batch by batch although their pairs may be sorted (the first word of the
    workspace tells), others and smaller batches are not; every caller's form of either."""
    gated = L >= (131072 if m == 64 else 262144)                         # otherwise nothing writes that word
    _say("few centres L=%d %s m=%d" % (L, few, m))
    K = (4, 4, 4, 4, 4, 4, 8, 8)
    g = torch.Generator(device=DEV)
    g.manual_seed(L + m)
    q = _around(16, 0.2, L, K, g) if few else torch.rand((L, 8), generator=g, device=DEV) * torch.tensor(K, device=DEV)
    q[::3, 5] = float("inf")                               # (not counted on either side)
    ws = torch.empty(lram.backward_workspace_bytes(L, 1, m, "merged"), dtype=torch.uint8, device=DEV)

    def word():
        return int(ws[:4].view(torch.int32).item())

    def plain(*a):
        ws.fill_(0xA5)
        return lram.backward(*a, mode="merged", workspace=ws)

    def ordered(q, table, K, G):
        ws.fill_(0xA5)
        return lram.backward(q, table, K, G, mode="merged", workspace=ws, order=lram.order(q, K))

    def saved(q, table, K, G):
        ws.fill_(0xA5)
        nl = lram.new_lists(q)
        lram.forward(q, table, K, lists=nl)
        return lram.backward(q, table, K, G, mode="merged", workspace=ws, lists=nl)

    _compare(q, K, m, dtype, 1, ordered)                   # (an order brings the gate with it at any size)
    assert word() == (L if few else 0)
    for form in (plain, saved):
        table, G = _compare(q, K, m, dtype, 1, form)
        assert gated == (word() in (0, L)) and (not gated or word() == (L if few else 0)), form
    z = torch.cat([torch.cos(q.double() * (2 * np.pi) / torch.tensor(K, device=DEV))[..., None],
                   torch.sin(q.double() * (2 * np.pi) / torch.tensor(K, device=DEV))[..., None]], -1)
    z = z.reshape(L, 16).float().nan_to_num(0.5).contiguous()
    ta, za = lram.theta_backward(z, table, K, G, mode="atomic")
    tb, zb = lram.theta_backward(z, table, K, G, mode="merged", workspace=ws)
    assert not gated or word() == (L if few else 0)
    assert torch.equal(za, zb)
    err, size = (ta.double() - tb.double()).norm(dim=1), ta.double().norm(dim=1)
    assert (err <= 2e-5 * size + 1e-6 * size.max()).all()


def test_long_runs():
    """One query below the sizes that the gate looks at: runs over many spans, no merge by batches."""
    K, L, m = (4,) * 8, 70001, 32
    q = torch.full((L, 8), 1.3, device=DEV) + torch.arange(8, device=DEV) * 0.11
    ws = torch.empty(lram.backward_workspace_bytes(L, 1, m, "merged"), dtype=torch.uint8, device=DEV)
    table = torch.randn((4 ** 8, m), device=DEV)
    G = torch.rand((L, m), device=DEV) + 0.5               # one sign: sums of L terms, relative error below L 2^-24
    gt, _ = lram.backward(q, table, K, G, mode="merged", workspace=ws)
    slot, w, _ = lram.neighbors(q[:1], K)
    ref = w[0].double()[:, None] * G.double().sum(0)[None]
    got = gt[slot[0].long()].double()
    assert ((got - ref).norm(dim=1) <= 1e-4 * ref.norm(dim=1)).all()


def test_gate_in_a_graph():
    """A captured backward chooses anew at every replay: uniform, clustered and again uniform queries in its buffer,
    with eager work between the replays."""
    K, L, m = (4, 4, 4, 4, 4, 4, 8, 8), 131072, 64
    g = torch.Generator(device=DEV)
    g.manual_seed(8)
    N = int(np.prod(K))
    batches = [torch.rand((L, 8), generator=g, device=DEV) * torch.tensor(K, device=DEV), _around(16, 0.2, L, K, g)]
    table = torch.randn((N, m), generator=g, device=DEV) * 0.02
    G = torch.randn((L, m), generator=g, device=DEV)
    ws = torch.empty(lram.backward_workspace_bytes(L, 1, m, "merged"), dtype=torch.uint8, device=DEV)
    q, gt, gq = batches[0].clone(), torch.zeros((N, m), device=DEV), torch.empty((L, 8), device=DEV)

    def step():
        lram.backward(q, table, K, G, grad_table=gt, grad_q=gq, mode="merged", workspace=ws)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for which in (0, 1, 0, 1):
        q.copy_(batches[which])
        gt.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert int(ws[:4].view(torch.int32).item()) == (L if which else 0)
        want, wq = lram.backward(q, table, K, G, mode="atomic")
        assert torch.equal(gq, wq)
        err, size = (gt.double() - want.double()).norm(dim=1), want.double().norm(dim=1)
        assert (err <= 2e-5 * size + 1e-6 * size.max()).all()


def _path(ws):
    """What the merged scatter did with a workspace that was 0xA5: "batch" -- an order of its own, whose header ends in
    a failure word of 0; "untouched"; "runs" -- sorted pairs, or the gate's choice between them and a batch merge, which
    writes the first word at most."""
    if int(ws[4:8].view(torch.int32).item()) == 0:
        return "batch"
    return "runs" if bool((ws[256:1024] != 0xA5).any()) else "untouched"


@pytest.mark.parametrize("m", [32, 64])
@pytest.mark.parametrize("L,K", [
    (65535, (4,) * 8),                     # the smallest batch that sorts, and one below
    (65536, (4,) * 8),
    (524288, (4,) * 8),                    # the largest, and one above
    (524289, (4,) * 8),
    (65536, (4, 4, 4, 4, 4, 8, 8, 8)),     # 2^19 rows, four pairs per row; one lookup less is below m = 32's line
    (131071, (4, 4, 4, 4, 8, 8, 8, 8)),
    (131072, (4, 4, 4, 4, 8, 8, 8, 8)),
    (100003, (4, 4, 4, 4, 8, 8, 8, 8)),    # between two and four
    (131071, (8, 8, 8, 8, 4, 4, 8, 4)),    # just below two
])
def test_line(L, K, m):
    """The rule's line (sizes, pairs per row) and every caller's form on both sides of it: with and without an order,
    lists and a query gradient."""
    N = int(np.prod(K))
    sorts = 65536 <= L <= 524288 and 32 * L >= (2 if m == 64 else 4) * N
    _say("line L=%d K=%s m=%d: %s" % (L, K, m, "runs" if sorts else "batch"))
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    q = torch.rand((L, 8), generator=g, device=DEV) * torch.tensor(K, device=DEV)
    order = lram.order(q, K)
    ws = torch.empty(max(lram.backward_workspace_bytes(L, 1, m, "merged"), lram.order_layout(L, 1)[0]),
                     dtype=torch.uint8, device=DEV)

    def call(q, table, K, G, **kw):
        ws.fill_(0xA5)
        return lram.backward(q, table, K, G, mode="merged", workspace=ws, **kw)

    table, G = _compare(q, K, m, torch.float32, 1, call)
    assert _path(ws) == ("runs" if sorts else "batch")
    _compare(q, K, m, torch.float32, 1, lambda *a: call(*a, order=order))
    assert _path(ws) == ("runs" if sorts else "untouched")
    nl = lram.new_lists(q)
    lram.forward(q, table, K, lists=nl)
    _compare(q, K, m, torch.float32, 1, lambda *a: call(*a, lists=nl, order=order))
    assert _path(ws) == ("runs" if sorts else "untouched")
    _compare(q, K, m, torch.float32, 1,
             lambda *a: (call(*a, want_grad_q=False)[0], lram.backward(*a, mode="atomic")[1]))
    assert _path(ws) == ("runs" if sorts else "batch")
