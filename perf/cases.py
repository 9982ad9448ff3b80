"""Cases that stand for the work users of this package have it do on one MI355X.

A case names an operation, a torus K, the value width m, the table's dtype, the
batch B x H of lookups and the kind of queries; ``run`` makes one pass through
the package's public entry points.  ``exact`` computes the same outputs in 64
bits with torch alone: it enumerates the lattice points around every query
straight from the definition (closest point, then every point of Lambda within
reach), keeps those that the documented fp32 distance selects, and forms
weights, sums and gradients in fp64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2107_03474_amd as lram
from paper_2107_03474_amd.memory_layer import MemorySubnetwork

DEV = "cuda"
STD = 0.02            # value tables are N(0, 0.02^2)
CENTRES = 4096        # clusters of the "zipf" queries, ranked Zipf(1.1)
SIGMA = 0.3           # their spread, and that of the "gmm" queries' 64 clusters
ADAM_STEP = 100       # the optimiser case is in the middle of a training run


def _K(case):
    return tuple(int(v) for v in case["K"].split())


def _N(case):
    return int(np.prod(_K(case)))


def _L(case):
    return case["B"] * case["H"]


def _uniform_K(k):
    return " ".join([str(k)] * 8)


def listed():
    return [
        # one token of a width-512 model at inference: 32 heads, latency is all there is
        {"name": "token", "op": "theta_forward", "K": _uniform_K(8), "m": 64, "dtype": "bf16", "B": 1, "H": 32,
         "queries": "uniform"},
        # the smallest training configuration: K = 4, 4,096 uniform lookups
        {"name": "k4-step", "op": "step", "K": _uniform_K(4), "m": 32, "dtype": "f32", "B": 4096, "H": 1,
         "queries": "uniform"},
        # autograd on an uneven torus with an odd batch, the lists kept for the backward
        {"name": "autograd-odd", "op": "lookup", "K": "4 6 4 8 4 4 6 4", "m": 64, "dtype": "bf16", "B": 333, "H": 7,
         "queries": "gmm"},
        # the neighbour lists themselves (indices, weights, distances), an odd number of lookups, K = 14
        {"name": "lists", "op": "neighbors", "K": _uniform_K(14), "m": 32, "dtype": "f32", "B": 100003, "H": 1,
         "queries": "uniform", "k": 32},
        # inference over a 4.3 GB fp32 table: K = 8, 65,536 x 8 uniform lookups
        {"name": "forward-k8", "op": "forward", "K": _uniform_K(8), "m": 64, "dtype": "f32", "B": 65536, "H": 8,
         "queries": "uniform", "k": 32},
        # every point of the support (no truncation), forward and backward, a ragged batch
        {"name": "untruncated", "op": "step", "K": _uniform_K(8), "m": 32, "dtype": "f32", "B": 9999, "H": 3,
         "queries": "uniform", "k": 0},
        # the activation layer trained through autograd at a memory size of the paper (2^20 locations):
        # 32 sequences of 256 tokens, 32 heads each
        {"name": "train-theta", "op": "theta", "K": "4 4 4 4 8 8 8 8", "m": 64, "dtype": "f32", "B": 8192, "H": 32,
         "queries": "zipf"},
        # a whole optimiser step on 2^18 locations: forward, backward, Adam on the touched rows
        {"name": "train-adam", "op": "adam", "K": "4 4 4 4 4 4 8 8", "m": 64, "dtype": "f32", "B": 8192, "H": 32,
         "queries": "zipf"},
        # access statistics of a batch on 2^22 locations
        {"name": "statistics", "op": "statistics", "K": "4 4 8 8 8 8 8 8", "m": 64, "dtype": "f32", "B": 8192, "H": 32,
         "queries": "zipf"},
        # projected hidden states (one Gaussian blob of queries, so rows repeat), forward and backward
        {"name": "projection", "op": "step", "K": "10 10 10 10 8 8 8 8", "m": 64, "dtype": "bf16", "B": 8192, "H": 16,
         "queries": "projection"},
        # the memory subnetwork at inference: w = 2048, 4,096 vectors, bf16 dense layers and table
        {"name": "subnetwork", "op": "subnetwork", "K": _uniform_K(8), "m": 64, "dtype": "bf16", "B": 4096, "H": 128,
         "queries": "uniform"},
        # the largest: 4.19 M lookups, half of them clustered, ordered once for the forward and the backward
        {"name": "large-step", "op": "ordered", "K": _uniform_K(10), "m": 32, "dtype": "bf16", "B": 262144, "H": 16,
         "queries": "zipf"},
    ]


def draw(rng):
    """The ranges of the listed cases: tori from 2^13 to 4e7 locations, some of them uneven, both value widths and
    dtypes, 32 to 1 M lookups, every operation but the subnetwork and every kind of queries."""
    while True:
        if rng.random() < 0.5:
            K = [rng.choice([4, 6, 8])] * 8
        else:
            K = [rng.choice([2, 4, 4, 6, 6, 8, 8, 10, 12]) for _ in range(8)]
        N = int(np.prod(K))
        if 1 << 13 <= N <= 40_000_000:
            break
    op = rng.choice(["forward", "forward", "step", "step", "ordered", "lookup", "theta_forward", "theta", "adam",
                     "neighbors", "statistics"])
    m = rng.choice([32, 64])
    H = rng.choice([1, 2, 3, 7, 8, 16, 32])
    top = {"lookup": 30_000, "theta": 300_000, "neighbors": 300_000, "adam": 300_000}.get(op, 1_000_000)
    L = math.exp(rng.uniform(math.log(32), math.log(top)))
    k = 32
    if op in ("forward", "step", "neighbors") and rng.random() < 0.3:
        k = rng.choice([16, 64, 0])
        L = min(L, 100_000)
    B = max(1, round(L / H))
    if N * m > 1 << 29 and op in ("theta", "adam"):
        m = 32
    c = {"op": op, "K": " ".join(map(str, K)), "m": m, "dtype": rng.choice(["f32", "bf16"]), "B": B, "H": H,
         "queries": rng.choice(["uniform", "uniform", "gmm", "zipf", "projection"])}
    if op in ("forward", "step", "neighbors"):
        c["k"] = k
    return c


# ---------------------------------------------------------------------------
# Inputs.

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _queries(case, g):
    """Queries [B, H, 8] fp32 in [0, K_i)."""
    B, H = case["B"], case["H"]
    n = B * H
    Kd = torch.tensor(_K(case), dtype=torch.float64, device=DEV)

    def uni(r):
        return torch.rand((r, 8), generator=g, device=DEV, dtype=torch.float64) * Kd

    def noise(r):
        return torch.randn((r, 8), generator=g, device=DEV, dtype=torch.float64)

    kind = case["queries"]
    if kind == "uniform":
        q = uni(n)
    elif kind == "gmm":
        mu = uni(64)
        comp = torch.randint(0, 64, (n,), generator=g, device=DEV)
        q = mu[comp] + SIGMA * noise(n)
    elif kind == "projection":
        W = torch.randn((1024, H * 8), generator=g, device=DEV) / 32.0
        X = torch.randn((B, 1024), generator=g, device=DEV)
        q = (X @ W).double().reshape(n, 8)
    else:  # half uniform, half around centres of Zipf-distributed popularity
        mu = uni(CENTRES)
        p = torch.arange(1, CENTRES + 1, device=DEV, dtype=torch.float64).pow(-1.1).cumsum(0)
        comp = torch.searchsorted(p, torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * p[-1])
        clustered = torch.rand((n, 1), generator=g, device=DEV) < 0.5
        q = torch.where(clustered, mu[comp.clamp(max=CENTRES - 1)] + SIGMA * noise(n), uni(n))
    q = torch.remainder(q, Kd).float()
    return torch.where(q >= Kd.float(), torch.zeros_like(q), q).reshape(B, H, 8).contiguous()


def _theta_input(case, q, g):
    """z [B, H, 16]: complex numbers whose arguments give q, with Rayleigh moduli."""
    t = q.double() * (2.0 * math.pi) / torch.tensor(_K(case), dtype=torch.float64, device=DEV)
    n = torch.randn(q.shape + (2,), generator=g, device=DEV, dtype=torch.float64)
    r = (0.5 * n.square().sum(-1)).sqrt()
    return torch.stack([r * t.cos(), r * t.sin()], -1).flatten(-2).float().contiguous()


def _table(case, g):
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    N, m = _N(case), case["m"]
    t = torch.empty((N, m), dtype=dt, device=DEV)
    for s in range(0, N, 1 << 22):
        t[s:s + (1 << 22)] = torch.randn((min(1 << 22, N - s), m), generator=g, device=DEV) * STD
    return t


def prepare(case, seed):
    g = _gen(seed)
    op = case["op"]
    s = {"case": case, "op": op, "K": _K(case)}
    lead = (case["B"], case["H"])
    if op == "subnetwork":
        w = case["H"] * 16
        table = _table(case, g)
        state = torch.random.get_rng_state(), torch.cuda.get_rng_state()
        torch.manual_seed(seed)
        net = MemorySubnetwork(w, s["K"], dtype=torch.bfloat16, table=table)
        # normalised queries of a trained layer: running statistics near those of the features
        with torch.no_grad():
            net.inp.weight.copy_(torch.randn((w, w), generator=g, device=DEV) / math.sqrt(w))
            net.bn.running_var.copy_(1.0 + 0.1 * torch.rand(w, generator=g, device=DEV))
        torch.random.set_rng_state(state[0])
        torch.cuda.set_rng_state(state[1])
        s["net"] = net.eval()
        s["x"] = torch.randn((case["B"], w), generator=g, device=DEV).to(torch.bfloat16)
        return s
    q = _queries(case, g)
    if op.startswith("theta"):
        s["z"] = _theta_input(case, q, g)
    else:
        s["q"] = q
    if op not in ("neighbors", "statistics"):
        s["table"] = _table(case, g)
    if op in ("step", "ordered", "lookup", "theta", "adam"):
        s["g"] = torch.randn(lead + (case["m"],), generator=g, device=DEV)
    if op in ("step", "ordered", "adam"):  # the accumulator that a training loop keeps
        s["gtab"] = torch.zeros((_N(case), case["m"]), dtype=torch.float32, device=DEV)
    if op == "adam":
        s["m1"] = torch.randn((_N(case), case["m"]), generator=g, device=DEV)
        s["m2"] = 0.5 + torch.rand((_N(case), case["m"]), generator=g, device=DEV)
        s["touched"] = torch.zeros(_N(case), dtype=torch.uint8, device=DEV)
    if op == "statistics":
        s["hist"] = torch.zeros(_N(case), dtype=torch.float32, device=DEV)
        s["touched"] = torch.zeros(_N(case), dtype=torch.uint8, device=DEV)
    if op == "lookup":
        s["q"].requires_grad_(True)
        s["table"].requires_grad_(True)
        s["g"] = s["g"].to(s["table"].dtype)
    if op == "theta":
        s["z"].requires_grad_(True)
        s["table"].requires_grad_(True)
        s["g"] = s["g"].to(s["table"].dtype)
    if op == "ordered":
        s["order"] = torch.empty(lram.order_layout(*lead)[0], dtype=torch.uint8, device=DEV)
    return s


# ---------------------------------------------------------------------------
# One pass.

def run(s):
    op, K, case = s["op"], s["K"], s["case"]
    if op == "forward":
        return lram.forward(s["q"], s["table"], K, k=case["k"])
    if op == "theta_forward":
        return lram.theta_forward(s["z"], s["table"], K)
    if op == "neighbors":
        return lram.neighbors(s["q"], K, k=case["k"])
    if op == "step":
        k = case.get("k", 32)
        out = lram.forward(s["q"], s["table"], K, k=k)
        gt, gq = lram.backward(s["q"], s["table"], K, s["g"], grad_table=s["gtab"], k=k)
        return {"out": out, "grad_table": gt, "grad_q": gq}
    if op == "ordered":
        o = lram.order(s["q"], K, s["order"])
        out = lram.forward(s["q"], s["table"], K, order=o)
        gt, gq = lram.backward(s["q"], s["table"], K, s["g"], grad_table=s["gtab"], order=o)
        return {"out": out, "grad_table": gt, "grad_q": gq}
    if op == "lookup":
        out = lram.lookup(s["q"], s["table"], K, save_lists=True)
        gq, gt = torch.autograd.grad(out, (s["q"], s["table"]), s["g"])
        return {"out": out, "grad_table": gt, "grad_q": gq}
    if op == "theta":
        out = lram.theta(s["z"], s["table"], K)
        gz, gt = torch.autograd.grad(out, (s["z"], s["table"]), s["g"])
        return {"out": out, "grad_table": gt, "grad_z": gz}
    if op == "adam":
        out = lram.forward(s["q"], s["table"], K)
        gt, gq = lram.backward(s["q"], s["table"], K, s["g"], grad_table=s["gtab"])
        lram.mark_touched(s["q"], K, s["touched"])
        lram.sparse_adam(s["table"], s["gtab"], s["m1"], s["m2"], ADAM_STEP, touched=s["touched"])
        return {"out": out, "grad_q": gq, "table": s["table"], "m1": s["m1"], "m2": s["m2"]}
    if op == "statistics":
        lram.access_histogram(s["q"], K, s["hist"])
        lram.mark_touched(s["q"], K, s["touched"])
        st = lram.access_stats(s["hist"])
        return {"hist": s["hist"], "touched": s["touched"], "used": st["used"], "kl": st["kl"], "total": st["total"]}
    if op == "subnetwork":
        with torch.no_grad():
            return s["net"](s["x"])
    raise ValueError(op)


def _distinct_rows(case):
    """Rows of the table that a batch touches, each counted once (expected value for uniform queries; clustered ones
    repeat rows: measured shares)."""
    N, L = _N(case), _L(case)
    pairs = L * {16: 16, 32: 32, 64: 61, 0: 65}[case.get("k", 32)]
    share = {"uniform": 1.0, "gmm": 0.3, "zipf": 0.52, "projection": 0.13}[case["queries"]]
    return N * -math.expm1(-share * pairs / N)


def work(case):
    """Each input read and each output written once; the table and its gradient by their touched rows.  Operations:
    the kernel at the list's points, the weighted sum, and the dot products and row updates of the backward."""
    N, L, m, op = _N(case), _L(case), case["m"], case["op"]
    st = 4 if case["dtype"] == "f32" else 2
    U = _distinct_rows(case)
    nk = {16: 16, 32: 32, 64: 64, 0: 65}[case.get("k", 32)]
    inp = 64 if op.startswith("theta") else 32
    search = 24.0 * nk * L
    gather = 2.0 * nk * m * L
    fwd = L * (inp + m * st) + U * m * st
    bwd = L * (inp + 4 * m + inp) + U * (m * st + 8 * m)
    if op in ("forward", "theta_forward"):
        return {"bytes": fwd, "flops": search + gather}
    if op == "neighbors":
        return {"bytes": L * (32 + 12 * (256 if case["k"] == 0 else case["k"])), "flops": search}
    if op in ("step", "ordered"):
        return {"bytes": fwd + bwd, "flops": 2 * search + 3 * gather}
    if op in ("lookup", "theta"):  # a dense gradient table is written
        return {"bytes": fwd + L * (inp + st * m + inp) + U * m * st + N * m * st, "flops": 2 * search + 3 * gather}
    if op == "adam":  # gradient rows stay inside the step; moments and values are read and written
        return {"bytes": fwd + L * (inp + 4 * m + inp) + U * m * (16 + st) + N, "flops": 2 * search + 3 * gather}
    if op == "statistics":
        return {"bytes": L * 32 + U * 9 + 4 * N, "flops": search}
    w = case["H"] * 16
    dense = case["B"] * w * (w + 4 * w) * 2.0
    return {"bytes": 2.0 * (5 * w * w + 2 * case["B"] * w) + U * m * st, "flops": dense + search + gather}


def tolerance(case):
    op = case["op"]
    bf = case["dtype"] == "bf16"
    if op == "neighbors":
        # the documented fp32 recipe: lists, weights and distances are the same bits
        return "exact"
    if op == "statistics":
        # sums of up to thousands of fp32 weights by atomics: rel 6.8e-7 from call to call
        return {"rel": 4e-6, "max": 2e-5}
    if op == "subnetwork":
        return {"rel": 8e-3, "max": 8e-2}
    # fp32 sums in another order differ by up to rel 2.2e-7, max 1.1e-5 (row sums of up to a few thousand terms);
    # bf16 results are rounded once (rel 1.7e-3) and a sum next to a rounding boundary may go either way
    return {"rel": 4e-3 if bf else 1e-6, "max": 4e-2 if bf else 1e-4}


# ---------------------------------------------------------------------------
# The same in 64 bits.

def _lattice_shells():
    """The 1 + 240 + 2160 points of Lambda = {k in (2Z)^8 u (2Z+1)^8 : sum k = 0 mod 4} with |k|^2 <= 16."""
    ev = np.stack(np.meshgrid(*([np.arange(-4, 5, 2)] * 8), indexing="ij"), -1).reshape(-1, 8)
    ev = ev[((ev ** 2).sum(1) <= 16) & (ev.sum(1) % 4 == 0)]
    od = np.stack(np.meshgrid(*([np.arange(-3, 4, 2)] * 8), indexing="ij"), -1).reshape(-1, 8)
    od = od[((od ** 2).sum(1) <= 16) & (od.sum(1) % 4 == 0)]
    p = np.concatenate([ev, od])
    assert p.shape[0] == 2401
    return p


def _closest(x):
    """A lattice point within the covering radius of x [n, 8] (fp64): the better of the two D8 cosets' decodings."""
    def d8(y):
        r = y.round()
        d = y - r
        j = d.abs().argmax(1, keepdim=True)
        odd = (r.sum(1, keepdim=True) % 2) != 0
        fix = torch.where(d.gather(1, j) > 0, 1.0, -1.0).to(r.dtype) * odd
        return r.scatter_add(1, j, fix)

    a, b = 2 * d8(x / 2), 2 * d8((x - 1) / 2) + 1
    return torch.where(((x - a) ** 2).sum(1, keepdim=True) <= ((x - b) ** 2).sum(1, keepdim=True), a, b)


_SHELLS = {}


def _lists(q, K, k):
    """(slot int64 [n, w], d2 fp32 recipe [n, w], x - k fp64 [n, w, 8], real [n, w]) of the closest w = k points (k = 0:
    the whole support, w = 256) in the documented order, padding last."""
    if "p" not in _SHELLS:
        _SHELLS["p"] = torch.from_numpy(_lattice_shells()).to(DEV)
    p = _SHELLS["p"]
    Kt = torch.tensor(K, device=DEV)
    x = torch.fmod(2.0 * q, 2.0 * Kt.float())          # exact
    c = _closest(x.double()).long()
    s = None
    for i in range(8):
        e = x[:, i:i + 1] - (c[:, i:i + 1] + p[None, :, i]).float()
        e = e * e
        s = e if s is None else s + e
    w = 256 if k == 0 else k
    n = min(2401, 256 if k == 0 else k + 32)           # room for equal distances at the last place
    d, idx = s.topk(n, dim=1, largest=False)
    pts = c[:, None, :] + p[idx]
    eps = pts[..., :1] & 1
    Y = torch.remainder((pts - eps) >> 1, Kt)
    slot = torch.zeros_like(idx)
    for i in range(7):
        slot = (slot + Y[..., i]) * (Kt[i + 1] if i < 6 else Kt[7] // 2)
    slot = eps[..., 0] * (int(np.prod(K)) // 2) + slot + (Y[..., 7] >> 1)
    o = ((d.view(torch.int32).long() << 32) | slot).argsort(dim=1, stable=True)[:, :w]
    d, slot = d.gather(1, o), slot.gather(1, o)
    err = x.double()[:, None, :] - pts.gather(1, o[..., None].expand(-1, -1, 8)).double()
    return slot, d, err, d < 8.0


def _theta_query(z, K):
    a, b = z[..., 0::2].double(), z[..., 1::2].double()
    cK = torch.tensor([v / (2.0 * math.pi) for v in K], dtype=torch.float64, device=DEV)
    r = (a * a + b * b).sqrt()
    return (torch.atan2(b, a) * cK).float(), a, b, r, 1.0 / (1.0 / r).sum(-1), cK


def _chunks(L, k):
    step = 4096 if k == 0 else 16384
    return [(b, min(L, b + step)) for b in range(0, L, step)]


def exact(case, seed):
    s = prepare(case, seed)
    op, K, m, N, L = s["op"], s["K"], case["m"], _N(case), _L(case)
    k = case.get("k", 32)
    lead = (case["B"], case["H"])
    f64 = dict(dtype=torch.float64, device=DEV)
    if op == "subnetwork":
        net = s["net"]
        d = torch.Tensor.double
        with torch.no_grad():
            h = d(s["x"]) @ d(net.inp.weight).T + d(net.inp.bias)
            h = (h - d(net.bn.running_mean)) / (d(net.bn.running_var) + net.bn.eps).sqrt() * d(net.bn.weight) + d(net.bn.bias)
            z = h.reshape(L, 16).float()
            th = torch.empty((L, m), **f64)
            for b, e in _chunks(L, k):
                q, _, _, _, sc, _ = _theta_query(z[b:e], K)
                slot, _, err, real = _lists(q, K, k)
                u = 1.0 - err.square().sum(-1) / 8.0
                th[b:e] = sc[:, None] * ((u ** 4 * real)[..., None] * net.table.data[slot].double()).sum(1)
            return th.reshape(case["B"], -1) @ d(net.out.weight).T + d(net.out.bias)
    if op == "neighbors":
        w = 256 if k == 0 else k
        slots, ws, ds = [], [], []
        for b, e in _chunks(L, k):
            slot, d, err, real = _lists(s["q"].reshape(-1, 8)[b:e], K, k)
            u = 1.0 - err.square().sum(-1) / 8.0
            slots.append(torch.where(real, slot, torch.full_like(slot, -1)))
            ws.append(torch.where(real, u ** 4, torch.zeros_like(u)))
            ds.append(torch.where(real, err.square().sum(-1), torch.full_like(u, math.inf)))
        return tuple(torch.cat(v).reshape(lead + (w,)) for v in (slots, ws, ds))
    th = op.startswith("theta")
    inp = (s["z"] if th else s["q"]).detach().reshape(L, -1)
    table = s["table"].detach() if "table" in s else None
    backward = op in ("step", "ordered", "lookup", "theta", "adam")
    out = torch.empty((L, m), **f64) if table is not None else None
    gin = torch.empty((L, 16 if th else 8), **f64) if backward else None
    gtab = torch.zeros((N, m), **f64) if backward else None
    hist = torch.zeros(N, **f64) if op == "statistics" else None
    touched = torch.zeros(N, dtype=torch.uint8, device=DEV) if op == "statistics" else None
    G = s["g"].detach().reshape(L, m) if backward else None
    for b, e in _chunks(L, k):
        if th:
            q, za, zb, r, sc, cK = _theta_query(inp[b:e], K)
        else:
            q, sc = inp[b:e], torch.ones(e - b, **f64)
        slot, _, err, real = _lists(q, K, k)
        u = torch.where(real, 1.0 - err.square().sum(-1) / 8.0, torch.zeros((), **f64))
        w = u ** 4
        if op == "statistics":
            hist.index_add_(0, slot[real], w[real])
            touched[slot[real]] = 1
            continue
        V = table[slot].double()
        out[b:e] = sc[:, None] * (w[..., None] * V).sum(1)
        if backward:
            g = G[b:e].double()
            dot = (V * g[:, None, :]).sum(-1)
            dq = ((-2.0 * u ** 3 * dot)[..., None] * err).sum(1)
            ws = w * sc[:, None]
            gtab.index_add_(0, slot.reshape(-1), (ws[..., None] * g[:, None, :]).reshape(-1, m))
            if th:
                ds = (w * dot).sum(1)[:, None] * sc[:, None] ** 2
                dqs = dq * sc[:, None] * cK
                gin[b:e, 0::2] = ds * za / r ** 3 - dqs * zb / r ** 2
                gin[b:e, 1::2] = ds * zb / r ** 3 + dqs * za / r ** 2
            else:
                gin[b:e] = dq
    if op == "statistics":
        tot = hist.sum()
        pr = hist[hist > 0] / tot
        return {"hist": hist, "touched": touched, "used": float((hist > 0).double().mean()),
                "kl": float((pr * (pr * N).log()).sum()), "total": float(tot)}
    out = out.reshape(lead + (m,))
    if op in ("forward", "theta_forward"):
        return out
    gin = gin.reshape(lead + (-1,))
    if op == "adam":
        hit = (gtab != 0).any(1)
        b1, b2 = 0.9, 0.999
        m1, m2, t = s["m1"].double(), s["m2"].double(), table.double()
        n1 = torch.where(hit[:, None], b1 * m1 + (1 - b1) * gtab, m1)
        n2 = torch.where(hit[:, None], b2 * m2 + (1 - b2) * gtab * gtab, m2)
        step = 1e-3 * (n1 / (1 - b1 ** ADAM_STEP)) / ((n2 / (1 - b2 ** ADAM_STEP)).sqrt() + 1e-8)
        t = torch.where(hit[:, None], t - step, t)
        return {"out": out, "grad_q": gin, "table": t, "m1": n1, "m2": n2}
    return {"out": out, "grad_table": gtab, ("grad_z" if th else "grad_q"): gin}
