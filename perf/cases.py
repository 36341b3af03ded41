"""The work that users of this package have it do, as a list of cases with their inputs, one
pass through the public entry points, the bytes a pass cannot do without and the tolerance of
its results.

A case is one kind of step on one shape:
  path      "forward"  sample + mean (a model that reads fixed features, or inference)
            "replay"   mean over saved IDs (recomputation, evaluation on a fixed sample)
            "train"    forward with its IDs, then the backward into a kept gradient table
            "autograd" the differentiable operator: forward, loss gradient, dense x.grad
  graph     "power"    power-law out-degrees (Chung-Lu), targets by the same weights
            "kg"       (head, tail) pairs with Zipf-popular endpoints, both directions
  nodes, degree, top   number of nodes, mean and largest out-degree ("kg": degree only)
  dim, dtype           feature table [nodes, dim]
  batch, k1, k2, k3    seeds per call and fanouts (0 = no such hop)
  emit                 sampled IDs and per-slot means are wanted (False: only the mean)
  h1                   training: a gradient also comes back into the per-slot means
  weighted             per-edge weights
  master               16-bit table, fp32 gradient table
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2511_13645_amd import binding, synth
from paper_2511_13645_amd.autograd import fused_sample_mean

DEVICE = "cuda:0"
ALPHA = 0.8                      # exponent of the power-law degree weights, as in synth
TURNS = 4                        # batches that a state holds: consecutive passes take different seeds
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
MOST_BYTES = 1.0e9               # a drawn case needs at most this (the largest listed ones need more)

_PLAIN = {"path": "forward", "graph": "power", "nodes": 0, "degree": 0.0, "top": 0, "dim": 0, "dtype": "f32",
          "batch": 0, "k1": 0, "k2": 0, "k3": 0, "emit": True, "h1": False, "weighted": False, "master": False}


def _case(**kw):
    return {**_PLAIN, **kw}


def listed():
    products = dict(nodes=2_449_029, degree=50.5, top=17_000, dim=100)
    citation = dict(nodes=111_000_000, degree=14.5, top=100_000, dim=128, dtype="bf16")
    return [
        # online scoring of a handful of nodes: a call is all latency, no IDs are asked for
        _case(name="serve_8_seeds", **{**products, "dim": 128}, batch=8, k1=15, k2=10, emit=False),
        # unit-scale 1-hop training: everything but the launches is negligible
        _case(name="tiny_train", path="train", nodes=10_000, degree=10.0, top=200, dim=64, batch=1024, k1=10),
        # product graph, frozen features: forward with IDs and per-slot means
        _case(name="products_forward", **products, batch=1024, k1=15, k2=10),
        # the same with learnable rows under a layer-wise model (gradients into both levels)
        _case(name="products_train", path="train", **products, batch=1024, k1=15, k2=10, h1=True),
        # dense social graph: long rows, wide features, heavily shared gradient rows
        _case(name="social_train", path="train", nodes=232_965, degree=492.0, top=21_700, dim=602, batch=1024,
              k1=25, k2=10, h1=True),
        # knowledge-graph embedding table: 1-hop, hub entities
        _case(name="kg_train", path="train", graph="kg", nodes=2_500_000, degree=12.88, dim=128, batch=4096, k1=15),
        # a learnable table in a torch model: the operator's autograd function, dense gradient
        _case(name="arxiv_autograd", path="autograd", nodes=169_343, degree=13.7, top=13_000, dim=128, batch=1024,
              k1=25, k2=10),
        # web-scale citation graph, bf16 features: the headline batch and a saturating one
        _case(name="citation_forward", **citation, batch=4096, k1=15, k2=10),
        _case(name="citation_forward_64k", **citation, batch=65536, k1=15, k2=10),
        # 16-bit training: bf16 table, gradients and gradient table, a fifth of the citation graph (hubs short
        # enough that a bf16 running sum of a row's additions still means something)
        _case(name="citation_train_bf16", path="train", **{**citation, "nodes": 22_000_000, "top": 10_000}, batch=4096,
              k1=15, k2=10),
        # one hop more
        _case(name="three_hop_train", path="train", **products, batch=1024, k1=15, k2=10, k3=5),
        # per-edge weights
        _case(name="weighted_train", path="train", **products, batch=1024, k1=15, k2=10, weighted=True),
    ]


def draw(rng):
    """One more case of the same ranges: every path, type and option, sizes over their logarithms."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        path = rng.choice(("forward", "forward", "replay", "train", "train", "train", "autograd"))
        graph = rng.choice(("power", "power", "power", "kg"))
        hops = rng.choice((1, 2, 2, 2, 3)) if path != "autograd" else rng.choice((1, 2))
        nodes = log_int(10_000, 3_000_000)
        degree = round(math.exp(rng.uniform(math.log(4.0), math.log(500.0))), 1)
        dtype = rng.choice(("f32", "f32", "bf16", "f16"))
        dim = log_int(16, 640)
        if rng.random() < 0.7:                       # most models use widths of a multiple of four; the rest stay ragged
            dim = max(16, dim // 4 * 4)
        weighted = hops < 3 and path != "autograd" and rng.random() < 0.2
        master = dtype != "f32" and path == "train" and rng.random() < 0.5
        if path == "train" and (hops == 3 or weighted):
            dtype, master = "f32", False
        if path == "train" and dtype != "f32" and not master and dim % 2:
            dim += 1                                 # 16-bit gradient tables take even widths
        case = _case(path=path, graph=graph, nodes=nodes, degree=degree, top=0, dim=dim, dtype=dtype,
                     batch=log_int(1, 65536), k1=rng.randint(1, 30), k2=rng.randint(1, 20) if hops > 1 else 0,
                     k3=rng.randint(1, 8) if hops > 2 else 0, emit=rng.random() < 0.7,
                     h1=hops == 2 and path == "train" and rng.random() < 0.5, weighted=weighted, master=master)
        if graph == "power":
            case["top"] = max(int(degree * 4), min(nodes // 8, log_int(200, 20_000)))
        slots = case["batch"] * case["k1"] * max(1, case["k2"]) * max(1, case["k3"])
        if nodes * degree > 1.3e8 or nodes * dim > 2.6e8 or case["top"] > nodes // 4 or slots * dim > 4e8:
            continue
        # (a gradient table's hub rows take their additions one after another: smaller batches on "kg")
        if path in ("train", "autograd") and slots * dim > (8e7 if graph == "power" else 1.2e7):
            continue
        if work(case)["bytes"] > MOST_BYTES:
            continue
        if path in ("train", "autograd") and dtype != "f32" and not master:
            _, _, p = _degree_law(case)                  # a 16-bit gradient row is of use for a few additions only
            if _rows(case)[-1] * float(p.max()) > 24:
                continue
        return case


# ----------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------
def _power_graph(case, gen):
    """CSR of a directed graph with power-law expected out-degrees (1 % of the rows empty); targets are
    drawn by the same weights through the inverse of their continuous CDF; hubs are scattered over the IDs."""
    n = case["nodes"]
    c, i0 = synth.solve_power_law(n, case["degree"] / 0.99, case["top"], ALPHA)
    a, b, inv_a = synth._affine_bijection(n)
    rank = (torch.arange(n, dtype=torch.int64, device=DEVICE) * a + b) % n
    u = torch.rand(n, generator=gen, device=DEVICE, dtype=torch.float64)
    deg = torch.floor(c * (rank.double() + i0) ** -ALPHA + u).to(torch.int64)
    deg *= torch.rand(n, generator=gen, device=DEVICE) >= 0.01
    indptr = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(deg, 0, out=indptr[1:])
    edges = int(indptr[-1])
    indices = torch.empty(max(1, edges), dtype=torch.int32, device=DEVICE)
    lo, hi = i0 ** (1 - ALPHA), (n + i0) ** (1 - ALPHA)
    step = 1 << 27
    for e in range(0, edges, step):
        m = min(step, edges - e)
        u = torch.rand(m, generator=gen, device=DEVICE, dtype=torch.float64)
        j = ((u * (hi - lo) + lo) ** (1 / (1 - ALPHA)) - i0).to(torch.int64).clamp_(0, n - 1)
        indices[e:e + m] = ((j - b) * inv_a % n).to(torch.int32)
    return (indptr if edges > 10 ** 9 else indptr.to(torch.int32)), indices


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(int(seed))
    n, d, batch, k1, k2, k3 = (case[k] for k in ("nodes", "dim", "batch", "k1", "k2", "k3"))
    dtype = DTYPES[case["dtype"]]
    if case["graph"] == "kg":
        g = synth.kg_graph(n, int(n * case["degree"] / 2), seed=int(seed), device=DEVICE)
        indptr, indices = g.indptr, g.indices
    else:
        indptr, indices = _power_graph(case, gen)
    x = torch.empty((n, d), dtype=dtype, device=DEVICE)
    x.normal_(generator=gen)
    seeds = torch.randint(0, n, (TURNS, batch), generator=gen, device=DEVICE, dtype=torch.int32)
    fan = [k for k in (k1, k2, k3) if k > 0]
    s = {"case": dict(case), "fan": fan, "indptr": indptr, "indices": indices, "x": x, "turn": 0,
         "seeds": [t.contiguous() for t in seeds], "w": None}
    if case["weighted"]:
        s["w"] = torch.rand(indices.shape[0], generator=gen, device=DEVICE)
    if case["path"] == "replay":
        s["ids"] = [_forward(s, t, True)[1] for t in range(TURNS)]
    if case["path"] in ("train", "autograd"):
        s["g"] = torch.randn((batch, d), generator=gen, device=DEVICE).to(dtype)
    if case["path"] == "autograd":
        s["x"] = torch.nn.Parameter(x)
        s["ws"] = _workspace(case) if dtype == torch.float32 else None
    if case["path"] == "train":
        grad_type = torch.float32 if case["master"] else dtype
        s["gh"] = torch.randn((batch, k1, d), generator=gen, device=DEVICE).to(dtype) if case["h1"] else None
        s["grad_x"] = torch.zeros((n, d), dtype=grad_type, device=DEVICE)
        s["work"] = torch.empty((batch, k1, d), device=DEVICE) if len(fan) == 3 else None
        s["ws"] = _workspace(case) if dtype == torch.float32 and len(fan) == 2 and not case["weighted"] else None
    return s


def _workspace(case):
    need = binding.fsa_mean_bwd_workspace_bytes(case["batch"], case["k1"], case["k2"], case["dim"]) if case["k2"] else 0
    return torch.empty(need, dtype=torch.uint8, device=DEVICE) if need else None


# ----------------------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------------------
def _forward(s, turn, emit):
    """(means, IDs): both as the entry point of the case returns them."""
    a = (s["indptr"], s["indices"])
    b = (s["x"], s["seeds"][turn], s["fan"], 0)
    if len(s["fan"]) == 3:
        r = binding.fsa_sample_mean3_fwd(*a, *b, emit_ids=emit)
        return (r["out"], r["out_h1"], r["out_m1"]), (r["ids1"], r["ids2"], r["ids3"])
    if s["w"] is not None:
        out, h1, i1, i2, w1, w2 = binding.fsa_sample_wmean_fwd(*a, s["w"], *b, emit_h1=emit, emit_ids=emit)
        return (out, h1), (i1, i2, w1, w2)
    out, h1, i1, i2 = binding.fsa_sample_mean_fwd(*a, *b, emit_h1=emit, emit_ids=emit)
    return (out, h1), (i1, i2)


def _replay(s, ids):
    if len(s["fan"]) == 3:
        r = binding.fsa_mean3_replay_fwd(s["x"], *ids)
        return r["out"], r["out_h1"], r["out_m1"], r["cnt2"]
    if s["w"] is not None:
        i1, i2, w1, w2 = ids
        return binding.fsa_wmean_replay_fwd(s["x"], i1, w1, i2, w2)
    return binding.fsa_mean_replay_fwd(s["x"], *ids)


def _backward(s, ids):
    g, gh, grad_x = s["g"], s["gh"], s["grad_x"]
    if len(s["fan"]) == 3:
        return binding.fsa_mean3_bwd(g, *ids, grad_m1=g, grad_x=grad_x, work=s["work"])
    if s["w"] is not None:
        i1, i2, w1, w2 = ids
        return binding.fsa_wmean_bwd(g, i1, w1, i2, w2, gh, grad_x=grad_x)
    if g.dtype != torch.float32:
        return binding.fsa_mean_bwd_lp(g, *ids, gh, grad_x=grad_x)
    if s["ws"] is not None:
        return binding.fsa_mean_bwd_ws(g, *ids, gh, grad_x=grad_x, workspace=s["ws"])
    return binding.fsa_mean_bwd(g, *ids, gh, grad_x=grad_x)


def run(s):
    path, turn = s["case"]["path"], s["turn"]
    s["turn"] = (turn + 1) % TURNS
    if path == "forward":
        return _forward(s, turn, s["case"]["emit"])
    if path == "replay":
        return _replay(s, s["ids"][turn])
    if path == "train":
        means, ids = _forward(s, turn, True)
        return means, ids, _backward(s, ids)
    x = s["x"]
    x.grad = None
    out, _, _, _ = fused_sample_mean(x, s["indptr"], s["indices"], s["seeds"][turn], s["fan"], 0, workspace=s["ws"])
    out.backward(s["g"])
    return out, x.grad


# ----------------------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------------------
def _degree_law(case):
    """Sample points of the degree law: (expected degrees, nodes each stands for, probability of one as a target)."""
    n = case["nodes"]
    edge = np.unique(np.concatenate([[0.0], np.geomspace(1.0, n, 4000).round()]))
    lo, hi = edge[:-1], edge[1:]
    if case["graph"] == "kg":
        w = ((lo + hi) / 2 + 0.5) ** -1.1
        w *= case["degree"] * n / float((w * (hi - lo)).sum())
    else:
        c, i0 = synth.solve_power_law(n, case["degree"] / 0.99, case["top"], ALPHA)
        w = c * ((lo + hi) / 2 + i0) ** -ALPHA
    m = hi - lo
    return w, m, w / float((w * m).sum())


def _expect_rows(w, k):
    """Expected min(k, degree) of nodes of expected degree w."""
    f = np.floor(w)
    r = w - f
    return 0.99 * ((1 - r) * np.minimum(k, f) + r * np.minimum(k, f + 1))


def _rows(case):
    """Expected number of slots with an ID after each hop."""
    w, m, p = _degree_law(case)
    rows, total = [], float(case["batch"])
    for k in (case["k1"], case["k2"], case["k3"]):
        if k > 0:
            got = _expect_rows(w, k)
            total *= float((got * m * p).sum()) if rows else float((got * m).sum() / m.sum())
            rows.append(total)
    return rows


def work(case):
    w, m, p = _degree_law(case)
    e = 4 if case["dtype"] == "f32" else 2
    d, batch = case["dim"], case["batch"]
    fan = [k for k in (case["k1"], case["k2"], case["k3"]) if k > 0]
    ptr = 16 if case["nodes"] * case["degree"] > 10 ** 9 else 8
    rows = _rows(case)
    distinct = float((m * (1 - np.exp(-rows[-1] * p))).sum())
    row = d * e
    nbytes = distinct * row + batch * row                            # leaf rows in, means out
    if case["path"] == "replay":
        nbytes += 4 * sum(rows)
    else:
        nbytes += batch * (4 + ptr) + 4 * sum(rows) + ptr * sum(rows[:-1])
    if case["weighted"]:
        nbytes += 4 * sum(rows)
    slots = [batch * int(np.prod(fan[:i + 1])) for i in range(len(fan))]
    ids_out = case["path"] in ("train", "autograd") or (case["path"] == "forward" and case["emit"])
    if ids_out:
        nbytes += 4 * sum(slots) * (2 if case["weighted"] else 1)
    if len(fan) > 1 and (len(fan) == 3 or case["path"] == "replay" or (ids_out and case["path"] != "autograd")):
        nbytes += slots[0] * row                                     # per-slot means
    flops = rows[-1] * d
    if len(fan) == 3:
        nbytes += batch * row + float((m * (1 - np.exp(-rows[0] * p))).sum()) * row
    if case["path"] in ("train", "autograd"):
        ge = 4 if case["master"] or case["dtype"] == "f32" else 2
        nbytes += 4 * sum(slots) * (2 if case["weighted"] else 1) + batch * row + (slots[0] * row if case["h1"] else 0)
        nbytes += case["nodes"] * d * ge if case["path"] == "autograd" else distinct * d * ge * 2
        flops += rows[-1] * d * 2
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times the error measured against the same path in 64 bits (the largest over listed and drawn cases:
    forward 1.2e-7 f32, 1.7e-3 bf16, 2.4e-4 f16; gradient tables 9.3e-7 in f32, 2.6e-3 in 16 bits, whose running
    sums are rounded at every addition, so that a single element of a hub row can be far off)."""
    if case["path"] in ("train", "autograd") and case["dtype"] != "f32" and not case["master"]:
        return {"rel": 1e-2, "max": 9e-1}
    return {"f32": {"rel": 4e-6, "max": 4.5e-4} if case["path"] in ("train", "autograd") else {"rel": 5e-7, "max": 4e-6},
            "bf16": {"rel": 7e-3, "max": 1.6e-2}, "f16": {"rel": 1e-3, "max": 2.6e-3}}[case["dtype"]]
