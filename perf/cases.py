"""The workloads by which this library's speed is judged: the graph shapes of the five
configurations in ``workloads/graphs.py`` (node counts, degree laws, value normalisations,
feature widths), run through the public entry points the way a GNN program runs them, and the
ranges those shapes stand for.

A case holds
  graph   "undirected" (random pairs, both directions), "powerlaw" (out-degree density ~
          d**-2.1 with uniform targets) or "clustered" (the same with 64 blocks of ids, 80 % of
          the entries inside the row's own block); every row has a self-loop, columns are
          sorted and unique inside a row
  N, mean, dmax    nodes, mean stored entries per row (self-loop included), largest degree
  F       feature columns; X and Y are dense with row stride F
  call    "forward" (es_spmm_ws with a kept workspace), "backward" (es_spmm_backward, the
          transposed product without any extra structure) or "pull" (es_spmm_backward_pull on
          the transposed graph that a training program builds once)
  mode, W, seed    the sampler
  values  "sym" (1/sqrt(d_i d_j)), "mean" (1/d_i) or "unit" (no value array)
  norm    row factor applied in the kernel
Graphs are generated on the GPU from the seed.
"""
import math

import torch

import paper_2104_10716_amd as es

_EXPONENT = 2.1
_BLOCKS = 64
_P_INTRA = 0.8


def _case(name, graph, N, mean, dmax, F, call, mode, W, seed, values, norm="none"):
    c = dict(graph=graph, N=N, mean=float(mean), dmax=dmax, F=F, call=call, mode=mode, W=W, seed=seed,
             values=values, norm=norm)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one aggregation of a GCN on a graph of a few thousand nodes: launches and the host path
        _case("tiny_exact", "undirected", 2_708, 5, 0, 16, "forward", "full", 0, 0, "sym"),
        # a citation graph of some 20k papers, hidden width 32, small enough for every cache
        _case("small_bucket_w16", "powerlaw", 19_717, 4.5, 171, 32, "forward", "bucket", 16, 0, "sym"),
        # inference on a mid-size citation graph: short rows, X larger than an L2
        _case("citation_fastrand_w16", "powerlaw", 170_000, 14, 13_000, 128, "forward", "fastrand", 16, 0, "sym"),
        # the same graph with the exact product: the skewed rows decide the tail
        _case("citation_exact", "powerlaw", 170_000, 14, 13_000, 128, "forward", "full", 0, 0, "sym"),
        # one training step's gradient on it, no transposed structure at hand
        _case("citation_backward_w16", "powerlaw", 170_000, 14, 13_000, 128, "backward", "bucket", 16, 0, "sym"),
        # dense social-like graph, the sampled calls the method is made for
        _case("social_bucket_w64", "powerlaw", 233_000, 490, 21_000, 64, "forward", "bucket", 64, 0, "mean"),
        # the same as an unweighted mean aggregation with a rotation per row (sampled training)
        _case("social_fastrand_w128_unit", "powerlaw", 233_000, 490, 21_000, 64, "forward", "fastrand", 128, 7,
              "unit", "mean"),
        # its exact product
        _case("social_exact", "powerlaw", 233_000, 490, 21_000, 64, "forward", "full", 0, 0, "mean"),
        # second layer of a GCN with 41 classes: rows of X that tile no cache line
        _case("gcn_f41_fastrand_w64", "powerlaw", 233_000, 490, 21_000, 41, "forward", "fastrand", 64, 0, "mean"),
        # training on the dense graph with a seed of its own per iteration
        _case("social_pull_fastrand_w64", "powerlaw", 233_000, 490, 21_000, 64, "pull", "fastrand", 64, 11, "mean"),
        # the largest graph: X far beyond every cache
        _case("copurchase_fastrand_w64", "clustered", 2_450_000, 50, 20_000, 128, "forward", "fastrand", 64, 0, "sym"),
        _case("copurchase_exact", "clustered", 2_450_000, 50, 20_000, 128, "forward", "full", 0, 0, "sym"),
    ]


# ---- sizes, without building the graph ----------------------------------------------------------
def _capped_mean(dmin, cap):
    """Mean of min(d, cap) for density ~ d**-2.1 from dmin on."""
    a = _EXPONENT - 1.0
    if cap <= dmin:
        return cap
    return dmin * a / (a - 1.0) - dmin ** a * cap ** (1.0 - a) / (a - 1.0)


def _dmin(mean, dmax):
    """Lower end of the degree law that gives `mean` (floor and self-loop allowed for)."""
    lo, hi = 0.05, float(dmax)
    for _ in range(80):
        mid = 0.5 * (lo + hi)
        if _capped_mean(mid, dmax) < mean - 0.5:
            lo = mid
        else:
            hi = mid
    return hi


def _entries(case):
    """(stored, kept) entries, to within a few percent."""
    N, mean = case["N"], case["mean"]
    stored = N * mean
    if case["mode"] == "full":
        return stored, stored
    if case["graph"] == "undirected":
        return stored, N * min(mean, case["W"])
    kept = N * min(mean, _capped_mean(_dmin(mean, case["dmax"]), case["W"]) + 0.5)
    return stored, min(stored, kept)


def draw(rng):
    """One more case of the same ranges; it costs no more than the dearest listed one."""
    def log_uniform(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    while True:
        graph = rng.choice(["undirected", "powerlaw", "powerlaw", "powerlaw", "clustered", "clustered"])
        N = int(log_uniform(2_700, 2_450_000))
        mean = round(log_uniform(4.5, 30 if graph == "undirected" else 490), 1)
        dmax = 0 if graph == "undirected" else max(16, int(min(N // 8, mean * log_uniform(40, 900), 21_000)))
        F = int(log_uniform(16, 256))
        if rng.random() < 0.6:
            F = F // 4 * 4
        call = rng.choice(["forward", "forward", "forward", "forward", "forward", "pull", "backward"])
        mode = rng.choice(["full", "bucket", "fastrand", "fastrand"])
        if call != "forward" and mode == "full":
            mode = "fastrand"
        W = 0 if mode == "full" else int(log_uniform(4, 256))
        values, norm = rng.choice([("sym", "none"), ("mean", "none"), ("sym", "none"), ("unit", "mean")])
        seed = rng.choice([0, rng.randrange(1, 1 << 40)])
        case = _case("", graph, N, mean, dmax, F, call, mode, W, seed, values, norm)
        if graph != "undirected" and dmax < 3 * mean:
            continue
        stored, kept = _entries(case)
        # rows that tile no line cost up to two lines more each; the atomic scatter moves its
        # entries some ten times slower than the gathers
        most = 0.6e9 if call == "backward" else 10.0e9 if F % 4 == 0 else 4.0e9
        if stored <= 120.0e6 and kept * F <= most:
            return case


# ---- inputs -----------------------------------------------------------------------------------
def _graph(case, gen, dev):
    N = case["N"]
    loops = torch.arange(N, device=dev)
    if case["graph"] == "undirected":
        m = int(N * (case["mean"] - 1.0) / 2.0)
        a = torch.randint(N, (m,), device=dev, generator=gen)
        b = torch.randint(N, (m,), device=dev, generator=gen)
        key = torch.cat([a * N + b, b * N + a, loops * (N + 1)])
        del a, b
    else:
        dmin = _dmin(case["mean"] - 1.0, case["dmax"])
        u = torch.rand(N, device=dev, generator=gen, dtype=torch.float64)
        deg = (dmin * (1.0 - u).pow(-1.0 / (_EXPONENT - 1.0))).floor().clamp(1, case["dmax"]).long()
        rows = torch.repeat_interleave(loops, deg)
        total = rows.numel()
        cols = torch.randint(N, (total,), device=dev, generator=gen)
        if case["graph"] == "clustered":
            size = -(-N // _BLOCKS)
            start = rows // size * size
            local = start + (torch.rand(total, device=dev, generator=gen) * (N - start).clamp(max=size)).long()
            intra = torch.rand(total, device=dev, generator=gen) < _P_INTRA
            cols = torch.where(intra, local.clamp(max=N - 1), cols)
            del start, local, intra
        key = torch.cat([rows * N + cols, loops * (N + 1)])
        del rows, cols, u, deg
    key = key.sort().values
    first = torch.ones_like(key, dtype=torch.bool)
    torch.ne(key[1:], key[:-1], out=first[1:])
    key = key[first]
    row = key // N
    colidx = (key - row * N).int()
    deg = torch.bincount(row, minlength=N)
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device=dev)
    rowptr[1:] = deg.cumsum(0).int()
    vals = None
    if case["values"] != "unit":
        inv = deg.double().rsqrt() if case["values"] == "sym" else deg.double().reciprocal()
        vals = inv[row]
        if case["values"] == "sym":
            vals *= inv[colidx.long()]
        vals = vals.float()
    return rowptr, colidx, vals


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 1_000_003 + 17)
    rowptr, colidx, vals = _graph(case, gen, dev)
    N, F = case["N"], case["F"]
    s = {"case": case, "rowptr": rowptr, "colidx": colidx, "vals": vals,
         "X": torch.randn((N, F), device=dev, generator=gen),
         "Y": torch.zeros((N, F), device=dev)}
    if case["call"] == "forward":
        s["workspace"] = torch.empty(max(1, es.es_spmm_workspace_bytes(N) // 4), dtype=torch.int32, device=dev)
    elif case["call"] == "pull":
        s["transposed"] = es.es_spmm_transpose_graph(rowptr, colidx, vals)
    return s


def run(state):
    c = state["case"]
    if c["call"] == "forward":
        return es.es_spmm_ws(state["rowptr"], state["colidx"], state["vals"], state["X"], state["Y"], c["W"],
                             c["mode"], c["seed"], c["norm"], None, state["workspace"])
    if c["call"] == "backward":
        return es.es_spmm_backward(state["rowptr"], state["colidx"], state["vals"], state["X"], state["Y"], c["W"],
                                   c["mode"], c["seed"], c["norm"])
    return es.es_spmm_backward_pull(state["rowptr"], state["transposed"], state["X"], state["Y"], c["W"], c["mode"],
                                    c["seed"], c["norm"])


def work(case):
    stored, kept = _entries(case)
    N, F = case["N"], case["F"]
    entry = 4.0 if case["values"] == "unit" else 8.0
    dense = 2.0 * 4.0 * N * F                               # X (dY) once, Y (dX) once
    return {"bytes": 4.0 * (N + 1) + entry * kept + dense, "flops": 2.0 * kept * F}


def tolerance(case):
    # fp32 sums in an unspecified order (es_spmm.h); rows of up to some 20 000 terms
    return {"rel": 1e-5, "max": 1e-3}
