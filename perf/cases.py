"""The work that a user of this library has it do, as cases that can be timed.

A case is one pass of one kind of program through the public entry points:
  epoch      forward + backward of a full-graph GCN (`GcnEpoch`), in each order it offers
  gat        forward + backward of a decoupled GAT (`GatEpoch`)
  worker     one tensor-parallel worker's share of a layer-wise epoch (`TensorParallelEpoch.run_worker`)
  aggregate  one forward and one backward aggregation of a column slice, on their own
  stream     one forward and one backward aggregation whose topology is copied from pinned host memory
  transform  the dense transform and its two gradients, on their own
  build      the graph build from a host edge list, and the built arrays
Sizes are those of the workloads in `ntp_inputs/configs.py`, whole or divided, and the ranges around them.
"""
import math

import numpy as np
import torch

import paper_2412_20379_amd as ntp
from paper_2412_20379_amd.gat import GatEpoch
from paper_2412_20379_amd.gcn import GcnEpoch
from paper_2412_20379_amd.tp import TensorParallelEpoch, line_padded_ld

DEV = "cuda:0"
RMAT = (0.57, 0.19, 0.19)        # quadrant probabilities a, b, c of the R-MAT workloads
MOST_ENTRIES = 63_000_000        # stored entries of the largest graph
SMALLEST_N, LARGEST_N = 1_000, 1_300_000


# ---- the cases ------------------------------------------------------------------------------------
def listed():
    return [
        # one slice of the citation-size graph: nothing but launches and latency
        dict(name="aggregate-tiny", kind="aggregate", graph="er", n=2708, m=5278, directed=False, f=16, dtype="f32"),
        # config 1 whole: a citation-size graph, wide sparse features, an epoch of small kernels
        dict(name="epoch-cfg1", kind="epoch", graph="er", n=2708, m=5278, dims="1433,16,7", order="layerwise"),
        # config 2 whole: full-width layer-wise epoch, low-degree power-law graph
        dict(name="epoch-cfg2", kind="epoch", graph="rmat", n=169343, m=1166243, dims="128,256,256,40", order="layerwise"),
        # config 4 at a quarter of its vertices (density kept), each layer on its narrower side
        dict(name="epoch-dense-auto", kind="epoch", graph="zipf", n=58241, m=3581250, dims="602,128,41", order="auto"),
        # decoupled order on an odd size, 47 classes as config 3
        dict(name="epoch-decoupled", kind="epoch", graph="rmat", n=40961, m=1030011, dims="100,256,47", order="decoupled"),
        # config 2's graph and widths with attention
        dict(name="gat-cfg2", kind="gat", graph="rmat", n=169343, m=1166243, dims="128,256,256,40", perm=True),
        # one of eight workers on config 3 at half its size
        dict(name="worker-cfg3", kind="worker", graph="rmat", n=1224514, m=30930000, dims="100,256,256,47", workers=8),
        # config 4 at half its vertices, its 76-column slice stored as bf16
        dict(name="aggregate-bf16", kind="aggregate", graph="zipf", n=116482, m=14325000, directed=False, f=76, dtype="bf16"),
        # a directed graph (two stored forms) and the ragged 13-column slice of config 3
        dict(name="aggregate-directed", kind="aggregate", graph="rmat", n=1224514, m=25000003, directed=True, f=13, dtype="f32"),
        # cold streaming of an eighth of config 3
        dict(name="stream-cfg3", kind="stream", graph="rmat", n=306128, m=7732500, f=32, dtype="f32", chunk=4000000),
        # the 256 x 256 hidden layer on one worker's rows of config 3
        dict(name="transform-256", kind="transform", n=306129, k=256, m=256, relu=True, dtype="f32"),
        # config 2's graph built from its edge list
        dict(name="build-cfg2", kind="build", graph="rmat", n=169343, m=1166243, directed=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, most_entries, kinds=("er", "rmat", "zipf"), directed=False):
    n = _log_int(rng, SMALLEST_N, LARGEST_N)
    degree = math.exp(rng.uniform(math.log(4), math.log(200)))         # stored entries per vertex, about
    forms = 1 if directed else 2
    m = int(min(n * degree / 2, (most_entries - n) / forms, n * n * 0.005)) | 1
    return dict(graph=rng.choice(kinds), n=n, m=max(m, n // 2))


def draw(rng):
    kind = rng.choice(["epoch", "epoch", "epoch", "gat", "worker", "aggregate", "aggregate", "stream", "transform", "transform", "build"])
    if kind == "transform":
        k, m = rng.choice([16, 41, 64, 100, 128, 200, 256, 256, 602]), rng.choice([16, 41, 47, 64, 128, 172, 256, 256])
        return dict(kind=kind, n=_log_int(rng, SMALLEST_N, 306129), k=k, m=m, relu=rng.random() < 0.5, dtype=rng.choice(["f32", "f32", "bf16"]))
    if kind == "aggregate":
        directed = rng.random() < 0.3
        f = _log_int(rng, 4, 256)
        g = _draw_graph(rng, min(MOST_ENTRIES // 2, int(31_000_000 * 76 / max(f, 32))), directed=directed)
        return dict(kind=kind, **g, directed=directed, f=f, dtype=rng.choice(["f32", "f32", "bf16"]))
    if kind == "stream":
        g = _draw_graph(rng, 15_000_000, ("er", "rmat"))
        return dict(kind=kind, **g, f=rng.choice([13, 16, 32, 76, 100]), dtype="f32", chunk=max(4096, (2 * g["m"] + g["n"]) // rng.randint(3, 12)))
    if kind == "build":
        return dict(kind=kind, **_draw_graph(rng, 8_000_000, ("er", "rmat")), directed=rng.random() < 0.3)
    if kind == "worker":
        dims = [rng.choice([100, 128, 602]), rng.choice([128, 256]), rng.choice([128, 256]), rng.choice([40, 47, 172])]
        return dict(kind=kind, **_draw_graph(rng, MOST_ENTRIES), dims=",".join(map(str, dims)), workers=8)
    hidden = [rng.choice([16, 64, 128, 256])] * rng.choice([1, 1, 2])
    dims = ",".join(map(str, [rng.choice([64, 100, 128, 300, 602])] + hidden + [rng.choice([7, 40, 41, 47])]))
    g = _draw_graph(rng, 3_000_000)
    g["n"] = min(g["n"], 250_000)
    g["m"] = min(g["m"], int(g["n"] * g["n"] * 0.005) | 1)
    if kind == "gat":
        return dict(kind=kind, **g, dims=dims, perm=rng.random() < 0.5)
    return dict(kind=kind, **g, dims=dims, order=rng.choice(["layerwise", "auto", "decoupled", "reordered"]))


# ---- inputs ---------------------------------------------------------------------------------------
def _edges(case, gen):
    """exactly case["m"] distinct edges without loops, as host int32 arrays (undirected: each edge once)"""
    n, m, graph = case["n"], case["m"], case["graph"]
    directed = case.get("directed", False)
    scale = max(1, math.ceil(math.log2(n)))
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    cdf = None
    if graph == "zipf":            # end points in proportion to a capped power-law degree sequence
        r = torch.arange(1, n + 1, device=DEV, dtype=torch.float64) ** -1.1
        deg = (r * (2.0 * m / float(r.sum()))).clamp(1, max(1, n // 8))
        for _ in range(30):
            deg = (deg * (2.0 * m / float(deg.sum()))).clamp(1, max(1, n // 8))
        cdf = torch.cumsum(deg, 0)
        cdf /= cdf[-1].clone()
    while keys.numel() < m:
        k = int((m - keys.numel()) * 1.4) + 1024
        if graph == "er":
            u, v = torch.randint(n, (2, k), generator=gen, device=DEV)
        elif graph == "zipf":
            u, v = torch.searchsorted(cdf, torch.rand(2, k, generator=gen, device=DEV, dtype=torch.float64)).clamp(max=n - 1)
        else:
            u = torch.zeros(k, dtype=torch.int64, device=DEV)
            v = torch.zeros(k, dtype=torch.int64, device=DEV)
            a, b, c = RMAT
            for _ in range(scale):
                r = torch.rand(k, generator=gen, device=DEV)
                u = (u << 1) | (r >= a + b)
                v = (v << 1) | (((r >= a) & (r < a + b)) | (r >= a + b + c))
        ok = (u != v) & (u < n) & (v < n)
        u, v = u[ok], v[ok]
        if not directed:
            u, v = torch.minimum(u, v), torch.maximum(u, v)
        keys = torch.unique(torch.cat([keys, u * n + v]))
    keys = keys[torch.randperm(keys.numel(), generator=gen, device=DEV)[:m]]
    relabel = torch.randperm(n, generator=gen, device=DEV).to(torch.int32)
    return relabel[keys // n].cpu().numpy(), relabel[keys % n].cpu().numpy()


def _graph(case, gen, more_flags=0, **kw):
    src, dst = _edges(case, gen)
    flags = ntp.NTP_DIRECTED_GCN_FLAGS if case.get("directed") else ntp.NTP_GCN_FLAGS
    return ntp.ntp_graph_build(case["n"], src, dst, flags=flags | more_flags, **kw)


def _entries(case):
    """stored entries of one form: one per direction of an edge and one self loop per vertex"""
    return (1 if case.get("directed") else 2) * case["m"] + case["n"]


def _dims(case):
    return tuple(int(x) for x in case["dims"].split(","))


def _weights(dims, gen):
    def glorot(a, b):
        return (torch.rand(a, b, generator=gen, device=DEV) * 2 - 1) * math.sqrt(6.0 / (a + b))
    return [glorot(a, b) for a, b in zip(dims[:-1], dims[1:])]


def _normal(shape, gen, dtype=torch.float32):
    return torch.randn(shape, generator=gen, device=DEV).to(dtype)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind, n = case["kind"], case["n"]
    s = dict(case=case, kind=kind)
    if kind == "transform":
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        k, m = case["k"], case["m"]
        s.update(A=_normal((n, k), gen, dt), W=_weights((k, m), gen)[0].to(dt), dH=_normal((n, m), gen, dt),
                 H=torch.empty(n, m, dtype=dt, device=DEV), dA=torch.empty(n, k, dtype=dt, device=DEV), dW=torch.empty(k, m, device=DEV))
        s["ws_bytes"] = ntp.ntp_nn_bwd_workspace_bytes(n, k, m)
        s["ws"] = torch.empty(max(4, s["ws_bytes"]), dtype=torch.uint8, device=DEV)
    elif kind == "build":
        s["src"], s["dst"] = _edges(case, gen)
    elif kind in ("aggregate", "stream"):
        f, bf16 = case["f"], case["dtype"] == "bf16"
        dt = torch.bfloat16 if bf16 else torch.float32
        ld = s["ld"] = line_padded_ld(f, 2 if bf16 else 4)
        if kind == "stream":
            s["g"] = _graph(case, gen, ntp.NTP_FORCE_STREAM, chunk_edges=case["chunk"])
            s["copy_stream"] = torch.cuda.Stream()
        else:
            s["g"] = _graph(case, gen)
        s.update(X=_normal((n, ld), gen, dt), G=_normal((n, ld), gen, dt),
                 Y=torch.empty(n, ld, dtype=dt, device=DEV), Gin=torch.empty(n, ld, dtype=dt, device=DEV))
    else:
        dims = _dims(case)
        g = s["g"] = _graph(case, gen, ntp.NTP_EDGE_PERM if case.get("perm") else 0)
        if dims[0] == 1433:        # the citation-size workload has sparse 0/1 features
            s["X"] = (torch.rand(n, dims[0], generator=gen, device=DEV) < 0.0127).float()
        else:
            s["X"] = _normal((n, dims[0]), gen)
        s["W"] = _weights(dims, gen)
        s["labels"] = torch.randint(dims[-1], (n,), generator=gen, device=DEV)
        if kind == "epoch":
            s["model"] = GcnEpoch(g, n, dims, order=case["order"])
        elif kind == "gat":
            s["a"] = _normal((2, dims[-1]), gen) * 0.7
            s["model"] = GatEpoch(g, n, _entries(case), dims)
        else:                      # a worker's share starts from what the other workers' exchange left in its buffers
            s["model"] = TensorParallelEpoch(g, n, dims, workers=case["workers"])
            s["model"].run(s["X"], s["W"], s["labels"])
    return s


# ---- one pass -------------------------------------------------------------------------------------
def run(s):
    case, kind = s["case"], s["kind"]
    st = torch.cuda.current_stream()
    if kind == "epoch":
        s["model"].run(s["X"], s["W"], s["labels"])
        return [s["model"].loss, s["model"].logits] + list(s["model"].dW)
    if kind == "gat":
        m = s["model"]
        m.run(s["X"], s["W"], s["a"][0], s["a"][1], s["labels"])
        return [m.loss, m.logits, m.alpha_in, m.da_src, m.da_dst] + list(m.dW)
    if kind == "worker":
        m = s["model"]
        m.run_worker(0)
        r0, r1 = m.rows[0]
        out = []
        for l in range(m.L):
            width = m.cols[l][0][1] - m.cols[l][0][0]
            out += [m.T[l][0][:, :width], m.H[l][r0:r1], m.dW_part[l][0]]
            if l > 0:
                out += [m.dA[l][r0:r1], m.dT[l][0][:, :width]]
        return out
    code = ntp.NTP_BF16 if case.get("dtype") == "bf16" else ntp.NTP_F32
    if kind == "aggregate":
        f, ld = case["f"], s["ld"]
        ntp.ntp_aggregate_fwd(s["g"], s["X"], s["Y"], f, ld, ld, code, st)
        ntp.ntp_aggregate_bwd(s["g"], s["G"], s["Gin"], f, ld, ld, code, st)
        return [s["Y"][:, :f], s["Gin"][:, :f]]
    if kind == "stream":
        f, ld = case["f"], s["ld"]
        ntp.ntp_chunked_aggregate(s["g"], ntp.NTP_FWD, s["X"], s["Y"], f, ld, ld, code, st, s["copy_stream"])
        ntp.ntp_chunked_aggregate(s["g"], ntp.NTP_BWD, s["G"], s["Gin"], f, ld, ld, code, st, s["copy_stream"])
        return [s["Y"][:, :f], s["Gin"][:, :f]]
    if kind == "transform":
        n, k, m = case["n"], case["k"], case["m"]
        act = ntp.NTP_ACT_RELU if case["relu"] else ntp.NTP_ACT_NONE
        ntp.ntp_nn_fwd(s["A"], s["W"], s["H"], n, k, m, act, code, st)
        ntp.ntp_nn_bwd(s["A"], s["W"], s["H"], s["dH"], s["dA"], s["dW"], n, k, m, act, code, s["ws"], s["ws_bytes"], st)
        return [s["H"], s["dA"], s["dW"]]
    flags = ntp.NTP_DIRECTED_GCN_FLAGS if case["directed"] else ntp.NTP_GCN_FLAGS
    g = ntp.ntp_graph_build(case["n"], s["src"], s["dst"], flags=flags)
    out = list(ntp.ntp_graph_export(g, ntp.NTP_CSR))
    if case["directed"]:
        out += list(ntp.ntp_graph_export(g, ntp.NTP_CSC))
    ntp.ntp_graph_free(g)
    return [np.asarray(x) for x in out]


# ---- what a pass cannot do without ----------------------------------------------------------------
def work(case):
    kind, n = case["kind"], case["n"]
    size = 2 if case.get("dtype") == "bf16" else 4
    if kind == "transform":
        k, m = case["k"], case["m"]
        return dict(bytes=size * (2 * n * k + 2 * n * m + k * m) + 4 * k * m, flops=6 * n * k * m)
    nnz = _entries(case)
    topology = 8 * nnz + 8 * (n + 1)
    forms = 2 if case.get("directed") else 1
    if kind == "build":
        return dict(bytes=8 * case["m"] + forms * topology, flops=0)
    if kind in ("aggregate", "stream"):
        f = case["f"]
        return dict(bytes=(1 if kind == "stream" else forms) * topology + 4 * n * f * size, flops=4 * nnz * f)
    dims = _dims(case)
    layers = list(zip(dims[:-1], dims[1:]))
    if kind == "worker":
        w = case["workers"]
        slices = [-(-d // w) for d in dims[:-1]]
        rows = -(-n // w)
        dense = sum((4 if l == 0 else 6) * rows * a * b for l, (a, b) in enumerate(layers))
        sparse = sum((2 if l == 0 else 4) * nnz * f for l, f in enumerate(slices))
        moved = sum((2 if l == 0 else 5) * n * f for l, f in enumerate(slices)) + sum((1 if l == 0 else 2) * rows * a + 2 * rows * b for l, (a, b) in enumerate(layers))
        return dict(bytes=topology + 4 * moved, flops=dense + sparse)
    dense = sum((4 if l == 0 else 6) * n * a * b for l, (a, b) in enumerate(layers))
    weights = sum(a * b for a, b in layers)
    moved = n * dims[0] + n * dims[-1] + 2 * weights + 2 * n
    if kind == "gat":
        return dict(bytes=topology + 4 * (moved + nnz), flops=dense + 2 * 2 * nnz * dims[-1] * 3)
    if case["order"] == "decoupled":
        sparse = 4 * len(layers) * nnz * dims[-1]
    else:
        sparse = 0
        for l, (a, b) in enumerate(layers):
            first = b < a and (case["order"] == "auto" or (case["order"] == "reordered" and l == len(layers) - 1))
            sparse += 4 * nnz * b if first else (2 if l == 0 else 4) * nnz * a
    return dict(bytes=topology + 4 * moved, flops=dense + sparse)


def tolerance(case):
    if case["kind"] == "build":
        return "exact"
    if case.get("dtype") == "bf16":
        return {"rel": 1e-2}
    # 32-bit sums.  Where a pass takes the sign of one (ReLU, LeakyReLU), a value that is zero to
    # rounding (about one in 10^7) may fall on either side, and one term of a gradient is there or not:
    # sqrt(2e-7) of a gradient's norm, and visible in the row of dA that the term belongs to
    if case["kind"] in ("epoch", "gat"):
        return {"rel": 1e-3}
    if case["kind"] == "transform" and case["relu"]:
        return {"rel": 1e-3, "max": 0.5}
    return {"rel": 1e-5}
