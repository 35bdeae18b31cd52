"""What the library's users have it do, as a list of measurable cases over the range of its configurations.

Every case goes through the public entry points the way a user's program does: the assignment and extraction calls of
``binding``, the trainers of ``trainer`` and the averaging of ``aggregation``.  ``prepare`` makes what such a program
holds beforehand (a graph, features, a trainer with its weights), ``run`` is one pass.  Graphs come in three families:
uniform random, power law (expected degrees ~ (i + i0)^(-1/(gamma-1)), gamma = 2.1, largest sqrt(sum)) and planted
communities; features are N(0,1), weights Glorot.

Paths
  node      one step of a trainer on its part: forward, loss, backward, optimizer; with ``whole`` also the assignment,
            the extraction of the part and the gathers of its rows, as when the partition is redrawn
  evaluate  the forward pass of a model over a whole graph
  link      one step of link prediction with the encoder on the whole local subgraph
  sampled   one step of link prediction on the sampled neighbourhood of a mini-batch
  rounds    several trainers on streams of their own, two local steps each, then the averaging of their weights
  extract   assignment and induced subgraph of one part of a large graph, sizes left on the device
"""
from __future__ import annotations

import math

import torch

from paper_2305_09887_amd import binding as B
from paper_2305_09887_amd import synth_torch as st
from paper_2305_09887_amd.aggregation import ModelAggregation
from paper_2305_09887_amd.trainer import LocalTrainer, SampledLinkTrainer

DEV = "cuda"
GAMMA = 2.1
LR = 1e-3
PART = 0
PART_SEED = 44      # of the assignment: the parts' node counts stay, whatever graph and features the inputs' seed gives


def _node(name, graph, n, degree, parts, dims, dtype="f32", encoder="sage", norm=False, optimizer="sgd", whole=False,
          pitch=0):
    return dict(name=name, path="node", graph=graph, n=n, degree=degree, parts=parts, dims=dims, dtype=dtype,
                encoder=encoder, norm=norm, optimizer=optimizer, whole=whole, pitch=pitch)


def listed():
    return [
        # the tiny configuration: 20,000 nodes, 100,000 edges, K = 4; a step is short kernels and launches
        _node("tiny_node_f32", "uniform", 20_000, 10.0, 4, "64,64,16", whole=True),
        # a mid-size part with widths that are no multiples of anything: features and classes as a dataset has them
        _node("ragged_node_f32", "uniform", 120_011, 13.0, 3, "90,150,41"),
        # the headline configuration: power-law graph of 1 M nodes, K = 8, the whole path each step
        _node("powerlaw_node_f32", "power", 1_000_000, 20.0, 8, "128,256,47", whole=True),
        # the same part with the GCN encoder, layer normalisation + PReLU and Adam
        _node("powerlaw_gcn_norm_f32", "power", 1_000_000, 20.0, 8, "128,256,47", encoder="gcn", norm=True,
              optimizer="adam"),
        # SuperTMA: 2.4 M nodes in 2,400 communities, 60 M edges, K = 16, bf16, feature rows padded to 128
        _node("community_node_bf16", "community", 2_400_000, 50.0, 16, "100,256,256,47", dtype="bf16", whole=True,
              pitch=128),
        # one trainer's share of the 100 M-node graph: 12.5 M local nodes, 20 M local edges, bf16 (the largest)
        _node("share_node_bf16", "power", 12_500_000, 3.26, 1, "128,256,256,47", dtype="bf16"),
        # the averaged model evaluated on the whole 1 M-node graph
        dict(name="evaluate_f32", path="evaluate", graph="power", n=1_000_000, degree=20.0, parts=1, dims="128,256,47",
             dtype="f32", encoder="sage", norm=False),
        # link prediction, encoder on the whole part, 65,536 positives and as many negatives
        dict(name="link_f32", path="link", graph="power", n=1_000_000, degree=20.0, parts=8, dims="128,256,256",
             dtype="f32", encoder="sage", norm=False, batch=65_536),
        # link prediction on sampled neighbourhoods, 1,024 positives, fan-outs 10 and 25
        dict(name="link_sampled_f32", path="sampled", graph="power", n=1_000_000, degree=20.0, parts=8,
             dims="128,256,256", dtype="f32", encoder="sage", batch=1024, fanouts="10,25"),
        # eight trainers on eight streams with averaging (the configuration of 10 M nodes at a fifth of its size)
        dict(name="rounds_f32", path="rounds", graph="power", n=2_000_000, degree=40.0, parts=8, dims="128,256,47",
             dtype="f32", steps=2),
        # the extraction alone on a graph that no cache holds, assignment recomputed inside
        dict(name="extract_fused", path="extract", graph="power", n=20_000_000, degree=20.0, parts=8, fused=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: local parts of 5 k to 4 M nodes, mean local degrees 1 to 40, widths 16 to 256."""
    path = rng.choice(["node", "node", "node", "node", "evaluate", "link", "sampled", "rounds", "extract"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    graph = rng.choice(["uniform", "power", "power"])
    enc = rng.choice(["sage", "sage", "gcn", "mlp"])
    width = lambda lo, hi: rng.choice([8, 8, 4, 1]) * rng.randint(1, 10 ** 6) % (hi - lo) + lo
    hidden = rng.choice([64, 128, 256, 256, width(48, 256)])
    feat, classes = rng.choice([64, 100, 128, width(16, 160)]), rng.randint(5, 64)
    if path in ("node", "evaluate"):
        deep = rng.random() < 0.4
        dims = [feat, hidden] + ([hidden] if deep else []) + [classes]
        norm = rng.random() < 0.35
        parts = rng.choice([2, 3, 4, 8, 16]) if path == "node" else 1
        n_loc = _log(rng, 5_000, 400_000 if dtype == "f32" else 2_000_000)
        whole = path == "node" and n_loc * parts <= 4_000_000 and rng.random() < 0.5
        degree = round(rng.uniform(8.0, 40.0), 2)
        if n_loc * parts * degree > 8e7:
            degree = round(max(3.0, 8e7 / (n_loc * parts)), 2)
        if n_loc * parts > 4_000_000:      # a share: only the local graph is made
            parts = 1
        c = dict(path=path, graph=graph, n=n_loc * parts, degree=degree, parts=parts, dims=",".join(map(str, dims)),
                 dtype=dtype, encoder=enc, norm=norm)
        if path == "node":
            c.update(optimizer=rng.choice(["sgd", "adam"]), whole=whole, pitch=0)
        return c
    if path == "link":
        return dict(path="link", graph=graph, n=8 * _log(rng, 8_000, 150_000), degree=round(rng.uniform(10.0, 40.0), 2),
                    parts=8, dims=f"{feat},{hidden},{hidden}", dtype=dtype, encoder=enc, norm=rng.random() < 0.3,
                    batch=_log(rng, 2_048, 70_000))
    if path == "sampled":
        return dict(path="sampled", graph=graph, n=8 * _log(rng, 20_000, 150_000), degree=round(rng.uniform(10.0, 40.0), 2),
                    parts=8, dims=f"{feat},{hidden},{hidden}", dtype=dtype, encoder=rng.choice(["sage", "gcn"]),
                    batch=_log(rng, 512, 8_192), fanouts=rng.choice(["10,25", "5,10", "15,15"]))
    if path == "rounds":
        return dict(path="rounds", graph=graph, n=_log(rng, 40_000, 1_600_000), degree=round(rng.uniform(10.0, 40.0), 2),
                    parts=rng.choice([4, 8]), dims=f"{feat},{hidden},{classes}", dtype=dtype, steps=2)
    return dict(path="extract", graph=graph, n=_log(rng, 300_000, 12_000_000), degree=round(rng.uniform(5.0, 25.0), 2),
                parts=rng.choice([4, 8, 16]), fused=rng.random() < 0.5)


# ---------------------------------------------------------------------------------------------------- inputs
def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _power_law_ids(g, n, m, i0, expo):
    """m node ids with probabilities ~ (i + i0)^-expo, by inverting the integral of the density."""
    a, b = i0 ** (1.0 - expo), (n + i0) ** (1.0 - expo)
    r = torch.rand(m, generator=g, device=DEV, dtype=torch.float64)
    return ((a + r * (b - a)) ** (1.0 / (1.0 - expo)) - i0).long().clamp_(0, n - 1)


def _graph(case, g):
    """(rowptr int64, colidx int32, community of each node or None)"""
    n, m = case["n"], int(case["n"] * case["degree"] / 2)
    if case["graph"] == "community":
        size = 1000
        rowptr, colidx, block = st.sbm_graph(n // size, size, int(0.9 * m), m - int(0.9 * m),
                                             seed=int(torch.randint(1 << 30, (1,), generator=g, device=DEV)), device=DEV)
        return rowptr, colidx, block
    if case["graph"] == "uniform":
        u, v = (torch.randint(0, n, (m,), generator=g, device=DEV) for _ in range(2))
    else:
        expo, total = 1.0 / (GAMMA - 1.0), 2.0 * m
        lo, hi = 1e-3, float(n)      # the shift at which the largest expected degree is sqrt(total)
        for _ in range(60):
            mid = 0.5 * (lo + hi)
            mass = ((n + mid) ** (1 - expo) - mid ** (1 - expo)) / (1 - expo)
            lo, hi = (mid, hi) if mid ** -expo * total / mass > math.sqrt(total) else (lo, mid)
        shuffled = torch.randperm(n, generator=g, device=DEV)
        u, v = (shuffled[_power_law_ids(g, n, m, hi, expo)] for _ in range(2))
    return st.csr_from_pairs(n, u, v) + (None,)


def _features(g, n, f, dtype, pitch=0):
    x = torch.zeros((n, max(f, pitch)), dtype=dtype, device=DEV)
    for a in range(0, n, 1 << 20):
        b = min(n, a + (1 << 20))
        x[a:b, :f] = torch.randn((b - a, f), generator=g, device=DEV).to(dtype)
    return x[:, :f]


def _glorot(g, a, b):
    return (torch.rand((a, b), generator=g, device=DEV) * 2 - 1) * math.sqrt(6.0 / (a + b))


def _params(g, dims, encoder, norm):
    out = []
    for l, (a, b) in enumerate(zip(dims[:-1], dims[1:])):
        layer = [_glorot(g, a, b) for _ in range(2 if encoder == "sage" else 1)]
        layer.append(torch.randn(b, generator=g, device=DEV) * 0.01)
        if norm and l < len(dims) - 2:
            layer += [torch.ones(b, device=DEV), torch.zeros(b, device=DEV), torch.full((1,), 0.25, device=DEV)]
        out.append(tuple(layer))
    return out


def _decoder(g, dims):
    last = len(dims) - 2
    return [(_glorot(g, a, b),) + ((torch.full((1,), 0.25, device=DEV),) if k < last else ())
            for k, (a, b) in enumerate(zip(dims[:-1], dims[1:]))]


def _dims(case):
    return [int(x) for x in case["dims"].split(",")]


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _kept(case):
    """Share of a graph's entries that one part keeps."""
    K = case["parts"]
    return 1.0 / K ** 2 if case["graph"] != "community" else (0.9 + 0.1 / K) / K


def _held(case, rowptr, colidx, part):
    """Extraction buffers at capacities chosen from the expected sizes; what is not written stays zero."""
    n, K = case["n"], case["parts"]
    cap, cap_nnz = n // K + n // (4 * K) + 1024, int(1.5 * n * case["degree"] * _kept(case)) + 4096
    held = B.tma_induced_subgraph_async(rowptr, colidx, part, PART, cap, cap_nnz)
    for t in held.values():
        t.zero_()
    return dict(held=held, cap=(cap, cap_nnz))


def prepare(case, seed):
    g = _generator(seed)
    rowptr, colidx, block = _graph(case, g)
    n, K, path = case["n"], case["parts"], case["path"]
    if path == "extract":
        part = B.tma_partition(n, K, PART_SEED)
        return dict(case=case, rowptr=rowptr, colidx=colidx, part=part, n_loc=int((part == PART).sum()),
                    **_held(case, rowptr, colidx, part))
    dims, dtype = _dims(case), _dtype(case)
    params = _params(g, dims, case.get("encoder", "sage"), case.get("norm", False))
    clusters = dict(cluster=block, n_clusters=n // 1000) if block is not None else {}
    part = B.tma_partition(n, K, PART_SEED, **clusters)
    if path == "rounds":
        X = _features(g, n, dims[0], dtype)
        y = torch.randint(0, dims[-1], (n,), generator=g, device=DEV, dtype=torch.int32)
        torch.cuda.synchronize()
        trainers = []
        for p in range(K):
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                sub = B.tma_induced_subgraph(rowptr, colidx, part, p)
                Xl, yl = B.tma_gather_rows(sub["l2g"], X), B.tma_gather_rows(sub["l2g"], y)
                trainers.append(LocalTrainer(sub["rowptr"], sub["colidx"], sub["inv_deg"], Xl, yl, dims, params=params,
                                             stream=stream))
            stream.synchronize()
        return dict(case=case, agg=ModelAggregation(trainers))
    sub = B.tma_induced_subgraph(rowptr, colidx, part, PART)
    n_loc, nnz = sub["n_loc"], sub["nnz_loc"]
    graph = (sub["rowptr"], sub["colidx"], sub["inv_deg"])
    s = dict(case=case)
    if path in ("link", "sampled"):
        dec = [dims[-1], dims[-1], 1]
        X = _features(g, n_loc, dims[0], dtype)
        if path == "link":
            tr = LocalTrainer(*graph, X, None, dims, norm_act=case["norm"], encoder=case["encoder"], decoder_dims=dec,
                              batch_size=case["batch"], batch_seed=seed, nnz=nnz)
            tr.load_params(params, _decoder(g, dec))
        else:
            tr = SampledLinkTrainer(sub["rowptr"], sub["colidx"], nnz, X, dims, dec,
                                    [int(f) for f in case["fanouts"].split(",")], case["batch"], batch_seed=seed,
                                    params=params, decoder_params=_decoder(g, dec), encoder=case["encoder"])
        return dict(s, trainer=tr)
    options = dict(params=params, norm_act=case["norm"], encoder=case["encoder"])
    if path == "evaluate":
        return dict(s, trainer=LocalTrainer(*graph, _features(g, n_loc, dims[0], dtype), None, dims, **options))
    pitch = case["pitch"]
    if not case["whole"]:
        X, y = _features(g, n_loc, dims[0], dtype, pitch), torch.randint(0, dims[-1], (n_loc,), generator=g, device=DEV,
                                                                         dtype=torch.int32)
        return dict(s, trainer=LocalTrainer(*graph, X, y, dims, optimizer=case["optimizer"], **options))
    # the whole path: global tables, capacity-sized extraction buffers, a trainer for the local sizes
    Xg = _features(g, n, dims[0], dtype, pitch)
    yg = torch.randint(0, dims[-1], (n,), generator=g, device=DEV, dtype=torch.int32)
    X = torch.zeros((n_loc, max(dims[0], pitch)), dtype=dtype, device=DEV)[:, :dims[0]]
    y = torch.empty(n_loc, dtype=torch.int32, device=DEV)
    return dict(s, trainer=LocalTrainer(*graph, X, y, dims, optimizer=case["optimizer"], **options), rowptr=rowptr,
                colidx=colidx, clusters=clusters, part=part, X=Xg, y=yg, Xl=X, yl=y, n_loc=n_loc, nnz=nnz,
                **_held(case, rowptr, colidx, part))


# ---------------------------------------------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    path = case["path"]
    if path == "extract":
        held = s["held"]
        if case["fused"]:
            B.tma_random_subgraph_async(s["rowptr"], s["colidx"], case["parts"], PART_SEED, PART, *s["cap"], out=held)
        else:
            B.tma_partition(case["n"], case["parts"], PART_SEED, out=s["part"])
            B.tma_induced_subgraph_async(s["rowptr"], s["colidx"], s["part"], PART, *s["cap"], out=held)
        n_loc = s["n_loc"]
        return [held["sizes"], held["g2l"], held["l2g"][:n_loc], held["rowptr"][:n_loc + 1], held["colidx"],
                held["inv_deg"][:n_loc]]
    if path == "rounds":
        agg = s["agg"]
        agg.run_rounds(1, case["steps"], LR)
        return [agg.W_global, [(t.H[t.L], t.loss, t.dW) for t in agg.trainers]]
    tr = s["trainer"]
    if path == "evaluate":
        return tr.forward()
    if path == "node" and case["whole"]:
        n_loc, nnz, held = s["n_loc"], s["nnz"], s["held"]
        B.tma_partition(case["n"], case["parts"], PART_SEED, out=s["part"], **s["clusters"])
        B.tma_induced_subgraph_async(s["rowptr"], s["colidx"], s["part"], PART, *s["cap"], out=held)
        l2g = held["l2g"][:n_loc]
        B.tma_gather_rows(l2g, s["X"], out=s["Xl"])
        B.tma_gather_rows(l2g, s["y"], out=s["yl"])
        rowptr, colidx = held["rowptr"][:n_loc + 1], held["colidx"][:nnz]
        tr.set_graph(rowptr, colidx, held["inv_deg"][:n_loc], nnz=nnz)
        tr.step(LR)
        return [l2g, rowptr, held["colidx"], tr.H[tr.L], tr.loss, tr.dW, tr.W]
    tr.step(LR)
    if path == "node":
        return [tr.H[tr.L], tr.loss, tr.dW, tr.W]
    if path == "link":
        return [tr.H[tr.L], tr.Zd[-1], tr.loss, tr.dW, tr.W]
    return [list(tr.count), tr.Zd[-1], tr.loss, tr.dW, tr.W]


# ---------------------------------------------------------------------------------------------------- expectations
def _encoder_work(n, nnz, dims, size, encoder, train):
    """Bytes and operations of the layers: a layer reads its input and the graph and writes its output; backward reads
    the saved input and the output's gradient and writes the input's.  A SAGE layer is two products, else one."""
    nbytes = flops = 0.0
    for l, (a, b) in enumerate(zip(dims[:-1], dims[1:])):
        product = 2.0 * n * a * b * (2 if encoder == "sage" else 1)
        edges = nnz * 4.0 + n * 8.0 if encoder != "mlp" else 0.0
        nbytes += n * (a + b) * size + edges
        flops += product + (nnz * min(a, b) if encoder != "mlp" else 0)
        if train:
            nbytes += n * (a + b) * size + (n * a * size + edges if l > 0 else 0.0)
            flops += product + (product + nnz * min(a, b) if l > 0 else 0.0)
    return nbytes, flops


def work(case):
    n, K, path = case["n"], case["parts"], case["path"]
    entries = float(n) * case["degree"]
    extract = n * 4.0 + n / K * (12.0 + 16.0) + entries / K * 4.0 + entries / K ** 2 * 4.0
    if path == "extract":
        return {"bytes": extract, "flops": 0.0}
    dims, size = _dims(case), 2 if case["dtype"] == "bf16" else 4
    encoder = case.get("encoder", "sage")
    n_loc, nnz = n / K, entries * _kept(case)
    if path == "evaluate":
        b, f = _encoder_work(n, entries, dims, size, encoder, False)
        return {"bytes": b, "flops": f}
    if path == "rounds":
        b, f = _encoder_work(n, entries / K, dims, size, encoder, True)
        return {"bytes": b * case["steps"], "flops": f * case["steps"]}
    if path == "node":
        b, f = _encoder_work(n_loc, nnz, dims, size, encoder, True)
        if case["whole"]:
            b += extract + 2 * n_loc * (dims[0] * size + 4)
        return {"bytes": b, "flops": f}
    batch, d = case["batch"], dims[-1]
    decoder_b = batch * (3 + 2 * 5) * d * size * 2.0
    decoder_f = 2.0 * 2 * batch * (d * d + d) * 3
    if path == "link":
        b, f = _encoder_work(n_loc, nnz, dims, size, encoder, True)
        return {"bytes": b + decoder_b, "flops": f + decoder_f}
    b, f, rows = 0.0, 0.0, min(n_loc, 2.7 * batch)
    for l in range(len(dims) - 2, -1, -1):       # a level's rows read their sampled neighbours' rows
        mean_kept = min(int(case["fanouts"].split(",")[l]), case["degree"] / K * 2)
        src = min(n_loc, rows * (1 + mean_kept))
        b += (src * dims[l] + rows * dims[l + 1]) * size * (3 if l > 0 else 2)
        f += 2.0 * rows * dims[l] * dims[l + 1] * (2 if encoder == "sage" else 1) * (3 if l > 0 else 2)
        rows = src
    return {"bytes": b + decoder_b, "flops": f + decoder_f}


class _Aggregate(torch.autograd.Function):
    """s_out (.) A (s_in (.) H) over a symmetric CSR, entries taken in pieces."""

    @staticmethod
    def forward(ctx, H, rows, cols, s_in, s_out):
        ctx.graph = rows, cols, s_in, s_out
        return _Aggregate.sum(H, rows, cols, s_in, s_out)

    @staticmethod
    def sum(H, rows, cols, s_in, s_out):
        H = H if s_in is None else H * s_in[:, None]
        out, piece = torch.zeros_like(H), max(1, (1 << 28) // H.shape[1])
        for a in range(0, rows.numel(), piece):
            out.index_add_(0, rows[a:a + piece], H[cols[a:a + piece]])
        return out if s_out is None else out * s_out[:, None]

    @staticmethod
    def backward(ctx, d):
        rows, cols, s_in, s_out = ctx.graph
        return _Aggregate.sum(d, cols, rows, s_out, s_in), None, None, None, None


def _exact_step(tr, case, W, labels=None, batch=None, backward=True):
    """One step of ``tr`` in 64 bits from the flat weights W: [output of the encoder, decoder's logits, loss, gradient]."""
    W = W.double().requires_grad_(backward)
    layers, dec = tr._views(W)
    n, f64 = tr.n, torch.float64
    deg = (tr.rowptr[1:] - tr.rowptr[:-1]).long()
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    cols = tr.colidx[:rows.numel()].long()
    H = tr.H[0].double()
    for l, layer in enumerate(layers):
        if tr.encoder == "sage":
            inv = torch.where(deg > 0, 1.0 / deg.clamp(min=1).to(f64), 0.0)
            Z = H @ layer[0] + _Aggregate.apply(H, rows, cols, None, inv) @ layer[1] + layer[2]
        elif tr.encoder == "gcn":
            s = (deg + 1).to(f64) ** -0.5
            Y = H @ layer[0]
            Z = _Aggregate.apply(Y, rows, cols, s, s) + Y * (s * s)[:, None] + layer[1]
        else:
            Z = H @ layer[0] + layer[1]
        if l == len(layers) - 1:
            H = Z
        elif tr.norm_act:
            gamma, beta, slope = layer[-3:]
            H = torch.nn.functional.prelu(torch.nn.functional.layer_norm(Z, Z.shape[1:], gamma, beta, 1e-5), slope)
        else:
            H = Z.relu()
    logits = loss = None
    if batch is not None:
        u, v, w = (b.long() for b in batch)
        E = torch.cat([H[u] * H[v], H[u] * H[w]])
        for k, layer in enumerate(dec):
            E = E @ layer[0]
            if k < len(dec) - 1:
                E = torch.nn.functional.prelu(E, layer[1])
        logits = E
        truth = torch.cat([torch.ones(u.numel()), torch.zeros(u.numel())]).to(DEV, f64)
        loss = torch.nn.functional.binary_cross_entropy_with_logits(E[:, 0], truth)
    elif backward:
        loss = torch.nn.functional.cross_entropy(H, labels.long())
    grad = torch.autograd.grad(loss, W)[0] if backward else None
    return [None if t is None else t.detach() for t in (H, logits, loss, grad)]


def _stepped(case, tr, g):
    """The weights after one optimizer step with gradient g from the trainer's initial ones."""
    if tr.optimizer == "adam":      # first step: the bias-corrected moments are g and g * g
        return tr.W.double() - LR * g / (g.abs() + 1e-8)
    return tr.W.double() - LR * g


def exact(case, seed):
    """What run() returns, in 64 bits and plain torch; None for whole numbers, and where it would take too long or the
    inputs of the arithmetic are themselves drawn inside the call (the sampled neighbourhoods)."""
    path = case["path"]
    if path in ("extract", "sampled") or case["n"] / case["parts"] * max(_dims(case)) > 1.2e9:
        return None
    s = prepare(case, seed)
    if path == "rounds":
        if case["n"] * max(_dims(case)) > 6e8:
            return None
        trainers, out, mean = s["agg"].trainers, [], 0.0
        torch.cuda.synchronize()
        for tr in trainers:
            W = tr.W.double()
            for _ in range(case["steps"]):
                H, _, loss, g = _exact_step(tr, case, W, tr.labels)
                W = W - LR * g
            out.append((H, loss.reshape(1), g))
            mean = mean + W / len(trainers)
        return [mean, out]
    tr = s["trainer"]
    if path == "evaluate":
        return _exact_step(tr, case, tr.W, backward=False)[0]
    if path == "link":
        tr._draw_batch()
        H, Z, loss, g = _exact_step(tr, case, tr.W, batch=tr.batch)
        return [H, Z, loss.reshape(1), g, _stepped(case, tr, g)]
    if case["whole"]:       # the rows that the gathers bring
        l2g = torch.nonzero(s["part"] == PART)[:, 0]
        tr.H[0].copy_(s["X"][l2g])
        tr.labels.copy_(s["y"][l2g])
    H, _, loss, g = _exact_step(tr, case, tr.W, tr.labels)
    out = [H, loss.reshape(1), g, _stepped(case, tr, g)]
    return [None, None, None] + out if case["whole"] else out


def tolerance(case):
    if case["path"] == "extract":
        return "exact"
    # About four times the largest relative error seen against exact().  Logits 4e-7 in fp32; gradients 1e-7 where no
    # decision falls differently, but a ReLU or PReLU input within rounding of zero opens or closes a row's share of
    # them: up to 2.9e-5 (the widest layers), 1.5e-5 in the link decoder.  bf16 storage: logits 4.4e-3, gradients 4.0e-3.
    if case["dtype"] == "bf16":
        return {"rel": 1.6e-2}
    return {"rel": 1e-5 if case["path"] == "evaluate" else 1.2e-4}
