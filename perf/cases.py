"""Performance cases of the partition-wise full-graph GNN library.

A case is one pass that a user's program makes through ``paper_2605_11517_amd.Session``: an epoch
(forward, loss, backward), a training step (dropout, epoch, optimizer), or a forward pass stepped
layer by layer and partition by partition, as an evaluation does it.  Graphs are seeded R-MAT graphs
with the quadrant probabilities of the repository's generator, drawn on the GPU so that inputs are
quick to make.  Widths, average degrees, partition counts, partitioners and switches are those of
the repository's workloads, tests and benchmark (with odd ones among them), vertex counts run from a
few thousand to three million.

Fields of a case
    do        "epoch" | "train" (dropout + epoch + Adam step) | "forward" (stepped by hand)
    model     "gcn" | "sage" | "gat";  dims: layer widths, "x" between them;  dtype: "f32" | "bf16"
    heads     attention heads per layer, "x" between them ("" = one everywhere)
    n, edges  vertices and drawn edges (distinct; mirrored when symmetric)
    k, part   partitions and the rule that assigns vertices to them
    tuned     True: the switches the benchmark sets (layer order by rows moved, gather fused into the
              aggregation, output layer's backward over train vertices, forward results kept);
              False: the library's defaults (the paper's order and steps, gather through staging)
    budget    0: everything resident; else share of the activations and gradients that the streaming
              schedule may keep in device memory
    train_frac  share of the vertices in the train mask
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_11517_amd import Session

DEVICE = "cuda:0"
RMAT_ABC = (0.57, 0.19, 0.19)

BASE = dict(do="epoch", dtype="f32", heads="", tuned=True, budget=0.0, train_frac=0.1)


def listed():
    def case(name, **kw):
        return dict(BASE, name=name, **kw)

    return [
        # the parity fixture: the smallest graph anybody trains on, where launches and latency count
        case("tiny_gcn", model="gcn", dims="64x64x16", n=10_000, edges=98_000, symmetric=True, k=4,
             part="random", train_frac=0.5),
        # a small graph with the library's default switches: every step of the paper's loop, through staging
        case("small_sage_default", model="sage", dims="100x256x256x47", n=3_000, edges=35_000, symmetric=True,
             k=5, part="lp", tuned=False),
        # odd sizes throughout: widths that are no multiple of a vector, a row count that fills no tile
        case("ragged_gcn", model="gcn", dims="61x77x33x19", n=50_021, edges=610_007, symmetric=True, k=7,
             part="lp", train_frac=0.3),
        # training on a graph of the size of the common citation and co-purchase sets
        case("train_sage", do="train", model="sage", dims="100x256x256x47", n=40_009, edges=500_000,
             symmetric=True, k=8, part="switching", train_frac=0.3),
        # the products-shaped workload (GraphSAGE, average degree 55) as the benchmark runs it
        case("products_sage", model="sage", dims="100x256x256x47", n=1_200_000, edges=32_800_000, symmetric=True,
             k=16, part="switching_device"),
        # the same shape in the paper's order: gather through staging, regather, recompute
        case("products_sage_default", model="sage", dims="100x256x256x47", n=150_000, edges=4_100_000,
             symmetric=True, k=16, part="lp", tuned=False),
        # evaluation: the forward pass alone, stepped through the per-partition entry points
        case("forward_sage", do="forward", model="sage", dims="128x256x256x64", n=250_000, edges=2_500_000,
             symmetric=True, k=16, part="lp"),
        # the papers-shaped workload (directed GCN, average degree 16, many partitions): the largest
        case("papers_gcn", model="gcn", dims="128x128x128x172", n=3_000_000, edges=49_000_000, symmetric=False,
             k=64, part="switching_device"),
        # wide hidden layers in bfloat16 storage
        case("dense_bf16", model="gcn", dims="512x1024x1024x64", n=240_000, edges=3_150_000, symmetric=True,
             k=16, part="lp", dtype="bf16"),
        # a bfloat16 training step at an ordinary size with widths that are odd multiples of eight
        case("train_bf16", do="train", model="gcn", dims="72x136x136x40", n=100_003, edges=1_000_000,
             symmetric=True, k=6, part="lp", dtype="bf16", train_frac=0.3),
        # graph attention, eight heads in the hidden layers
        case("attention", model="gat", heads="8x8x1", dims="100x256x256x47", n=150_000, edges=3_000_000,
             symmetric=True, k=16, part="switching_device"),
        # arrays in pinned host memory, partition blocks streamed through device memory
        case("streaming_sage", model="sage", dims="128x256x256x64", n=60_000, edges=600_000, symmetric=True,
             k=32, part="switching_device", budget=0.56),
    ]


# (model, dims, dtype, heads, symmetric, largest average degree): the repository's workloads and test shapes
SHAPES = (
    ("gcn", "64x64x16", "f32", "", True, 24),
    ("gcn", "7x9x5", "f32", "", True, 16),
    ("gcn", "36x40x8", "f32", "", True, 60),
    ("gcn", "128x128x128x172", "f32", "", False, 20),
    ("sage", "100x256x256x47", "f32", "", True, 56),
    ("sage", "100x256x256x47", "f32", "", True, 56),
    ("sage", "128x256x256x64", "f32", "", True, 24),
    ("gcn", "512x1024x1024x64", "bf16", "", True, 28),
    ("gcn", "64x128x64x16", "bf16", "", True, 24),
    ("sage", "72x136x8", "bf16", "", True, 24),
    ("gat", "100x256x256x47", "f32", "", True, 56),
    ("gat", "100x256x256x47", "f32", "8x8x1", True, 56),
)


def draw(rng):
    """One more case of the ranges above, no dearer than the dearest listed one."""
    model, dims, dtype, heads, symmetric, top = rng.choice(SHAPES)
    if model != "gat" and dtype == "f32" and rng.random() < 0.3:
        # generic widths, odd ones among them
        dims = "x".join(str(rng.randint(5, 300)) for _ in range(rng.choice((3, 4))))
    n = int(math.exp(rng.uniform(math.log(2_000), math.log(3_000_000))))
    degree = math.exp(rng.uniform(math.log(6), math.log(top)))
    c = dict(BASE, model=model, dims=dims, dtype=dtype, heads=heads, symmetric=symmetric, n=n,
             k=int(round(math.exp(rng.uniform(0.0, math.log(64))))), part=rng.choice(("random", "lp", "switching_device")),
             tuned=rng.random() < 0.75, train_frac=rng.choice((0.1, 0.1, 0.3, 0.5)),
             do=rng.choice(("epoch", "epoch", "epoch", "train", "forward")))
    if model != "gat" and c["do"] == "epoch" and n < 150_000 and rng.random() < 0.15:
        c.update(budget=rng.choice((0.4, 0.56, 0.8)), k=max(16, c["k"]))
    dearest = max(_cost(x) for x in listed())
    while True:
        c["edges"] = max(64, int(c["n"] * degree / (2 if symmetric else 1)))
        if _cost(c) <= dearest:
            return c
        c["n"] = int(c["n"] * 0.8)


def _dims(case):
    return [int(d) for d in case["dims"].split("x")]


def _entries(case):
    """Entries of the aggregation operator: GCN and attention have one self-loop per vertex."""
    return case["edges"] * (2 if case["symmetric"] else 1) + (case["n"] if case["model"] != "sage" else 0)


def work(case):
    """Bytes: features, operator (one column index per entry, one row offset per vertex), labels and
    mask read once; every activation, activation gradient and weight gradient that the pass returns
    written once.  Flops: the contractions (forward, weight gradient, input gradient of every layer
    but the first) and two per operator entry and column for each aggregation, taken at the narrower
    side of the layer."""
    d, n, nnz = _dims(case), case["n"], _entries(case)
    es = 2 if case["dtype"] == "bf16" else 4
    L = len(d) - 1
    sides = 2 if case["model"] == "sage" else 1
    backward = case["do"] != "forward"
    moved = n * d[0] * es + 4 * nnz + 8 * n
    flops = 0
    for l in range(1, L + 1):
        moved += n * d[l] * (4 if l == L else es)
        params = sides * d[l - 1] * d[l]
        moved += params * es
        flops += 2 * n * params
        narrow = d[l] if case["model"] == "gat" else min(d[l - 1], d[l])
        # attention: a row of scores, the edge-wise products of the backward pass beside the sums
        passes = 1
        if backward:
            moved += n * d[l] * 4 + params * 4
            if case["do"] == "train":
                moved += params * 4 * 5          # moments read and written, weights written
            flops += 2 * n * params * (2 if l >= 2 else 1)
            passes += 1 if l >= 2 else 0
            if case["model"] == "gat":
                passes = 3
        flops += 2 * nnz * narrow * passes
    if backward:
        moved += 5 * n
    return {"bytes": moved, "flops": flops}


def _cost(case):
    """Seconds a pass takes, roughly: rows fetched once per operator entry and pass at 6 TB/s, contractions
    at a good share of the matrix rate, the link for the streaming schedule."""
    d, n, nnz = _dims(case), case["n"], _entries(case)
    es = 2 if case["dtype"] == "bf16" else 4
    rows = sum(nnz * min(d[l], d[l - 1]) * es * (1 if l == 1 else 2) for l in range(1, len(d)))
    t = rows * (1 if case["tuned"] else 2.5) * (3 if case["model"] == "gat" else 1) / 6e12
    t += work(case)["flops"] / (500e12 if es == 2 else 80e12) + 6 * n * sum(d) * 4 / 5e12
    if case["budget"]:
        t += 12 * n * sum(d) * 4 / 40e9
    return t


def tolerance(case):
    """Largest relative error of another correct implementation at the same precision, from runs of
    the listed cases in the other layer order and with other partitions, which add the same terms in
    other orders.  fp32 sums alone differ by 4e-7 (forward results 3.8e-7, largest element 6e-6).
    The backward pass branches on the sign of the pre-activations: the few in 1e8 that lie within
    rounding of zero take the other branch, which moved a hidden gradient by 2.8e-4 (largest
    element 0.35) and weight gradients by 1.7e-4.  bfloat16 storage rounds sums that differ in the
    last fp32 bits to neighbouring values: 3e-4 (6e-2) with other partitions, and up to 1.4e-2
    (largest element 1.9) where the other layer order rounds other intermediates."""
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.99}
    if case["do"] == "forward":
        return {"rel": 4e-6, "max": 6e-5}
    return {"rel": 1e-3, "max": 0.99}


def _graph(case, seed):
    """Distinct R-MAT edges as CSR by destination (rowptr int64, colidx int32, numpy), columns ascending."""
    n, edges = case["n"], case["edges"]
    g = torch.Generator(device=DEVICE).manual_seed(seed * 1_000_003 + 17)
    scale = max(1, (n - 1).bit_length())
    a, b, c = RMAT_ABC
    perm = torch.randperm(n, generator=g, device=DEVICE)
    keys = torch.empty(0, dtype=torch.int64, device=DEVICE)
    for _ in range(16):
        m = int(1.3 * (edges - keys.numel())) + 1024
        s = torch.zeros(m, dtype=torch.int64, device=DEVICE)
        t = torch.zeros(m, dtype=torch.int64, device=DEVICE)
        for _level in range(scale):
            r = torch.rand(m, generator=g, device=DEVICE)
            sbit = r >= a + b
            tbit = ((r >= a) & ~sbit) | (r >= a + b + c)
            s = s * 2 + sbit
            t = t * 2 + tbit
        s, t = perm[(s * n) >> scale], perm[(t * n) >> scale]
        if case["symmetric"]:
            s, t = torch.minimum(s, t), torch.maximum(s, t)
        keep = s != t
        keys = torch.unique(torch.cat([keys, (t * n + s)[keep]]))
        if keys.numel() >= edges:
            break
    if keys.numel() > edges:
        keys = keys[torch.randperm(keys.numel(), generator=g, device=DEVICE)[:edges]]
    t, s = keys // n, keys % n
    if case["symmetric"]:
        s, t = torch.cat([s, t]), torch.cat([t, s])
    if case["model"] == "gcn":
        v = torch.arange(n, device=DEVICE)
        s, t = torch.cat([s, v]), torch.cat([t, v])
    keys = torch.sort(t * n + s).values
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    rowptr[1:] = torch.cumsum(torch.bincount(keys // n, minlength=n), 0)
    return rowptr.cpu().numpy(), (keys % n).to(torch.int32).cpu().numpy()


def _weights(case, seed):
    """Glorot-uniform weights, small biases, attention vectors for attention layers (host, fp32)."""
    d = _dims(case)
    rng = np.random.default_rng([seed, 3])
    heads = [int(h) for h in case["heads"].split("x")] if case["heads"] else [1] * (len(d) - 1)
    out = []
    for l in range(len(d) - 1):
        bound = math.sqrt(6.0 / (d[l] + d[l + 1]))
        layer = {"W": rng.uniform(-bound, bound, (d[l], d[l + 1])).astype(np.float32),
                 "b": (0.1 * rng.standard_normal(d[l + 1])).astype(np.float32)}
        if case["model"] == "sage":
            layer["Ws"] = rng.uniform(-bound, bound, (d[l], d[l + 1])).astype(np.float32)
        if case["model"] == "gat":
            layer["heads"] = heads[l]
            for key in ("a_src", "a_dst"):
                layer[key] = (rng.standard_normal(d[l + 1]) * 0.5 / math.sqrt(d[l + 1])).astype(np.float32)
        out.append(layer)
    return out


def prepare(case, seed):
    d, n = _dims(case), case["n"]
    rowptr, colidx = _graph(case, seed)
    g = torch.Generator(device=DEVICE).manual_seed(seed * 1_000_003 + 29)
    x = torch.randn((n, d[0]), generator=g, device=DEVICE).cpu().numpy()
    labels = torch.randint(0, d[-1], (n,), generator=g, device=DEVICE, dtype=torch.int32).cpu().numpy()
    mask = (torch.rand(n, generator=g, device=DEVICE) < case["train_frac"]).to(torch.uint8).cpu().numpy()
    mask[0] = 1
    switches = {}
    if case["budget"]:
        switches = dict(hbm_budget_bytes=int(case["budget"] * n * (sum(d) + sum(d[1:])) * 4) + (8 << 20),
                        layer_order="auto" if case["tuned"] else "aggregate")
    elif case["tuned"]:
        switches = dict(layer_order="auto", fuse_gather=True, masked_backward=True, keep_forward="auto")
    session = Session(case["model"], d, rowptr, colidx, case["k"], case["part"], seed, x, _weights(case, seed),
                      labels, mask, dtype=case["dtype"], **switches)
    return {"case": case, "session": session, "seed": seed, "step": 0,
            "order": [int(p) for p in session.ctx.get_schedule()],
            "transform_first": [session.ctx.layer_is_transform_first(l) for l in range(1, len(d))]}


def run(state):
    s, do = state["session"], state["case"]["do"]
    if do == "forward":
        ctx, stream = s.ctx, s.stream
        for l in range(1, s.L + 1):
            if state["transform_first"][l - 1]:
                for p in state["order"]:
                    ctx.layer_transform_fwd(l, p, stream)
            for p in state["order"]:
                ctx.gather_boundary(l, p, stream)
                ctx.layer_fwd(l, p, stream)
        return {"act": s.act}
    if do == "train":
        loss = s.train(1, optimizer="adam", lr=0.003, dropout=0.5, seed=state["seed"], first_epoch=state["step"])[0]
        state["step"] += 1
    else:
        loss = s.epoch()
    out = {"loss": loss, "act": s.act, "grad_act": s.gact, "grad_w": s.gw}
    if do == "train":
        out["w"] = s.w
    return out
