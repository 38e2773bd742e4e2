"""The work that a user of the framework has it do, case by case.

A case is one pass through the public entry points on a surface point cloud:
building its multi-scale kNN graph, predicting on it (whole, or partition by
partition with halo rows dropped), one training step (forward, masked MSE,
backward, gradients summed over partitions), the optimizer step, and the
whole way from a new geometry to its prediction.  Sizes are those of the
repository's own workloads and tests, or lie between them.  Contexts run at
the library's default tiles, as a program does that sets none.
"""
import math

import numpy as np
import torch

from paper_2411_17164_amd import api

DEV = "cuda:0"
OUT_DIM = 4
AXES = (4.0, 1.5, 1.0)
EXACT_MAX_NODES = 110_000      # brute-force neighbours in 64 bits stay quick up to here
EXACT_MAX_BYTES = 1.5e11       # what exact() may keep of the edges' values


def _case(name, kind, n, levels=3, hidden=128, layers=15, precision="bf16", activation="relu", aggregate="message",
          node_in=6, parts=1, keep_hidden=True):
    return {"name": name, "kind": kind, "n": n, "levels": levels, "hidden": hidden, "layers": layers,
            "precision": precision, "activation": activation, "aggregate": aggregate, "node_in": node_in,
            "parts": parts, "keep_hidden": keep_hidden}


def listed():
    return [
        # the smallest training call: the 2,000-point sphere workload, where launches and latency count
        _case("train-fp32-sphere-2k", "train", 2000, levels=1, layers=2, precision="fp32"),
        # serving a small geometry: 15 layers of short kernels, no tape
        _case("infer-bf16-12k", "infer", 12000),
        # the headline workload: one training step of the 400k-point 3-level ellipsoid, 15 layers
        _case("train-bf16-400k", "train", 400_000),
        # a middling cloud of ragged size, shallow (the parity tests' depth)
        _case("train-bf16-70k-ragged", "train", 70271, layers=4),
        # the 4M-point car's width (H = 256) on a cloud of one partition's order
        _case("train-bf16-h256-100k", "train", 100_000, hidden=256, layers=3),
        # the production model: H = 512, SiLU, 24 inputs (position, normal, Fourier features)
        _case("train-bf16-h512-silu-50k", "train", 50_001, hidden=512, layers=2, activation="silu", node_in=24),
        # gradient aggregation over halo partitions, one partition at a time, SiLU
        _case("train-silu-3-parts-60k", "train", 60_000, layers=5, activation="silu", parts=3),
        # the plain FP32 form that the BF16 one is held against
        _case("train-fp32-50k", "train", 50_000, layers=3, precision="fp32"),
        # prediction on a large cloud, partition by partition, halo rows dropped
        _case("infer-bf16-4-parts-200k", "infer", 200_000, parts=4),
        # a new geometry end to end: graph, partition plan, first prediction on it
        _case("new-geometry-bf16-50k", "geometry", 50_000),
        # graph construction of the headline cloud
        _case("knn-400k", "knn", 400_000),
        # the optimizer step on the parameters of the production model (H = 512, 15 layers)
        _case("adam-h512", "adam", 0, hidden=512, activation="silu", node_in=24),
    ]


def _edges_of(case):
    """Edges of the union graph, about: 6 per node within a level, 3 across."""
    return 6.0 * case["n"] if case["levels"] == 1 else 8.85 * case["n"]


def _param_count(case):
    H, L = case["hidden"], case["layers"]
    enc = sum(H * k + H + 2 * (H * H + H) + 2 * H for k in (case["node_in"], 4))
    layer = (3 * H * H + H) + (H * H + H) + 2 * H + (2 * H * H + H) + (H * H + H) + 2 * H
    return enc + L * layer + 2 * (H * H + H) + OUT_DIM * H + OUT_DIM


def _cost(case):
    """Relative time of a case: edge products, FP32 ones at their slower rate."""
    c = _edges_of(case) * case["layers"] * case["hidden"] ** 2
    c *= {"train": 3.0, "infer": 1.0, "geometry": 1.0}.get(case["kind"], 0.0)
    c *= 4.0 if case["precision"] == "fp32" else 1.0
    return c * (1.0 + 0.3 * (case["parts"] - 1))  # halo rows


def draw(rng):
    most = 0.7 * _cost(listed()[2])
    while True:
        kind = rng.choice(["train"] * 6 + ["infer"] * 3 + ["geometry", "knn", "adam"])
        precision = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        hidden = rng.choice([128, 128, 128, 256, 512] if precision == "bf16" else [128, 128, 256])
        n = int(round(math.exp(rng.uniform(math.log(1000), math.log(400_000)))))
        layers = rng.choice([1, 2, 3, 4, 5, 15])
        if kind == "adam":  # any parameter count
            n, layers = 0, rng.randint(1, 24)
        parts = rng.choice([1, 1, 2, 3]) if kind in ("train", "infer") and n >= 10_000 else 1
        case = _case(None, kind, n, levels=rng.choice([1, 3, 3]), hidden=hidden,
                     layers=layers, precision=precision,
                     activation=rng.choice(["relu", "relu", "silu"]),
                     aggregate=rng.choice(["message", "message", "message", "edge"]),
                     node_in=rng.choice([6, 6, 24]), parts=parts, keep_hidden=rng.random() < 0.8)
        del case["name"]
        if _cost(case) <= most:
            return case


def _model(case):
    return api.Model(case["hidden"], case["layers"], node_in=case["node_in"], out_dim=OUT_DIM,
                     activation=case["activation"], precision=case["precision"], aggregate=case["aggregate"])


def _level_end(case):
    n = case["n"]
    return [n] if case["levels"] == 1 else [n // 16, n // 4, n]


def _cloud(n, gen):
    """n points of a bumpy ellipsoid, uniform by area, and their normals (FP32)."""
    ax = torch.tensor(AXES, dtype=torch.float64, device=DEV)
    dens = ax.prod() / ax
    got, have = [], 0
    while have < n:
        u = torch.randn(2 * n + 1024, 3, dtype=torch.float64, device=DEV, generator=gen)
        u = u / u.norm(dim=1, keepdim=True)
        keep = torch.rand(len(u), dtype=torch.float64, device=DEV, generator=gen) * dens.max() < (dens * u).norm(dim=1)
        got.append(u[keep])
        have += len(got[-1])
    p = torch.cat(got)[:n] * ax
    nrm = p / ax ** 2
    nrm = nrm / nrm.norm(dim=1, keepdim=True)
    phase = torch.rand(8, dtype=torch.float64, device=DEV, generator=gen) * (2 * math.pi)
    way = torch.randn(3, 8, dtype=torch.float64, device=DEV, generator=gen)
    p = p + (0.05 / 8) * torch.sin(2.0 * (p @ way) + phase).sum(dim=1, keepdim=True) * nrm
    return p.float().contiguous(), nrm.float()


def _inputs(case, seed):
    """Everything a program brings to the model: positions, node inputs, targets, parameters."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    s = {}
    if case["n"]:
        pos, nrm = _cloud(case["n"], gen)
        cols = [pos.double(), nrm.double()]
        if case["node_in"] == 24:
            for f in (1, 2, 4):
                cols += [torch.sin(2 * math.pi * f * pos.double()), torch.cos(2 * math.pi * f * pos.double())]
        x = torch.cat(cols, dim=1)
        sd = x.std(dim=0, unbiased=False)
        s["pos"] = pos
        s["node_in"] = ((x - x.mean(dim=0)) / torch.where(sd > 0, sd, torch.ones_like(sd))).float().contiguous()
        s["target"] = torch.randn(case["n"], OUT_DIM, device=DEV, generator=gen)
        ext = (pos.max(dim=0).values - pos.min(dim=0).values).double().tolist()
        area = 2.0 * (ext[0] * ext[1] + ext[1] * ext[2] + ext[0] * ext[2])
        w = math.sqrt(area / case["n"])
        s["edge_norm"] = np.array([[0, 0, 0, w], [w, w, w, 0.5 * w]], dtype=np.float32)
    if case["kind"] != "knn":
        parts = []
        for _, _, _, kind, shape, _ in _tensors(case):
            v = torch.randn(shape, dtype=torch.float64, device=DEV, generator=gen)
            if kind == "weight":
                v = v * math.sqrt(2.0 / (shape[0] + shape[1]))
            else:
                v = 0.05 * v + (1.0 if kind == "gamma" else 0.0)
            parts.append(v.reshape(-1))
        s["params"] = torch.cat(parts).float()
    if case["kind"] == "adam":
        s["grad"] = torch.randn(len(s["params"]), device=DEV, generator=gen) * 1e-2
    return s


def _tensors(case):
    """(block, layer, tensor, kind, shape, offset) of the parameter blob, in its documented order."""
    H, out, off = case["hidden"], [], 0
    mlps = [(0, 0, [case["node_in"], H, H, H]), (1, 0, [4, H, H, H])]
    for l in range(case["layers"]):
        mlps += [(2, l, [3 * H, H, H]), (3, l, [2 * H, H, H])]
    mlps.append((4, 0, [H, H, H, OUT_DIM]))
    for block, layer, dims in mlps:
        ents = []
        for i in range(len(dims) - 1):
            ents += [("weight", (dims[i + 1], dims[i])), ("bias", (dims[i + 1],))]
        if block != 4:
            ents += [("gamma", (H,)), ("beta", (H,))]
        for t, (kind, shape) in enumerate(ents):
            out.append((block, layer, t, kind, shape, off))
            off += int(np.prod(shape))
    return out


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    s["ctx"] = api.Context(0)
    if not case["keep_hidden"]:
        s["ctx"].set_tape(False)
    s["levels"] = _level_end(case)
    s["k_cross"] = 3 if case["levels"] > 1 else 0
    kind = case["kind"]
    if kind == "adam":
        s["opt"] = api.Adam(s["ctx"], s["params"])
        return s
    if kind == "knn":
        # repeated pairs are dropped, so the edge count varies: the senders are padded to the most there can be
        s["most_edges"] = 6 * s["levels"][0] + sum(9 * end for end in s["levels"][1:])
        return s
    s["model"] = _model(case)
    s["pos_host"] = s["pos"].cpu().numpy()
    s["out"] = torch.zeros(case["n"], OUT_DIM, device=DEV)
    if kind == "geometry":
        return s
    graph = s["ctx"].build_knn(s["pos"], s["levels"], 6, s["k_cross"])
    P = case["parts"]
    n = case["n"]
    sizes = None if P == 1 else [n * (p + 1) // P - n * p // P for p in range(P)]
    s["ps"] = api.Partset.halo(graph, s["pos_host"], sizes, case["layers"])
    if kind == "train":
        s["d_out"] = torch.zeros_like(s["out"])
        s["loss"] = torch.zeros(P, device=DEV)
        s["grad"] = torch.zeros_like(s["params"])
        s["part_grad"] = torch.zeros_like(s["params"]) if P > 1 else None
    return s


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "knn":
        row_ptr, col = ctx.build_knn(s["pos"], s["levels"], 6, s["k_cross"]).export()
        return {"row_ptr": row_ptr, "col": np.pad(col, (0, s["most_edges"] - len(col)), constant_values=-1)}
    if kind == "adam":
        opt = s["opt"]
        opt.step(s["grad"], 1e-3)
        return {"params": s["params"], "m": opt.m, "v": opt.v, "norm": opt.norm}
    if kind == "geometry":
        graph = ctx.build_knn(s["pos"], s["levels"], 6, s["k_cross"])
        ps = api.Partset.halo(graph, s["pos_host"], None, case["layers"])
        ctx.forward(s["model"], s["params"], ps, [0], s["node_in"], s["pos"], s["edge_norm"], s["out"], keep_tape=False)
        return {"out": s["out"]}
    if kind == "infer":
        for p in range(case["parts"]):
            ctx.forward(s["model"], s["params"], s["ps"], [p], s["node_in"], s["pos"], s["edge_norm"], s["out"],
                        keep_tape=False)
        return {"out": s["out"]}
    for p in range(case["parts"]):
        into = s["grad"] if p == 0 else s["part_grad"]
        ctx.forward(s["model"], s["params"], s["ps"], [p], s["node_in"], s["pos"], s["edge_norm"], s["out"])
        ctx.mse_grad(s["out"], s["target"], case["n"], s["d_out"], s["loss"][p:p + 1])
        ctx.backward(s["model"], s["params"], s["d_out"], into)
        if p:
            api.grad_accumulate(s["grad"], s["part_grad"])
    return {"out": s["out"], "loss": s["loss"], "grad": s["grad"]}


def work(case):
    """Inputs read once, outputs written once, and per layer the latents that
    the next one needs whole: a layer gathers over the graph, so it cannot
    start before the last has ended.  Halo rows are the partitions' own cost
    and are not counted."""
    n, E, H, L = case["n"], _edges_of(case), case["hidden"], case["layers"]
    s = 2 if case["precision"] == "bf16" else 4
    P = 4 * _param_count(case)
    kind = case["kind"]
    if kind == "adam":
        return {"bytes": 7 * P, "flops": 14 * (P // 4)}
    graph = 4.0 * (n + 2 * E)
    if kind == "knn":
        return {"bytes": 12.0 * n + graph, "flops": 8.0 * 32 * n}
    io = graph + n * 4.0 * (3 + case["node_in"] + OUT_DIM) + P
    latents = 2.0 * (E + n) * H * s  # in and out of a layer
    flops = 2.0 * (E * (4 * H + 2 * H * H) + n * (case["node_in"] * H + 4 * H * H + OUT_DIM * H))
    flops += L * 2.0 * (4 * E + 3 * n) * H * H
    if kind in ("infer", "geometry"):
        return {"bytes": io + L * latents, "flops": flops}
    # backward: the checkpoint in, the adjoint of the latents in and out (FP32)
    back = (E + n) * H * s + 2.0 * (E + n) * H * 4
    return {"bytes": io + P + L * (latents + back), "flops": 3.0 * flops}


def _neighbours(q, c, k):
    """k nearest of c (a prefix-sharing cloud: index i of q is index i of c where both hold it) for each q, self excluded."""
    out = []
    step = max(1, int(1.5e8 // len(c)))
    for a in range(0, len(q), step):
        x = q[a:a + step]
        d = (x[:, None, 0] - c[None, :, 0]) ** 2
        d += (x[:, None, 1] - c[None, :, 1]) ** 2
        d += (x[:, None, 2] - c[None, :, 2]) ** 2
        i = torch.arange(a, a + len(x), device=DEV)
        own = i < len(c)
        d[own.nonzero()[:, 0], i[own]] = math.inf
        out.append(d.topk(k, dim=1, largest=False).indices)
    return torch.cat(out)


def _union(case, pos):
    p, levels = pos.double(), _level_end(case)
    n, keys = len(p), []
    for l, end in enumerate(levels):
        lists = [_neighbours(p[:end], p[:end], 6)]
        if l:
            lists.append(_neighbours(p[:end], p[:levels[l - 1]], 3))
        for nb in lists:
            keys.append((torch.arange(end, device=DEV)[:, None] * n + nb).reshape(-1))
    keys = torch.unique(torch.cat(keys))
    return keys // n, keys % n


def exact(case, seed):
    """run()'s outputs in 64 bits, from the paper's equations."""
    kind = case["kind"]
    if kind == "knn":
        return None
    s = _inputs(case, seed)
    if kind == "adam":
        p, g = s["params"].double(), s["grad"].double()
        norm = g.norm()
        g = g * min(1.0, 32.0 / (norm.item() + 1e-6))
        m, v = (1 - 0.9) * g, (1 - 0.999) * g * g
        return {"params": p - 1e-3 * (m / (1 - 0.9)) / ((v / (1 - 0.999)).sqrt() + 1e-8), "m": m, "v": v,
                "norm": norm.reshape(1)}
    kept = _edges_of(case) * case["hidden"] * 8.0 * (16.0 * (case["layers"] + 1) if kind == "train" else 16.0)
    if case["n"] > EXACT_MAX_NODES or kept > EXACT_MAX_BYTES:
        return None
    recv, send = _union(case, s["pos"])
    w = s["params"].double().requires_grad_(kind == "train")
    W = {}
    for block, layer, t, _, shape, off in _tensors(case):
        W[block, layer, t] = w[off:off + int(np.prod(shape))].reshape(shape)
    act = torch.relu if case["activation"] == "relu" else torch.nn.functional.silu

    def mlp(b, l, x, depth):
        for i in range(depth):
            x = x @ W[b, l, 2 * i].T + W[b, l, 2 * i + 1]
            x = act(x) if i + 1 < depth else x
        if b == 4:
            return x
        return torch.nn.functional.layer_norm(x, (case["hidden"],), W[b, l, 2 * depth], W[b, l, 2 * depth + 1], 1e-5)

    p, norm = s["pos"].double(), torch.from_numpy(s["edge_norm"]).double().to(DEV)
    d = p[send] - p[recv]
    with torch.set_grad_enabled(kind == "train"):
        h = mlp(0, 0, s["node_in"].double(), 3)
        e = mlp(1, 0, (torch.cat([d, d.norm(dim=1, keepdim=True)], dim=1) - norm[0]) / norm[1], 3)
        for l in range(case["layers"]):
            v = mlp(2, l, torch.cat([h[recv], h[send], e], dim=1), 2)
            e = e + v
            m = torch.zeros_like(h).index_add(0, recv, e if case["aggregate"] == "edge" else v)
            h = h + mlp(3, l, torch.cat([h, m], dim=1), 2)
            del v, m
        out = mlp(4, 0, h, 3)
        if kind != "train":
            return {"out": out}
        sq = (out - s["target"].double()) ** 2 / (case["n"] * OUT_DIM)
        (grad,) = torch.autograd.grad(sq.sum(), w)
    # the loss comes by partition; its parts are the framework's own choice of cut
    loss = sq.sum().detach().reshape(1) if case["parts"] == 1 else None
    return {"out": out.detach(), "loss": loss, "grad": grad}
