"""The work that users of the package have it do, as cases to be timed.

Sizes and constants follow the package's own configurations (synth.CONFIGS:
2,000 x 32, 70,000 x 784, 1,400,000 x 100, 1,000,000 x 64 and the encoder's
784 -> 512 -> 512 -> 2 on 1,000,000 points in batches of 8,192) and the data
sets of the thesis (48,600 points).  A case is a dict of plain values; its
``kind`` names the entry point:

  loop     Context.step: ``iters`` iterations of the layout loop
  staged   late_stage.staged_run: a whole run from the data's kNN graph on
           (contexts made and destroyed, helper graph, mask, l1 stage)
  stress   IVHDStress forward and backward on an edge plan (loss, gradient)
  knn      ivhd_knn_build: the exact kNN graph
  ivf      ivf_knn_graph: the approximate kNN graph, training included
  train    one training step of the parametric encoder (loss, gradients)
  embed    new points placed by the encoder's forward pass
  quality  evaluate.quality: neighbourhoods, ranks and scores on sampled rows

Inputs are Gaussian mixtures like synth's, made on the GPU from the seed; the
loop's graphs are kNN-shaped (in-cluster targets with a Pareto popularity, as
synth.standin_graph draws them).
"""
import math

import numpy as np
import torch

import paper_2303_05455_amd as ivhd
from paper_2303_05455_amd import autograd, evaluate, late_stage, parametric

A, EPS = 0.9, 1e-12
HIDDEN = 512
TAU_PER_POINT = 1e-4   # the benchmark's threshold of the adaptive b


# ---- the cases -------------------------------------------------------------

def listed():
    return [
        # one animation frame of an interactive layout of a small data set
        dict(name="frame_2k", kind="loop", M=2000, nn=2, rn=1, R=0, c=0.1, mode="det", opt="plain", iters=10),
        # the MNIST-sized loop: launches of a few microseconds each
        dict(name="loop_70k", kind="loop", M=70000, nn=5, rn=1, R=0, c=0.01, mode="det", opt="plain", iters=100),
        # the headline loop: 1.4M points, random neighbours redrawn every 100 iterations
        dict(name="loop_1400k", kind="loop", M=1400000, nn=2, rn=1, R=100, c=0.1, mode="det", opt="plain", iters=100),
        # the same in the atomic mode
        dict(name="loop_1400k_atomic", kind="loop", M=1400000, nn=2, rn=1, R=100, c=0.1, mode="atomic", opt="plain",
             iters=100),
        # a whole refinement run at a data set's size in the thesis (48,600 points)
        dict(name="staged_48k", kind="staged", M=48600, N=128, nn=5, rn=1, R=50, c=0.01, T=200, mask=100, l1=10),
        # the stress as a training loss at a million points
        dict(name="stress_1m", kind="stress", M=1000000, nn=5, rn=1, c=0.1),
        # exact graphs: narrow data, many points; and the MNIST shape
        dict(name="knn_400k_100", kind="knn", M=400000, N=100, k=2, clusters=50),
        dict(name="knn_70k_784", kind="knn", M=70000, N=784, k=5, clusters=10),
        # the approximate graph of more points than one wants to pay the exact one for
        dict(name="ivf_200k_100", kind="ivf", M=200000, N=100, k=5, clusters=20, nlist=512, nprobe=8, lloyd=4),
        # the encoder: one training batch, and held-out points
        dict(name="train_57k", kind="train", batch=8192, nn=5, rn=1, N=784),
        dict(name="embed_200k", kind="embed", rows=200000, N=784),
        # the layout's quality on a sample of the points
        dict(name="quality_200k", kind="quality", M=200000, N=100, rows=2000, clusters=20),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["loop", "loop", "loop", "loop", "staged", "stress", "stress", "knn", "knn", "ivf", "train",
                       "embed", "quality"])
    if kind == "loop":
        mode = rng.choice(["det", "det", "det", "atomic"])
        opt = rng.choice(["plain", "plain", "nesterov", "adaptive"] if mode == "det" else ["plain", "nesterov"])
        return dict(kind=kind, M=_log_uniform(rng, 1500, 1400000), nn=rng.choice([2, 2, 3, 5, 8]),
                    rn=rng.choice([1, 1, 1, 2]), R=rng.choice([0, 25, 100]), c=rng.choice([0.01, 0.1]), mode=mode,
                    opt=opt, iters=rng.randint(1, 100))
    if kind == "staged":
        T = rng.randint(60, 200)
        return dict(kind=kind, M=_log_uniform(rng, 3000, 48600), N=rng.randint(20, 128), nn=rng.choice([2, 3, 5]),
                    rn=1, R=rng.choice([0, 50]), c=rng.choice([0.01, 0.1]), T=T, mask=T // 2, l1=10)
    if kind == "stress":
        return dict(kind=kind, M=_log_uniform(rng, 5000, 1000000), nn=rng.choice([2, 3, 5]), rn=rng.choice([1, 1, 2]),
                    c=rng.choice([0.01, 0.1]))
    if kind == "knn":
        N = rng.choice([_log_uniform(rng, 16, 128), _log_uniform(rng, 129, 784)])
        # no more multiplications than the largest listed case
        top = int(math.sqrt(400000.0 ** 2 * 128 / max(128, 2 * N)))
        return dict(kind=kind, M=_log_uniform(rng, 5000, top), N=N, k=rng.choice([2, 3, 5, 10, 20]),
                    clusters=rng.choice([10, 20, 50]))
    if kind == "ivf":
        return dict(kind=kind, M=_log_uniform(rng, 30000, 200000), N=_log_uniform(rng, 32, 128),
                    k=rng.choice([2, 3, 5, 10]), clusters=20, nlist=rng.choice([128, 256, 512]),
                    nprobe=rng.choice([4, 8, 16]), lloyd=rng.randint(2, 4))
    if kind == "train":
        return dict(kind=kind, batch=_log_uniform(rng, 500, 8192), nn=rng.choice([2, 5]), rn=1,
                    N=rng.choice([784, 100, _log_uniform(rng, 30, 784)]))
    if kind == "embed":
        return dict(kind=kind, rows=_log_uniform(rng, 1000, 200000), N=rng.choice([784, 100,
                                                                                   _log_uniform(rng, 30, 784)]))
    return dict(kind=kind, M=_log_uniform(rng, 10000, 200000), N=_log_uniform(rng, 16, 128),
                rows=_log_uniform(rng, 300, 2000), clusters=rng.choice([10, 20]))


# ---- inputs ----------------------------------------------------------------

def _gen(seed, stream=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + stream)
    return g


def _labels(M, K, seed):
    """Cluster of every point, shuffled (equal clusters)."""
    order = torch.randperm(M, generator=_gen(seed, 1), device="cuda")
    return order % K


def _mixture(M, N, K, seed, labels=None, positive=False):
    """Points of a Gaussian mixture, centres ~ N(0, 16 I), sigma 1: float32 [M, N]."""
    labels = _labels(M, K, seed) if labels is None else labels
    centres = 4.0 * torch.randn((K, N), generator=_gen(seed, 2), device="cuda")
    x = torch.randn((M, N), generator=_gen(seed, 3), device="cuda")
    x += centres[labels]
    return x.clamp_(min=0.0) if positive else x


def _graph(M, nn, K, seed):
    """kNN-shaped lists: nn distinct in-cluster targets per point with a
    Pareto(2.2) popularity (a tail of hubs, as in high dimensions)."""
    labels = _labels(M, K, seed)
    order = torch.argsort(labels, stable=True)
    u = torch.rand(M, generator=_gen(seed, 4), device="cuda", dtype=torch.float64)
    weight = (1024.0 * (1.0 - u) ** (-1.0 / 2.2)).to(torch.int64)     # whole numbers: exact sums
    cdf = torch.cumsum(weight[order], 0)
    count = torch.bincount(labels, minlength=K)
    last = torch.cumsum(count, 0) - 1
    hi = cdf[last][labels]
    lo = torch.where(labels > 0, cdf[last[(labels - 1).clamp(min=0)]], torch.zeros_like(hi))
    g = _gen(seed, 5)
    ids = torch.arange(M, device="cuda")
    out = torch.full((M, nn), -1, device="cuda", dtype=torch.int64)
    for q in range(nn):
        todo = ids
        while todo.numel():
            r = torch.rand(todo.numel(), generator=g, device="cuda", dtype=torch.float64)
            at = lo[todo] + (r * (hi - lo)[todo]).to(torch.int64)
            j = order[torch.searchsorted(cdf, at, right=True).clamp(max=M - 1)]
            bad = (j == todo) | (out[todo, :q] == j[:, None]).any(1)
            out[todo, q] = j
            todo = todo[bad]
    return out.to(torch.int32)


def _clusters_of(M):
    return max(1, min(50, M // 200))


def _step_b(nn_idx, rn):
    """A quarter of the heavy-ball stability bound (ParametricIVHD.embed's rule)."""
    flat = nn_idx.reshape(-1).long()
    indeg = torch.bincount(flat[flat >= 0], minlength=nn_idx.shape[0])
    return 0.25 * 2 * (1 + A) / (int(indeg.max()) + nn_idx.shape[1] + 2 * rn + 2)


def _layout(M, seed):
    return torch.rand((M, 2), generator=_gen(seed, 6), device="cuda")


def _loop_inputs(case, seed):
    M = case["M"]
    nn_idx = _graph(M, case["nn"], _clusters_of(M), seed)
    b = _step_b(nn_idx, case["rn"]) * (0.5 if case["opt"] == "nesterov" else 1.0)
    return nn_idx, _layout(M, seed), b


def _stress_inputs(case, seed):
    M = case["M"]
    nn_idx = _graph(M, case["nn"], _clusters_of(M), seed)
    rn_idx = torch.from_numpy(_draw_rn(nn_idx.cpu().numpy(), case["rn"], seed, 0)).cuda() if M <= 20000 else \
        (torch.arange(M, device="cuda")[:, None]
         + torch.randint(1, M, (M, case["rn"]), generator=_gen(seed, 7), device="cuda")) % M
    return nn_idx, rn_idx.to(torch.int32).contiguous(), _layout(M, seed)


def _staged_inputs(case, seed):
    x = _mixture(case["M"], case["N"], 10, seed)
    return x, ivhd.ivhd_knn_build(x, case["nn"]), _layout(case["M"], seed)


def _mlp_params(N, seed):
    """Glorot-uniform weights and zero biases in the encoder's flat order."""
    parts = []
    for k, (o, i) in enumerate(((HIDDEN, N), (HIDDEN, HIDDEN), (2, HIDDEN))):
        s = math.sqrt(6.0 / (i + o))
        w = (2 * torch.rand((o, i), generator=_gen(seed, 10 + k), device="cuda") - 1) * s
        parts += [w.reshape(-1), torch.zeros(o, device="cuda")]
    return torch.cat(parts)


def _train_inputs(case, seed):
    """A batch as the training epoch lays it out: B sources, their nn targets
    (points of the source's cluster), their rn targets; and its edge lists."""
    B, nn, rn, N = case["batch"], case["nn"], case["rn"], case["N"]
    g = _gen(seed, 8)
    lab = torch.randint(0, 20, (B,), generator=g, device="cuda")
    labels = torch.cat([lab, lab.repeat_interleave(nn),
                        torch.randint(0, 20, (B * rn,), generator=g, device="cuda")])
    x = _mixture(labels.numel(), N, 20, seed, labels=labels, positive=True)
    R = labels.numel()
    lnn = torch.full((R, nn), -1, device="cuda", dtype=torch.int32)
    lrn = torch.full((R, rn), -1, device="cuda", dtype=torch.int32)
    src = torch.arange(B, device="cuda", dtype=torch.int32)[:, None]
    lnn[:B] = B + src * nn + torch.arange(nn, device="cuda", dtype=torch.int32)
    lrn[:B] = B + B * nn + src * rn + torch.arange(rn, device="cuda", dtype=torch.int32)
    return x.to(torch.bfloat16), lnn, lrn


def _bits(x16):
    return x16.contiguous().view(torch.int16)


def _quality_inputs(case, seed):
    M, K = case["M"], case["clusters"]
    labels = _labels(M, K, seed)
    x = _mixture(M, case["N"], K, seed, labels=labels)
    at = 3.0 * torch.randn((K, 2), generator=_gen(seed, 14), device="cuda")
    y = at[labels] + 0.2 * x[:, :2] + 0.1 * torch.randn((M, 2), generator=_gen(seed, 15), device="cuda")
    rows = torch.randperm(M, generator=_gen(seed, 16), device="cuda")[:case["rows"]].sort().values
    return x, y.contiguous(), rows.cpu().numpy().astype(np.int32), labels.cpu().numpy().astype(np.int32)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "seed": seed}
    if kind == "loop":
        nn_idx, y, b = _loop_inputs(case, seed)
        s["ctx"] = ivhd.Context(nn_idx, y, rn=case["rn"], a=A, b=b, c=case["c"], eps=EPS, seed=seed,
                                rn_resample_every=case["R"], mode=case["mode"], nesterov=case["opt"] == "nesterov")
        if case["opt"] == "adaptive":
            s["ctx"].set_adaptive(True, tau=TAU_PER_POINT * case["M"])
    elif kind == "staged":
        s["x"], s["nn"], s["y0"] = _staged_inputs(case, seed)
        s["b"] = _step_b(s["nn"], case["rn"])
    elif kind == "stress":
        nn_idx, rn_idx, y = _stress_inputs(case, seed)
        s["edges"] = autograd.StressEdges(nn_idx, rn_idx, c=case["c"], eps=EPS)
        s["y"] = y.requires_grad_(True)
    elif kind in ("knn", "ivf"):
        s["x"] = _mixture(case["M"], case["N"], case["clusters"], seed)
    elif kind == "train":
        x16, lnn, lrn = _train_inputs(case, seed)
        s["x16"] = _bits(x16)
        s["enc"] = parametric.ParametricIVHD(case["N"], (HIDDEN, HIDDEN), seed=seed, max_rows=x16.shape[0])
        s["enc"].set_params(_mlp_params(case["N"], seed))
        s["edges"] = autograd.StressEdges(lnn, lrn, reorder=False)
        s["loss"] = torch.zeros((), dtype=torch.float64, device="cuda")
    elif kind == "embed":
        x = _mixture(case["rows"], case["N"], 20, seed, positive=True)
        s["x16"] = _bits(x.to(torch.bfloat16))
        s["enc"] = parametric.ParametricIVHD(case["N"], (HIDDEN, HIDDEN), seed=seed)
        s["enc"].set_params(_mlp_params(case["N"], seed))
    else:
        s["x"], s["y"], s["rows"], s["labels"] = _quality_inputs(case, seed)
    return s


# ---- one pass --------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "loop":
        ctx = s["ctx"].step(case["iters"])
        return {"y": ctx.y, "v": ctx.v}
    if kind == "staged":
        y = s["y0"].clone()
        v = torch.zeros_like(y)
        info = late_stage.staged_run(s["nn"], y, v, T=case["T"], x=s["x"], mask_iters=case["mask"],
                                     l1_iters=case["l1"], rn=case["rn"], a=A, b=s["b"], c=case["c"], eps=EPS,
                                     seed=s["seed"], rn_resample_every=case["R"])
        return {"y": y, "v": v, "masked": info["nn_masked"]}
    if kind == "stress":
        y = s["y"]
        y.grad = None
        loss = autograd.ivhd_stress_loss(y, s["edges"])
        loss.backward()
        return {"loss": loss.detach(), "grad": y.grad}
    if kind == "knn":
        return ivhd.ivhd_knn_build(s["x"], case["k"])
    if kind == "ivf":
        return ivhd.ivf_knn_graph(s["x"], case["k"], case["nlist"], case["nprobe"], case["lloyd"])
    if kind == "train":
        ivhd.ivhd_enc_train_step(s["enc"].handle, s["x16"], s["edges"].handle, 0.1, EPS, 1e-3, 1.0 / case["batch"],
                                 s["loss"])
        return {"loss": s["loss"].to(torch.float32), "grads": s["enc"].grads()}
    if kind == "embed":
        return s["enc"].embed(s["x16"])
    q = evaluate.quality(s["x"], s["y"], s["rows"], labels=s["labels"])
    return {"q_nx": q["q_nx"], "cf": q["cf"], "trust": q["trust"], "nx": q["nx"]}


# ---- what a pass cannot do without ------------------------------------------

def work(case):
    kind = case["kind"]
    if kind in ("loop", "staged"):
        M, nn, rn = case["M"], case["nn"], case["rn"]
        iters = case["iters"] if kind == "loop" else case["T"]
        # per iteration: positions and velocities read and written, and per
        # edge its index and its reaction at the other end
        w = {"bytes": iters * (32.0 * M + 8.0 * M * (nn + rn)), "flops": iters * M * (8.0 * nn + 24.0 * rn + 8.0)}
        if kind == "staged":
            w["bytes"] += 4.0 * M * case["N"] + 16.0 * nn * M
            w["flops"] += 2.0 * M * M * case["N"]
        return w
    if kind == "stress":
        M, nn, rn = case["M"], case["nn"], case["rn"]
        return {"bytes": 16.0 * M + 8.0 * M * (nn + rn), "flops": M * (14.0 * nn + 36.0 * rn)}
    if kind == "knn":
        M, N = case["M"], case["N"]
        return {"bytes": 4.0 * M * (N + case["k"]), "flops": 2.0 * M * M * N}
    if kind == "ivf":
        M, N, nl = case["M"], case["N"], case["nlist"]
        return {"bytes": 4.0 * M * (N + case["k"]),
                "flops": 2.0 * M * nl * N * (case["lloyd"] + 2) + 2.0 * M * N * (M / nl) * case["nprobe"]}
    n1 = case["N"] * HIDDEN + HIDDEN * HIDDEN + 2 * HIDDEN
    if kind == "train":
        R = case["batch"] * (1 + case["nn"] + case["rn"])
        # forward, weight gradients, and the input gradients of all but the first layer
        return {"bytes": 2.0 * R * case["N"] + 36.0 * n1, "flops": R * (4.0 * n1 + 2.0 * (n1 - case["N"] * HIDDEN))}
    if kind == "embed":
        R = case["rows"]
        return {"bytes": 2.0 * R * case["N"] + 8.0 * R + 2.0 * n1, "flops": 2.0 * R * n1}
    M, N, Q = case["M"], case["N"], case["rows"]
    # distances in the data for the neighbourhoods and for the ranks, and in the layout
    return {"bytes": 4.0 * M * (N + 2), "flops": 3.0 * Q * M * (2.0 * N + 2.0)}


# ---- the same in 64 bits ----------------------------------------------------

def _splitmix(x):
    with np.errstate(over="ignore"):
        z = x + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _draw_rn(nn_idx, rn, seed, epoch):
    """The random neighbours of one epoch by the rule of the C header."""
    M = nn_idx.shape[0]
    out = np.full((M, rn), -1, np.int64)
    with np.errstate(over="ignore"):
        for r in range(rn):
            todo = np.arange(M)
            for t in range(256):
                i = todo.astype(np.uint64)
                ctr = ((np.uint64(epoch) * np.uint64(M) + i) * np.uint64(rn) + np.uint64(r)) * np.uint64(256)
                h = _splitmix(np.uint64(seed) ^ _splitmix(ctr + np.uint64(t)))
                j = (h % np.uint64(M - 1)).astype(np.int64)
                j += j >= todo
                out[todo, r] = j
                clash = (nn_idx[todo] == j[:, None]).any(1) | (out[todo, :r] == j[:, None]).any(1)
                todo = todo[clash]
                if not todo.size:
                    break
    return out.astype(np.int32)


class _Edges64:
    """Force and stress of fixed lists in float64 (absent slots: -1)."""

    def __init__(self, nn_idx, rn_idx, c):
        def pairs(idx):
            src = torch.arange(idx.shape[0], device="cuda")[:, None].expand_as(idx).reshape(-1)
            dst = idx.reshape(-1).long()
            keep = dst >= 0
            return src[keep], dst[keep]
        self.nn, self.rn, self.c = pairs(nn_idx), pairs(rn_idx), float(np.float32(c))

    def force(self, y, l1=False):
        f = torch.zeros_like(y)
        s, t = self.nn
        d = y[t] - y[s]
        if l1:
            d = d.abs().sum(1, keepdim=True) * d.sign()
        f.index_add_(0, s, d).index_add_(0, t, -d)
        s, t = self.rn
        d = y[s] - y[t]
        if l1:
            d = self.c * (1 - d.abs().sum(1, keepdim=True)) * d.sign()
        else:
            r = d.norm(dim=1, keepdim=True)
            d = self.c * (1 - r) * d / r.clamp(min=EPS)
        return f.index_add_(0, s, d).index_add_(0, t, -d)

    def stress(self, y):
        s, t = self.nn
        e = (y[s] - y[t]).square().sum()
        s, t = self.rn
        return e + self.c * (1 - (y[s] - y[t]).norm(dim=1)).square().sum()


def _loop64(nn_idx, y, v, *, rn, b, c, seed, R, n0, iters, opt="plain", l1=False, tau=0.0):
    """Iterations n0 .. n0 + iters - 1 in float64."""
    host = nn_idx.cpu().numpy()
    a, b = float(np.float32(A)), float(np.float32(b))
    edges, held = None, -1
    for n in range(n0, n0 + iters):
        epoch = n // R if R > 0 else 0
        if epoch != held:
            edges, held = _Edges64(nn_idx, torch.from_numpy(_draw_rn(host, rn, seed, epoch)).cuda(), c), epoch
        v1 = a * v + b * edges.force(y + a * v if opt == "nesterov" else y, l1)
        if opt == "adaptive":
            dT = float(v1.square().sum() - v.square().sum())
            if not abs(dT) <= tau:
                b *= float(np.float32(1.05)) if dT < -tau else 0.5
                continue
        v = v1
        y = y + v
    return y, v


def _knn64(x, k, rows=None):
    """Neighbours by (distance, index) in float64, the row itself left out."""
    x = x.double()
    sq = x.square().sum(1)
    rows = torch.arange(x.shape[0], device="cuda") if rows is None else rows
    out = []
    for part in rows.split(2048):
        d = sq[None, :] - 2 * x[part] @ x.T
        d[torch.arange(part.numel(), device="cuda"), part] = math.inf
        out.append(d.topk(k, dim=1, largest=False).indices)
    return torch.cat(out)


def _staged64(case, seed):
    x, nn_idx, y = _staged_inputs(case, seed)
    T, mask, l1, nn = case["T"], case["mask"], case["l1"], case["nn"]
    kw = dict(rn=case["rn"], c=case["c"], seed=seed, R=case["R"])
    b = _step_b(nn_idx, case["rn"])
    y, v = _loop64(nn_idx, y.double(), torch.zeros_like(y).double(), b=b, n0=0, iters=T - mask, **kw)
    helper = _knn64(x, 4 * nn)
    me = torch.arange(case["M"], device="cuda")
    kept = [torch.where((helper[nn_idx[:, q].long()] == me[:, None]).any(1), nn_idx[:, q], -1) for q in range(nn)]
    masked = torch.stack(kept, 1).to(torch.int32)
    y, v = _loop64(masked, y, v, b=b, n0=T - mask, iters=mask - l1, **kw)
    y, v = _loop64(masked, y, v, b=b / 2, n0=T - l1, iters=l1, l1=True, **kw)
    return {"y": y, "v": v, "masked": None}


def _mlp64(N, params, x16):
    at, out = 0, []
    for o, i in ((HIDDEN, N), (HIDDEN, HIDDEN), (2, HIDDEN)):
        out.append((params[at:at + o * i].view(o, i), params[at + o * i:at + o * i + o]))
        at += o * i + o
    h = x16.double()
    for k, (w, bias) in enumerate(out):
        h = h @ w.T + bias
        h = h.relu() if k < 2 else h
    return h


def _rank_lists64(z, rows, k):
    """Positions 1..k of the float64 (distance, index) order around each row."""
    z = z.double()
    out = []
    for part in rows.split(256):
        d = torch.zeros((part.numel(), z.shape[0]), dtype=torch.float64, device="cuda")
        for n in range(z.shape[1]):
            d += (z[:, n][None, :] - z[part, n][:, None]).square()
        out.append(torch.sort(d, dim=1, stable=True).indices)
    return out


def _quality64(case, seed):
    x, y, rows, labels = _quality_inputs(case, seed)
    rows, labels = torch.from_numpy(rows).cuda().long(), torch.from_numpy(labels).cuda()
    M, Q = case["M"], case["rows"]
    ky, hit, same, trust = 100, 0, {2: 0, 10: 0, 100: 0}, 0
    oy = torch.cat([o[:, 1:ky + 1] for o in _rank_lists64(y, rows, ky)])
    for part, o, n in zip(rows.split(256), _rank_lists64(x, rows, 10), oy.split(256)):
        rank = torch.empty_like(o).scatter_(1, o, torch.arange(M, device="cuda").expand_as(o))
        r10 = rank.gather(1, n[:, :10])
        inside = (o[:, 1:11, None] == n[:, None, :10]).any(1)
        hit += int(inside.sum())
        trust += int(torch.where(inside, 0, r10 - 10).sum())
        for k in same:
            same[k] += int((labels[n[:, :k]] == labels[part][:, None]).sum())
    return {"q_nx": {10: hit / (10 * Q)}, "cf": {k: v / (k * Q) for k, v in same.items()},
            "trust": {10: 1 - 2 / (Q * 10 * (2 * M - 31)) * trust}, "nx": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "loop":
        nn_idx, y, b = _loop_inputs(case, seed)
        y, v = _loop64(nn_idx, y.double(), torch.zeros_like(y).double(), rn=case["rn"], b=b, c=case["c"], seed=seed,
                       R=case["R"], n0=0, iters=case["iters"], opt=case["opt"], tau=TAU_PER_POINT * case["M"])
        return {"y": y, "v": v}
    if kind == "staged":
        return _staged64(case, seed)
    if kind == "stress":
        nn_idx, rn_idx, y = _stress_inputs(case, seed)
        e = _Edges64(nn_idx, rn_idx, case["c"])
        y = y.double()
        return {"loss": e.stress(y), "grad": -2 * e.force(y)}
    if kind == "train":
        x16, lnn, lrn = _train_inputs(case, seed)
        p = _mlp_params(case["N"], seed).double().requires_grad_(True)
        z = _mlp64(case["N"], p, x16)
        e = _Edges64(lnn, lrn, 0.1)
        loss = e.stress(z)
        loss.backward()
        return {"loss": loss.detach(), "grads": p.grad}
    if kind == "embed":
        x = _mixture(case["rows"], case["N"], 20, seed, positive=True)
        return _mlp64(case["N"], _mlp_params(case["N"], seed).double(), x.to(torch.bfloat16))
    if kind == "quality":
        return _quality64(case, seed)
    return None     # knn, ivf: whole numbers
