"""The work that a user of this library has it do, through the public entry points of the binding: training steps of
a class-split fully-connected + softmax layer (forward, combine, backward), the step with the weight update folded
in, validation loss, softmax probabilities, arg-max predictions, and the two ends of the bridge layer.

A case is a dict of plain values:
  kind     step | sgd | loss | probs | top1 | bridge
  B, D     rows and features
  widths   widths of the shards that this GPU runs one after another, as text ("500,500")
  offset   global id of the first class of the first shard
  classes  classes of the whole layer (labels range over these)
  peers    shards that other GPUs hold: their row statistics take part in the combine
  bias     whether the layer has a bias
  mean     gradient of the mean loss (1/B, and the mean loss is asked for) instead of the summed loss
  relu     features are ReLU outputs (pooled image features) instead of normal (hidden states)
  w_sigma  standard deviation of the weights
  zipf     exponent of the Zipf label distribution, 0 = uniform labels
"""
import math

import torch

from paper_2011_09208_amd import binding as ws


def _case(name, kind, B, D, widths, **kw):
    c = dict(name=name, kind=kind, B=B, D=D, widths=widths, offset=0, classes=sum(int(w) for w in widths.split(",")),
             peers=0, bias=False, mean=False, relu=True, w_sigma=0.01, zipf=0.0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest training step: a small batch on a small layer cut in two; launches and latency count
        _case("step_tiny", "step", 32, 256, "500,500", relu=False, w_sigma=0.02),
        # the 100K-class classifier at one GPU's ordinary batch, unsharded: more bytes than flops
        _case("step_b256", "step", 256, 2048, "100000"),
        # one GPU's equal share of that layer in an eight-way split; the other GPUs' row statistics have arrived
        _case("step_shard", "step", 1024, 2048, "12500", offset=37500, classes=100000, peers=7),
        # uneven shards of a 3:1 capacity ratio, hot classes first
        _case("step_uneven", "step", 1024, 2048, "37500,12500,37500,12500", zipf=1.1),
        # the whole 100K-class layer at the large batch (the benchmark's workload)
        _case("step_b1024", "step", 1024, 2048, "100000"),
        # token rows against one GPU's share of a 400K vocabulary: long contraction over the rows in dW
        _case("step_vocab", "step", 8192, 1024, "50000", classes=400000, peers=7, relu=False, w_sigma=0.02, zipf=1.0),
        # nothing a multiple of any tile: a last partial batch, odd widths, a bias, the mean loss
        _case("step_ragged", "step", 777, 1088, "9001,14450", bias=True, mean=True, relu=False, w_sigma=0.03),
        # one GPU's share of a 1M-class layer, trained with the update folded into the backward call
        _case("sgd_million", "sgd", 1024, 2048, "125000", classes=1000000, peers=7, bias=True, mean=True),
        # validation: loss of a large batch, forward only
        _case("loss_b4096", "loss", 4096, 2048, "37500,12500", bias=True, mean=True),
        # serving: the class of one sample among 100K
        _case("top1_b1", "top1", 1, 2048, "100000", bias=True),
        # serving: softmax probabilities of a small batch over one GPU's share
        _case("probs_b32", "probs", 32, 2048, "12500", classes=100000, peers=7, bias=True),
        # the bridge's two ends: eight replicas' features in, eight shards' feature gradients summed and cut
        _case("bridge_b1024", "bridge", 1024, 2048, "100000", peers=7),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "sgd", "loss", "probs", "top1", "bridge"])
    D = 64 * _log(rng, 1, 32)
    B = _log(rng, 32, 8192) if kind in ("step", "sgd", "loss") else _log(rng, 1, 512)
    if kind == "bridge":
        B = 8 * _log(rng, 4, 256)
    # no dearer than the 1M-class share: B * D * C, and the bytes of W and of the dz scratch
    most = min(125000, 1024 * 2048 * 125000 // (B * D), 1024 * 125000 // B)
    C = _log(rng, 500, max(500, most))
    n = rng.choice([1, 1, 2, 3]) if C >= 3000 else 1
    cut = sorted(rng.sample(range(100, C - 100), n - 1)) if n > 1 else []
    widths = [b - a for a, b in zip([0] + cut, cut + [C])]
    peers = rng.choice([0, 0, 3, 7]) if kind != "bridge" else rng.choice([3, 7])
    relu = rng.random() < 0.5
    sigma = 0.01 * math.sqrt(2048.0 / D)
    return dict(kind=kind, B=B, D=D, widths=",".join(str(w) for w in widths), offset=0 if peers == 0 else rng.randrange(0, C),
                classes=C if peers == 0 else (peers + 2) * C, peers=peers, bias=rng.random() < 0.5, mean=rng.random() < 0.5,
                relu=relu, w_sigma=round(sigma, 4), zipf=rng.choice([0.0, 0.0, 1.0, 1.1]))


def _labels(case, g, dev):
    B, n = case["B"], case["classes"]
    if case["zipf"] == 0.0:
        return torch.randint(0, n, (B,), generator=g, device=dev).to(torch.int32)
    p = torch.arange(1, n + 1, device=dev, dtype=torch.float64).pow_(-case["zipf"])
    edges = torch.cumsum(p / p.sum(), 0)
    u = torch.rand(B, generator=g, device=dev, dtype=torch.float64)
    return torch.searchsorted(edges, u).clamp_(max=n - 1).to(torch.int32)


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    B, D = case["B"], case["D"]
    if case["kind"] == "bridge":
        n = case["peers"] + 1
        blocks = [torch.empty((B // n, D), device=dev, dtype=torch.bfloat16).normal_(generator=g).relu_() for _ in range(n)]
        partials = [torch.empty((B, D), device=dev).normal_(0.0, 1e-3, generator=g) for _ in range(n)]
        return dict(kind="bridge", blocks=blocks, partials=partials, X=torch.empty((B, D), device=dev, dtype=torch.bfloat16),
                    outs=[torch.empty((B // n, D), device=dev) for _ in range(n)])
    widths = [int(w) for w in case["widths"].split(",")]
    C, S = sum(widths), len(widths) + case["peers"]
    X = torch.empty((B, D), device=dev, dtype=torch.bfloat16).normal_(generator=g)
    if case["relu"]:
        X.relu_()
    W = torch.empty((C, D), device=dev, dtype=torch.bfloat16).normal_(0.0, case["w_sigma"], generator=g)
    bias = torch.empty(C, device=dev).normal_(0.0, 0.1, generator=g) if case["bias"] else None
    y = _labels(case, g, dev)
    shards, at = [], 0
    for w in widths:
        shards.append((case["offset"] + at, W[at:at + w], None if bias is None else bias[at:at + w], at, w))
        at += w
    st = dict(kind=case["kind"], X=X, W=W, bias=bias, y=y, shards=shards, peers=case["peers"], g=1.0 / B if case["mean"] else 1.0)
    st["lr"] = 0.05 if case["mean"] else 0.05 / B                  # the same step for either scale of the gradient
    nbytes = max(ws.fwd_workspace_bytes(B, D, w) for w in widths)
    if case["kind"] in ("step", "sgd"):
        nbytes = max([nbytes] + [ws.bwd_workspace_bytes(B, D, w) for w in widths])
    st["work"] = torch.empty(nbytes, device=dev, dtype=torch.uint8)
    # row statistics of the shards on other GPUs: of the size that logits of this spread give
    m, s, t = (torch.zeros((S, B), device=dev) for _ in range(3))
    if case["peers"]:
        spread = case["w_sigma"] * math.sqrt(D * (0.5 if case["relu"] else 1.0))
        first, k = len(widths), case["peers"]
        m[first:] = torch.empty((k, B), device=dev).normal_(4.0 * spread, 0.2 * spread, generator=g)
        s[first:] = torch.empty((k, B), device=dev).uniform_(0.01 * C, 0.05 * C, generator=g)
        away = (y < case["offset"]) | (y >= case["offset"] + C)
        t[first] = torch.where(away, torch.empty(B, device=dev).normal_(0.0, spread, generator=g), t[first])
    st.update(m=m, s=s, t=t, lse=torch.empty(B, device=dev), loss=torch.empty(B, device=dev),
              mean=torch.empty(1, device=dev) if case["mean"] else None)
    st["rows"] = [(m[i], s[i], t[i]) for i in range(S)]
    if case["kind"] in ("step", "sgd"):
        st["dX"] = torch.empty((B, D), device=dev)
    if case["kind"] == "step":
        st["dW"] = torch.empty((C, D), device=dev, dtype=torch.bfloat16)
        st["db"] = torch.empty(C, device=dev)
        st["grads"] = [(st["dW"][at:at + w], st["db"][at:at + w]) for _, _, _, at, w in shards]
    if case["kind"] == "probs":
        st["P"] = [torch.zeros((B, (w + 7) // 8 * 8), device=dev, dtype=torch.bfloat16)[:, :w] for w in widths]
    if case["kind"] == "top1":
        st["tv"] = torch.empty((len(widths), B), device=dev)
        st["tc"] = torch.empty((len(widths), B), device=dev, dtype=torch.int32)
        st["bv"] = torch.empty(B, device=dev)
        st["bc"] = torch.empty(B, device=dev, dtype=torch.int32)
        st["rows"] = [(st["tv"][i], st["tc"][i]) for i in range(len(widths))]
    return st


def run(st):
    if st["kind"] == "bridge":
        ws.bridge_gather(0, st["blocks"], st["X"])
        ws.bridge_reduce_partition(st["partials"], st["outs"])
        return [st["X"]] + st["outs"]
    X, y, work = st["X"], st["y"], st["work"]
    if st["kind"] == "top1":
        for (off, W, b, _, _), (tv, tc) in zip(st["shards"], st["rows"]):
            ws.split_fc_top1(X, W, b, off, tv, tc, work)
        ws.combine_top1(st["tv"], st["tc"], st["bv"], st["bc"])
        return [st["bv"], st["bc"]]
    for (off, W, b, _, _), (m, s, t) in zip(st["shards"], st["rows"]):
        ws.split_fc_fwd(X, W, b, y, off, m, s, t, work)
    ws.combine_partials(st["m"], st["s"], st["t"], st["lse"], st["loss"], st["mean"])
    out = [st["lse"], st["loss"]] + ([] if st["mean"] is None else [st["mean"]])
    if st["kind"] == "loss":
        return out + [st["m"], st["s"], st["t"]]
    if st["kind"] == "probs":
        for (off, W, b, _, _), P in zip(st["shards"], st["P"]):
            ws.split_fc_predict(X, W, b, st["lse"], P)
        return out + st["P"]
    if st["kind"] == "sgd":
        for i, (off, W, b, _, _) in enumerate(st["shards"]):
            ws.split_fc_bwd_sgd(X, W, b, st["lse"], y, off, st["g"], st["lr"], st["dX"], i > 0, work)
        return out + [st["dX"], st["W"]] + ([] if st["bias"] is None else [st["bias"]])
    for i, ((off, W, b, _, _), (dW, db)) in enumerate(zip(st["shards"], st["grads"])):
        ws.split_fc_bwd(X, W, b, st["lse"], y, off, st["g"], st["dX"], i > 0, dW, db, work)
    return out + [st["dX"], st["dW"], st["db"]]


def work(case):
    B, D = case["B"], case["D"]
    if case["kind"] == "bridge":
        n = case["peers"] + 1
        return {"bytes": 4.0 * B * D + 4.0 * (n + 1) * B * D, "flops": 1.0 * (n - 1) * B * D}
    C = sum(int(w) for w in case["widths"].split(","))
    S = case["widths"].count(",") + 1 + case["peers"]
    once = 2.0 * B * D + 2.0 * C * D + 4.0 * B                       # X, W, labels
    if case["bias"]:
        once += 4.0 * C
    stats = 12.0 * case["peers"] * B + 8.0 * B                       # the peers' statistics in, lse and loss out
    if case["kind"] == "top1":
        return {"bytes": once + 8.0 * B, "flops": 2.0 * B * D * C}
    if case["kind"] == "loss":
        return {"bytes": once + stats + 12.0 * S * B, "flops": 2.0 * B * D * C}
    if case["kind"] == "probs":                                       # the logits once, their exponentials out
        return {"bytes": once + stats + 2.0 * B * C, "flops": 2.0 * B * D * C}
    # a step: logits, dX and dW, two flops for each of B x D x C
    out = 4.0 * B * D + 2.0 * C * D + 4.0 * C                        # dX, dW (or the new W), db (or the new bias)
    return {"bytes": once + stats + out, "flops": 6.0 * B * D * C}


def tolerance(case):
    # Bridge: copies, and fp32 sums in the stated order of the shards.
    if case["kind"] == "bridge":
        return "exact"
    # Statistics, lse, loss and the arg-max logit are fp32 sums of exact bf16 products: up to 3e-7 (2-norm) and 1.1e-6
    # (largest) from the same path in 64 bits; two classes whose logits agree to fp32 rounding may swap.
    if case["kind"] == "top1":
        return {"rel": 1.2e-6, "max": 5e-6, "differ": 1e-2}
    if case["kind"] == "loss":
        return {"rel": 1.2e-6, "max": 5e-6}
    # dz, dW, the new W and the probabilities are bf16 (2^-9 each): up to 2.5e-3 (2-norm) and 5.9e-3 (largest) from
    # the same path in 64 bits.
    return {"rel": 1e-2, "max": 2.5e-2}
