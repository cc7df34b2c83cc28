"""Timed cases of libarctopk: whole calls of its public entry points.

A case is one compressor step (``Compressor.step``), one EF21M iteration with
the model update (``Compressor.model_step``) or one allocation-free step
(``arc_step_static``), over the layouts, data types, compressors and optimisers
the library accepts.  ``listed()`` gives the fixed cases, ``draw()`` further ones
of the same ranges, ``prepare()`` the buffers and the context a training program
holds, ``run()`` one pass, and ``exact()`` the same pass in 64 bits from plain
torch and numpy.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2510_26709_amd as arc

ETA = 0.1
LR, MOMENTUM, BETA1, BETA2, EPS, DECAY = 1e-3, 0.9, 0.9, 0.999, 1e-8, 5e-4
FIRST_STEP = 1000          # compressed iterations start after the warm-up
DENSE_STEPS = 1 << 30      # a case of the warm-up stays in it


# ---------------------------------------------------------------- layouts

def _conv_views(case):
    """A ResNet-18 of the given width: convolutions as out x (in*kh*kw), the
    classifier as out x in, batch-norm vectors and the bias as one row."""
    w, k = case["width"], case["stem"]
    views = [(w, 3 * k * k), (1, w), (1, w)]
    cin = w
    for cout in (w, 2 * w, 4 * w, 8 * w):
        for block in range(2):
            first = cin if block == 0 else cout
            views += [(cout, first * 9), (1, cout), (1, cout),
                      (cout, cout * 9), (1, cout), (1, cout)]
            if block == 0 and cout != cin:
                views += [(cout, cin), (1, cout), (1, cout)]
        cin = cout
    return views + [(case["classes"], 8 * w), (1, case["classes"])]


def _gpt_views(case):
    """A GPT-2 of the given hidden size, in its stored in x out shapes."""
    h = case["hidden"]
    views = [(case["vocab"], h), (1024, h)]
    for _ in range(case["layers"]):
        views += [(1, h), (1, h), (h, 3 * h), (1, 3 * h), (h, h), (1, h), (1, h), (1, h),
                  (h, 4 * h), (1, 4 * h), (4 * h, h), (1, h)]
    return views + [(1, h), (1, h)]


def _llama_views(case):
    """A Llama decoder with grouped key/value heads and an untied head."""
    h, f, kv = case["hidden"], case["ffn"], case["kv"]
    views = [(case["vocab"], h)]
    for _ in range(case["layers"]):
        views += [(h, h), (kv, h), (kv, h), (h, h), (f, h), (f, h), (h, f), (1, h), (1, h)]
    return views + [(1, h), (case["vocab"], h)]


def _views(case):
    """[(rows, cols)] of the per-tensor layouts; None for one m x n view."""
    make = {"conv": _conv_views, "gpt": _gpt_views, "llama": _llama_views}.get(case["layout"])
    return make(case) if make else None


def _dim(case):
    views = _views(case)
    return sum(r * c for r, c in views) if views else case["d"]


def _parts(case):
    """The independent selections: [(first row, rows, cols, first coordinate, K)]."""
    mu, views = case["mu"], _views(case)
    parts, row, at = [], 0, 0
    if views:
        for r, c in views:
            parts.append((row, r, c, at, 1 if r == 1 else math.ceil(mu * r)))
            row, at = row + r, at + r * c
        return parts
    n = case["n"]
    m = -(-case["d"] // n)
    nb = min(max(1, case["buckets"]), m)
    for b in range(nb):
        lo, hi = m * b // nb, m * (b + 1) // nb
        parts.append((lo, hi - lo, n, lo * n, math.ceil(mu * (hi - lo))))
    return parts


def _layout_args(case):
    parts = _parts(case)
    if _views(case):
        return {"tensors": [(r, c, k) for _, r, c, _, k in parts]}
    if len(parts) == 1:
        return {"n": case["n"], "K": parts[0][4]}
    return {"n": case["n"], "buckets": ([p[0] for p in parts] + [parts[-1][0] + parts[-1][1]],
                                        [p[4] for p in parts])}


def _kept(case):
    """Rows kept and payload values, of one node."""
    parts = _parts(case)
    return sum(p[4] for p in parts), sum(p[4] * p[2] for p in parts)


# ---------------------------------------------------------------- cases

_BASE = {"entry": "step", "compressor": "arc", "optimizer": "", "dense": False, "layout": "view",
         "N": 4, "grad": "f32", "r": 4, "mu": 0.01}


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    if c["layout"] == "view":
        c.setdefault("buckets", 0)
    return dict({"name": name}, **c) if name else c


def listed():
    return [
        # The smallest call, where launches and latency count: one million
        # coordinates of four workers, one global selection.
        _case("tiny_view", d=1_048_576, n=256),
        # A ResNet-18's flat gradient of eight workers as one view.
        _case("resnet18_view", d=11_689_512, n=512, N=8),
        # The same network with each tensor in its own view and the
        # experiments' optimiser (heavy ball with weight decay).
        _case("resnet18_tensors", entry="model", optimizer="msgd", layout="conv", width=64,
              stem=7, classes=1000, N=8),
        # The CIFAR form of that network: 3 x 3 stem (rows of 27 values), ten
        # classes, a coordinate count that is not a multiple of four.
        _case("cifar_tensors", entry="model", optimizer="msgd", layout="conv", width=64, stem=3,
              classes=10, mu=0.1),
        # GPT-2 small's flat gradient of eight workers.
        _case("gpt2s_view", d=124_439_808, n=768, N=8, mu=0.001),
        # GPT-2 small per tensor: a whole training iteration with Adam at the
        # large ratio of the pre-training runs.
        _case("gpt2s_tensors", entry="model", optimizer="adam", layout="gpt", hidden=768,
              layers=12, vocab=50257, mu=0.2),
        # The largest: a 1.1B-parameter decoder, bf16 gradients of four workers.
        _case("llama1b_view", d=1_100_048_384, n=2048, grad="bf16"),
        # One rank's own share of a deployment: the same decoder per tensor,
        # one worker, Adam.
        _case("llama1b_rank", entry="model", optimizer="adam", layout="llama", hidden=2048,
              ffn=5632, kv=256, layers=22, vocab=32000, N=1, grad="bf16"),
        # The dense iterations before compression starts.
        _case("gpt2s_warmup", entry="model", optimizer="adam", dense=True, d=124_439_808, n=768,
              grad="bf16"),
        # Rand-K of the comparison, 16 buckets of wide rows.
        _case("randk_buckets", entry="model", compressor="randk", optimizer="sgd", d=404_750_336,
              n=4096, buckets=16, N=2, grad="bf16"),
        # Top-K of the comparison, per tensor, with the merge into the model.
        _case("topk_tensors", entry="model", compressor="topk", optimizer="msgd", layout="gpt",
              hidden=768, layers=12, vocab=50257),
        # The allocation-free call on a small flat vector of odd length.
        _case("static_odd", entry="static", d=3_000_017, n=640, grad="bf16"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    c = {"N": rng.choice([1, 2, 3, 4, 4, 6, 8, 8]), "grad": rng.choice(["f32", "bf16"]),
         "r": rng.choice([4, 4, 4, 4, 2, 8]), "mu": round(_log(rng, 0.001, 0.2), 5),
         "compressor": rng.choice(["arc", "arc", "arc", "arc", "randk", "topk"]),
         "layout": rng.choice(["view", "view", "view", "conv", "gpt", "llama"])}
    if c["layout"] == "view":
        # Row widths of models (multiples of 64), of flat vectors cut anywhere
        # (multiples of 4), and odd ones; coordinate counts likewise.
        n = int(_log(rng, 64, 8192))
        c["n"] = rng.choice([n // 64 * 64, n // 64 * 64, n // 4 * 4, n | 1])
        whole = c["n"] % 4 == 0
        d = int(_log(rng, 1 << 18, 1 << (29 if whole else 28)) / c["N"])
        c["d"] = rng.choice([d // 4 * 4, d // 4 * 4, d]) if whole and d < 1 << 25 else d // 4 * 4
        c["buckets"] = rng.choice([0, 0, rng.randint(2, 40)])
    elif c["layout"] == "conv":
        c.update(width=rng.randint(24, 96), stem=rng.choice([3, 7]),
                 classes=rng.choice([10, 100, 1000]))
    elif c["layout"] == "gpt":
        c.update(hidden=64 * rng.randint(3, 14), layers=rng.randint(2, 12),
                 vocab=rng.randint(8000, 50257), N=min(c["N"], 4))
    else:
        c.update(hidden=128 * rng.randint(3, 14), layers=rng.randint(2, 12),
                 vocab=rng.randint(8000, 32000), N=min(c["N"], 2), kv=128)
        c["ffn"] = c["hidden"] * 11 // 4 // 16 * 16
    c["entry"] = rng.choice(["step", "step", "model", "model", "static"])
    if c["entry"] == "static" and (c["layout"] != "view" or c["compressor"] != "arc" or
                                   8 * c["r"] * c["N"] * (c["d"] // c["n"] + 1) > 1 << 25):
        c["entry"] = "step"
    if c["entry"] == "model":
        c["optimizer"] = rng.choice(["sgd", "msgd", "adam"])
        c["dense"] = rng.random() < 0.2
    return _case(**c)


# ---------------------------------------------------------------- one pass

def _model_config(case):
    return arc.make_model_config(
        case["optimizer"], lr=LR, momentum=MOMENTUM, beta1=BETA1, beta2=BETA2, eps=EPS,
        weight_decay=DECAY if case["optimizer"] == "msgd" else 0.0,
        dense_steps=DENSE_STEPS if case["dense"] else 0)


def _inputs(case, seed):
    """Gradients and state in the middle of a run: a shared part and every
    worker's noise, at a scale of its own for each tensor (or stretch of a flat
    vector); h follows the gradients and g follows h."""
    d, N = _dim(case), case["N"]
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    views = _views(case)
    sizes = [r * c for r, c in views] if views else [d * (i + 1) // 64 - d * i // 64
                                                     for i in range(64)]
    scale = torch.exp(torch.randn(len(sizes), generator=gen, device=dev)) * 1e-3
    scale = torch.repeat_interleave(scale, torch.tensor(sizes, device=dev), output_size=d)
    base = torch.randn(d, generator=gen, device=dev)
    grad = torch.empty((N, d), device=dev,
                       dtype=torch.bfloat16 if case["grad"] == "bf16" else torch.float32)
    h = torch.empty((N, d), device=dev)
    g = torch.empty((N, d), device=dev)
    e = torch.empty(d, device=dev)
    for i in range(N):
        grad[i] = e.normal_(generator=gen).mul_(0.3).add_(base).mul_(scale)
        h[i].normal_(generator=gen).mul_(0.2).add_(base, alpha=0.8).mul_(scale)
        g[i].copy_(e.normal_(generator=gen).mul_(0.3).mul_(scale).add_(h[i], alpha=0.7))
    got = {"grad": grad, "h": h, "g": g}
    if case["entry"] == "model":
        got["G"] = g.sum(0) if N > 1 else g[0].clone()
        got["x"] = torch.empty(d, device=dev).normal_(generator=gen).mul_(0.02)
        if case["optimizer"] in ("msgd", "adam"):
            got["m"] = e.normal_(generator=gen).mul_(0.3).add_(base).mul_(scale).clone()
        if case["optimizer"] == "adam":
            got["v"] = got["m"].square().mul_(0.1)
    return got


def prepare(case, seed):
    s = _inputs(case, seed)
    N, r = case["N"], case["r"]
    s.update(entry=case["entry"], dense=case["dense"], t=0 if case["dense"] else FIRST_STEP)
    if case["entry"] == "static":
        K, payload = _kept(case)
        s["cfg"], s["keep"] = arc.make_config(
            d=_dim(case), N=N, r=r, eta=ETA, seed=seed, compressor=case["compressor"],
            grad_dtype=arc.ARC_DTYPE_BF16 if case["grad"] == "bf16" else arc.ARC_DTYPE_F32,
            **_layout_args(case))
        s["stream"] = torch.cuda.current_stream()
        s["idx"] = torch.empty(K, dtype=torch.int32, device="cuda")
        s["agg"] = torch.empty(payload, device="cuda")
        return s
    s["comp"] = arc.Compressor(d=_dim(case), N=N, r=r, eta=ETA, seed=seed,
                               grad_dtype=case["grad"], compressor=case["compressor"],
                               **_layout_args(case))
    if case["entry"] == "model":
        s["mc"] = _model_config(case)
    return s


def run(state):
    s = state
    t = s["t"]
    s["t"] = t + 1
    if s["entry"] == "static":
        arc.arc_step_static(s["cfg"], s["stream"], t, s["grad"], s["h"], s["g"], s["idx"],
                            s["agg"])
        return {"idx": s["idx"], "agg": s["agg"], "h": s["h"], "g": s["g"]}
    if s["entry"] == "step":
        idx, agg = s["comp"].step(t, s["grad"], s["h"], s["g"])
        return {"idx": idx, "agg": agg, "h": s["h"], "g": s["g"]}
    idx, agg = s["comp"].model_step(t, s["grad"], s["h"], s["g"], s["G"], s["x"], s["mc"],
                                    s.get("m"), s.get("v"))
    out = {k: s[k] for k in ("h", "g", "G", "x", "m", "v") if k in s}
    if not s["dense"]:  # a dense iteration writes no payload
        out.update(idx=idx, agg=agg)
    return out


def work(case):
    """Bytes and operations of one pass: every input read once, every output
    written once."""
    d, N, b = _dim(case), case["N"], 2 if case["grad"] == "bf16" else 4
    K, payload = _kept(case)
    nodes = N if case["compressor"] == "topk" else 1
    if case["dense"]:
        bytes_, flops = N * d * (b + 16), N * d * 6
    else:
        # grad, h in, h out, g; Rand-K needs g at the kept rows alone
        bytes_ = N * d * (b + 8) + 4 * N * (payload if case["compressor"] == "randk" else d)
        bytes_ += 4 * N * payload + 4 * nodes * (payload + K)  # g out, agg, idx
        flops = N * d * 3 + N * payload * 3
        flops += {"arc": 2 * case["r"] * N * d + N * d, "topk": 3 * N * d, "randk": 0}[
            case["compressor"]]
    if case["entry"] == "model":
        rows = d if case["dense"] else payload
        bytes_ += 4 * d + 4 * min(d, nodes * rows)  # G in, G out
        bytes_ += {"sgd": 8, "msgd": 16, "adam": 24}[case["optimizer"]] * d
        flops += {"sgd": 4, "msgd": 6, "adam": 16}[case["optimizer"]] * d
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # The interface fixes the order and rounding of every operation
    # (include/libarctopk.h), so a correct result has these bits and no others.
    return "exact"


# ---------------------------------------------------------------- 64 bits

def _projection(seed, t, n, r):
    """V_t: SplitMix64 outputs 2c and 2c+1, c = (t*n + j)*r + k, through
    Box-Muller in binary64, rounded once to binary32 (as the definition says)."""
    with np.errstate(over="ignore"):
        c = np.arange(n * r, dtype=np.uint64) + np.uint64(t * n * r)

        def output(x):
            z = np.uint64(seed) + (x + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
            z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
            return z ^ (z >> np.uint64(31))

        w1, w2 = output(c * np.uint64(2)), output(c * np.uint64(2) + np.uint64(1))
    u1 = ((w1 >> np.uint64(11)) + np.uint64(1)).astype(np.float64) * 2.0 ** -53
    u2 = (w2 >> np.uint64(11)).astype(np.float64) * 2.0 ** -53
    z = np.sqrt(-2.0 * np.log(u1)) * np.cos(2.0 * np.pi * u2)
    return torch.from_numpy(z.astype(np.float32).reshape(n, r)).cuda().double()


def _random_keys(seed, t, m):
    with np.errstate(over="ignore"):
        x = np.arange(m, dtype=np.uint64) + np.uint64(t * m + 1)
        z = np.uint64(seed) + x * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z ^= z >> np.uint64(31)
    return torch.from_numpy((z >> np.uint64(40)).astype(np.float64)).cuda()


def _largest(keys, k):
    """The k rows of largest key, ascending, and whether 32 bits might keep
    other ones."""
    order = torch.sort(keys, descending=True, stable=True)
    near = 0 < k < keys.numel() and bool(
        order.values[k - 1] - order.values[k] <= 2e-5 * order.values[k - 1])
    return torch.sort(order.indices[:k]).values, near


def exact(case, seed):
    s = _inputs(case, seed)
    d, N, t = _dim(case), case["N"], 0 if case["dense"] else FIRST_STEP
    eta = float(np.float32(ETA))
    h = s["h"].double()
    for i in range(N):
        h[i].mul_(1.0 - eta).add_(s["grad"][i].double(), alpha=eta)
    g = s["g"].double()
    del s["grad"], s["h"], s["g"]
    G = s["G"].double() if case["entry"] == "model" else None
    out = {"h": h, "g": g}
    if case["dense"]:
        for i in range(N):
            G += h[i] - g[i]
        g.copy_(h)
    else:
        idx, agg, near = [[] for _ in range(N)], [[] for _ in range(N)], False
        nodes = N if case["compressor"] == "topk" else 1
        keys = None
        if case["compressor"] == "randk":
            keys = _random_keys(seed, t, sum(p[1] for p in _parts(case)))
        V = {}
        for row0, rows, cols, at, k in _parts(case):
            end = min(at + rows * cols, d)

            def delta(i):  # this part's rows of h - g, zero past d
                x = h[i, at:end] - g[i, at:end]
                if end < at + rows * cols:
                    x = torch.cat([x, x.new_zeros(at + rows * cols - end)])
                return x.view(rows, cols)

            if case["compressor"] == "arc":
                if cols not in V:
                    V[cols] = _projection(seed, t, cols, case["r"])
                P = sum(delta(i) @ V[cols] for i in range(N))
                found = [_largest(P.square().sum(1), k)]
            elif case["compressor"] == "randk":
                found = [_largest(keys[row0:row0 + rows], k)]
                found = [(found[0][0], False)]  # whole numbers: no rounding
            else:
                found = [_largest(delta(i).square().sum(1), k) for i in range(N)]
            near = near or any(f[1] for f in found)
            for q in range(nodes):
                rows_q = found[q][0]
                own = [q] if nodes > 1 else range(N)
                parts = {i: delta(i)[rows_q] for i in own}
                total = sum(parts.values())
                idx[q].append((rows_q + row0).int())
                agg[q].append(total.reshape(-1))
                where = (at + rows_q[:, None] * cols +
                         torch.arange(cols, device=rows_q.device)).reshape(-1)
                inside = where < d
                for i in own:
                    g[i, where[inside]] += parts[i].reshape(-1)[inside]
                if G is not None:
                    G[where[inside]] += total.reshape(-1)[inside]
        idx = [torch.cat(x) for x in idx[:nodes]]
        agg = [torch.cat(x) for x in agg[:nodes]]
        idx, agg = (torch.stack(idx), torch.stack(agg)) if nodes > 1 else (idx[0], agg[0])
        if not _views(case) and case["entry"] != "static":
            agg = agg.view(*idx.shape, case["n"])
        out.update(idx=idx, agg=None if near else agg)
    if case["entry"] == "model":
        f = lambda v: float(np.float32(v))  # noqa: E731
        x = s["x"].double()
        step = G / N
        if case["optimizer"] == "msgd":
            step += f(DECAY) * x
            step = out["m"] = f(MOMENTUM) * s["m"].double() + step
        elif case["optimizer"] == "adam":
            m = out["m"] = f(BETA1) * s["m"].double() + (1 - f(BETA1)) * step
            v = out["v"] = f(BETA2) * s["v"].double() + (1 - f(BETA2)) * step.square()
            c1, c2 = 1 - f(BETA1) ** (t + 1), 1 - f(BETA2) ** (t + 1)
            step = (m / c1) / ((v / c2).sqrt() + f(EPS))
        out.update(G=G, x=x - f(LR) * step)
    return out
