"""Workloads for measuring the library's speed, through its public entry points.

Two groups of cases:

* ``run``: whole forward passes (``FusionModel.run``) of the configured
  workloads, from one image to a full batch, in both precisions;
* single steps through the kernel-level entry points (``kernels.gemm``,
  ``kernels.attention``, ``kernels.merge``, ``kernels.topk_compact``) on packed
  ragged tokens, at the sizes that the configured backbones give them.

``listed()`` names twelve of them, ``draw()`` gives more of the same ranges,
``exact()`` computes a case in 64 bits with plain torch.
"""
import math
import random

import torch

from paper_2607_02612_amd import FusionModel
from paper_2607_02612_amd import kernels
from synth import blob, configs, weights

GPU = "cuda"
CONFIDENCE = 0.15  # exit threshold of the top-k cases: about half the samples leave


# ------------------------------------------------------------------ cases --
def listed():
    return [
        # one image at a time: an interactive or on-device style request,
        # where the number of launches and the latency of each decide
        {"name": "run_deit_s_b1", "kind": "run", "config": "deit_s", "batch": 1,
         "rho": 1.0, "exits": False},
        # the fp32 path, the precision used for reference results
        {"name": "run_tiny_fp32_b8", "kind": "run", "config": "tiny", "batch": 8,
         "rho": 1.0, "exits": True},
        # the paper's Tab. I model with its own rules and heads at the batch
        # its timings are quoted on; part of the batch exits at block 8
        {"name": "run_deit_s_paper_b64", "kind": "run", "config": "deit_s_paper", "batch": 64,
         "rho": 1.0, "exits": True},
        # the headline throughput workload
        {"name": "run_deit_s_b256", "kind": "run", "config": "deit_s", "batch": 256,
         "rho": 1.0, "exits": False},
        # long sequences: 577 tokens per image
        {"name": "run_deit_s_384_b64", "kind": "run", "config": "deit_s_384", "batch": 64,
         "rho": 1.0, "exits": False},
        # the MLP's widening product with GELU for a full batch
        {"name": "gemm_fc1_gelu_bf16", "kind": "gemm", "precision": "bf16", "rows": 50432,
         "n": 1536, "k": 384, "epi": "gelu", "mapped": False},
        # the MLP's narrowing product into the residual stream for one image,
        # through a row map as inside a block after merging
        {"name": "gemm_fc2_resid_bf16_one", "kind": "gemm", "precision": "bf16", "rows": 197,
         "n": 384, "k": 1536, "epi": "resid", "mapped": True},
        # an fp32 product of a small batch, odd number of rows
        {"name": "gemm_qkv_fp32", "kind": "gemm", "precision": "fp32", "rows": 1573,
         "n": 1152, "k": 384, "epi": "store", "mapped": False},
        # attention over ragged samples of a full batch with the CLS rows that
        # pruning reads, merged tokens of several sizes
        {"name": "attention_bf16_b256", "kind": "attention", "precision": "bf16", "batch": 256,
         "tokens": 197, "heads": 6, "cls": True},
        # attention on the fp32 path
        {"name": "attention_fp32_b8", "kind": "attention", "precision": "fp32", "batch": 8,
         "tokens": 197, "heads": 6, "cls": True},
        # the bipartite merge of a ragged batch
        {"name": "merge_b64", "kind": "merge", "batch": 64, "tokens": 189, "d": 384, "r": 8},
        # exit check, top-k prune, compaction and the next LayerNorm
        {"name": "topk_compact_b256", "kind": "topk", "batch": 256, "tokens": 165, "d": 384,
         "heads": 6, "keep": 0.7, "exits": True},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# largest batch a drawn run may have, so that it costs no more than the
# largest listed run
_MAX_BATCH = {"deit_ti": 256, "deit_s": 256, "deit_b": 48, "deit_s_384": 64,
              "deit_s_paper": 192, "tiny": 512, "tiny_paper": 512}


def draw(rng):
    kind = rng.choice(["run", "run", "gemm", "gemm", "attention", "merge", "topk"])
    if kind == "run":
        config = rng.choice(["deit_ti", "deit_s", "deit_s", "deit_b", "deit_s_384",
                             "deit_s_paper", "tiny", "tiny_paper"])
        rho = rng.choice([0.5, 1.0, 1.0, 1.5])
        most = int(_MAX_BATCH[config] * min(1.0, 0.4 + 0.6 * rho))  # less merging, fewer images
        return {"kind": kind, "config": config, "batch": _logint(rng, 1, most),
                "rho": rho, "exits": rng.random() < 0.5}
    if kind == "gemm":
        d = rng.choice([192, 384, 384, 768])
        n, k, epi, mapped = rng.choice([(3 * d, d, "store", False), (d, d, "resid", True),
                                        (4 * d, d, "gelu", False), (d, 4 * d, "resid", True),
                                        (d, 4 * d, "resid", False), (1000, d, "f32", True)])
        if rng.random() < 0.3:
            return {"kind": kind, "precision": "fp32", "rows": _logint(rng, 1, 6400),
                    "n": n, "k": k, "epi": epi, "mapped": mapped}
        most = 256 if epi == "f32" else 50432 if d < 768 else 12608
        return {"kind": kind, "precision": "bf16", "rows": _logint(rng, 1, most),
                "n": n, "k": k, "epi": epi, "mapped": mapped}
    if kind == "attention":
        if rng.random() < 0.3:
            return {"kind": kind, "precision": "fp32", "batch": _logint(rng, 1, 16),
                    "tokens": rng.randint(2, 197), "heads": rng.choice([3, 6, 12]),
                    "cls": rng.random() < 0.5}
        long = rng.random() < 0.3
        return {"kind": kind, "precision": "bf16", "batch": _logint(rng, 1, 48 if long else 256),
                "tokens": rng.randint(258, 640) if long else rng.randint(2, 256),
                "heads": rng.choice([3, 6, 12]), "cls": rng.random() < 0.5}
    tokens = rng.choice([rng.randint(8, 128), rng.randint(129, 256), rng.randint(257, 577)])
    batch = _logint(rng, 1, 256 if tokens <= 256 else 64)
    d = rng.choice([192, 384, 384, 768])
    if kind == "merge":
        return {"kind": kind, "batch": batch, "tokens": tokens, "d": d,
                "r": rng.randint(0, max(1, tokens // 16))}
    return {"kind": kind, "batch": batch, "tokens": tokens, "d": d,
            "heads": rng.choice([3, 6, 12]), "keep": rng.choice([0.5, 0.7, 0.9]),
            "exits": rng.random() < 0.5}


# ----------------------------------------------------------------- inputs --
def _gen(seed, salt=0):
    g = torch.Generator(device=GPU)
    g.manual_seed(1000003 * (seed + 1) + salt)
    return g


def _images(cfg, batch, seed):
    """Sums of three low-frequency sinusoids per channel plus noise of a
    per-image strength, the distribution of synth.images drawn on the GPU."""
    g, C, S = _gen(seed), cfg["in_ch"], cfg["img"]

    def uniform(*shape):
        return torch.rand(*shape, generator=g, device=GPU)

    yy = torch.arange(S, device=GPU).view(1, 1, S, 1) / S
    xx = torch.arange(S, device=GPU).view(1, 1, 1, S) / S
    out = torch.randn(batch, C, S, S, generator=g, device=GPU) * uniform(batch, 1, 1, 1)
    for _ in range(3):
        a, fx, fy, phi = (uniform(batch, C, 1, 1) for _ in range(4))
        out += a * torch.sin(2 * math.pi * ((8 * fx - 4) * xx + (8 * fy - 4) * yy + phi))
    return out


def _config(case):
    return configs.get(case["config"])


_model = {}  # the one model a serving program would hold: {key: (model, weights)}


def _served(case):
    key = (case["config"], case["batch"])
    if key not in _model:
        _model.clear()
        cfg = _config(case)
        W = weights.make_weights(cfg, affine="random")
        _model[key] = FusionModel(blob.pack(cfg, W), case["batch"]), W
    return _model[key]


def _deltas(case, cfg):
    return [float(v) if case["exits"] else 1.0 for v in cfg["delta"]]


def _lengths(batch, tokens, seed):
    """Offsets of ragged samples, as after a few merges with per-sample
    counts: lengths from three quarters of `tokens` up to it, in an order of
    the seed (their sum is the same for every seed)."""
    n = [tokens - (i * (tokens // 4)) // max(1, batch - 1) for i in range(batch)]
    random.Random(seed).shuffle(n)
    cu = [0]
    for v in n:
        cu.append(cu[-1] + v)
    return cu


def _sizes(M, g):
    """Token sizes after merging: mostly 1, some 2 to 4."""
    u = torch.rand(M, generator=g, device=GPU)
    return 1.0 + (u > 0.7).float() + (u > 0.85).float() + (u > 0.95).float()


def _tokens(cu, d, g):
    """Hidden states with a shared direction per sample and similar
    neighbours, as residual-stream rows have."""
    M, B = cu[-1], len(cu) - 1
    lens = torch.tensor([cu[i + 1] - cu[i] for i in range(B)], device=GPU)
    x = torch.randn(M, d, generator=g, device=GPU)
    x = x + 0.7 * torch.roll(x, 1, 0) + 0.5 * torch.roll(x, 3, 0)
    x += torch.repeat_interleave(torch.randn(B, d, generator=g, device=GPU), lens, 0,
                                 output_size=M)
    return x.contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "run":
        cfg = _config(case)
        model, _ = _served(case)
        model.set_exit_thresholds(_deltas(case, cfg))
        model.set_router_strength(case["rho"])
        return {"case": case, "model": model, "images": _images(cfg, case["batch"], seed)}
    g = _gen(seed, 1)
    if kind == "gemm":
        M, N, K = case["rows"], case["n"], case["k"]
        dt = torch.bfloat16 if case["precision"] == "bf16" else torch.float32
        st = {"case": case,
              "A": torch.randn(M, K, generator=g, device=GPU).to(dt),
              "W": (torch.randn(N, K, generator=g, device=GPU) / math.sqrt(K)).to(dt),
              "bias": torch.randn(N, generator=g, device=GPU) * 0.05, "rows": None}
        phys = M
        if case["mapped"]:  # the kept rows of a stream of about 1.25 times as many
            phys = M + M // 4
            st["rows"] = torch.randperm(phys, generator=g, device=GPU)[:M].sort().values.int()
        if case["epi"] in ("store", "gelu"):
            st["out"] = torch.empty(M, N, dtype=dt, device=GPU)
        else:
            st["out"] = torch.randn(phys, N, generator=g, device=GPU)
        return st
    cu = _lengths(case["batch"], case["tokens"], seed)
    M, B = cu[-1], case["batch"]
    st = {"case": case, "cu": cu, "size": _sizes(M, g)}
    if kind == "attention":
        d = 64 * case["heads"]
        dt = torch.bfloat16 if case["precision"] == "bf16" else torch.float32
        st["qkv"] = torch.randn(M, 3 * d, generator=g, device=GPU).to(dt)
        return st
    d = case["d"]
    st["x"] = _tokens(cu, d, g)
    st["origin"] = torch.cat([torch.arange(cu[i + 1] - cu[i], device=GPU, dtype=torch.int32)
                              for i in range(B)])
    if kind == "merge":
        st["r"] = [min(case["r"], (cu[i + 1] - cu[i] - 1) // 2) for i in range(B)]
        return st
    st["scores"] = torch.softmax(
        torch.randn(B, case["heads"], case["tokens"], generator=g, device=GPU) * 1.5, -1)
    st["ln"] = (0.5 + torch.rand(d, generator=g, device=GPU),
                0.05 * torch.randn(d, generator=g, device=GPU))
    st["logits"] = torch.randn(B, 1000, generator=g, device=GPU) * 3 if case["exits"] else None
    return st


# -------------------------------------------------------------------- run --
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "run":
        logits, exit_block, counts = st["model"].run(st["images"])
        return {"logits": logits, "exit_block": exit_block, "counts": counts}
    if kind == "gemm":
        return kernels.gemm(st["A"], st["W"], st["bias"], case["epi"], st["out"], st["rows"])
    if kind == "attention":
        out, cls = kernels.attention(st["qkv"], st["size"], st["cu"], case["heads"], True,
                                     case["tokens"] if case["cls"] else None)
        return {"out": out, "cls": cls}
    if kind == "merge":
        o, dst = kernels.merge(st["x"], st["size"], st["origin"], st["cu"], st["r"],
                               case["tokens"])
        return dict(o, x=st["x"], dst=dst)
    o, logits, exit_block, ln = kernels.topk_compact(
        st["x"], st["size"], st["origin"], st["cu"], case["keep"], scores=st["scores"],
        heads=case["heads"], exit_logits=st["logits"], delta=CONFIDENCE, ln=st["ln"])
    return dict(o, logits=logits, exit_block=exit_block, ln=ln)


# ------------------------------------------------------- work and tolerance --
def _plan(cfg, rho):
    """Tokens entering each block with neutral routers and no exits."""
    T, out = cfg["N0"] + 1, []
    for b in range(1, cfg["L"] + 1):
        out.append(T)
        N = T - 1
        if b in cfg["merges"]:
            if cfg["merge_rule"] == "fraction":
                m = 1 / (1 + math.exp(-cfg["router_bias"]))
                N -= min(int(rho * m * N / 2), N // 2)
            else:
                N -= min(int(rho * cfg["r_b"][b - 1] + 0.5), N // 2)
        if b in cfg["prunes"]:
            N = int(min(1.0, max(0.0, 1 - rho * (1 - cfg["tau"]))) * N)
        T = 1 + N
    return out


def work(case):
    kind = case["kind"]
    if kind == "run":
        cfg, B = _config(case), case["batch"]
        d, C = cfg["d"], cfg["C"]
        f = 2.0 * cfg["N0"] * cfg["patch_dim"] * d + 2.0 * d * C
        live, w = 1.0, d * cfg["patch_dim"] + d * C
        for b, T in enumerate(_plan(cfg, case["rho"]), 1):
            f += live * (8.0 * T * d * d + 4.0 * T * d * cfg["mlp"] + 4.0 * T * T * d)
            w += 4 * d * d + 2 * d * cfg["mlp"]
            if case["exits"] and b in cfg["exits"]:
                live *= 0.5
        size = 2 if cfg["precision"] == "bf16" else 4
        return {"bytes": 4.0 * B * (cfg["in_ch"] * cfg["img"] ** 2 + C) + size * w,
                "flops": B * f}
    if kind == "gemm":
        M, N, K = case["rows"], case["n"], case["k"]
        e = 2 if case["precision"] == "bf16" else 4
        o = {"store": e, "gelu": e, "resid": 8, "f32": 4}[case["epi"]]
        return {"bytes": float(e * (M * K + N * K) + M * N * o), "flops": 2.0 * M * N * K}
    B = case["batch"]
    M = B * case["tokens"] * 0.875
    if kind == "attention":
        d, e = 64 * case["heads"], 2 if case["precision"] == "bf16" else 4
        return {"bytes": M * 4 * d * e, "flops": 4.0 * M * case["tokens"] * 0.875 * d}
    d = case["d"]
    if kind == "merge":
        return {"bytes": M * (4 * d + 24) + 12.0 * B * case["r"] * d,
                "flops": 0.5 * M * case["tokens"] * 0.875 * d}
    kept = case["keep"] * M
    return {"bytes": 4 * M * case["heads"] + kept * (6 * d + 24) + 8000.0 * B * case["exits"],
            "flops": 8.0 * kept * d}


def tolerance(case):
    """About four times what an equally exact implementation shows.

    Whole bf16 runs: with GELU evaluated by the erf function in place of its
    rational approximation (7e-7 apart) the logits move by 2.5e-3 to 9.5e-3,
    single values by up to 0.13, and up to 1.3 % of the token counts by one
    (near ties of the router's rounding, the matching and the pruning).  fp32
    runs: 7e-7 unless one of their near ties falls the other way, which moves
    that sample as in bf16.  Products and attention with bf16 outputs: one
    rounding step (0.8 %) in a few values; fp32 outputs: sums in another
    order, 3.5e-7 against 64 bits."""
    kind = case["kind"]
    if kind == "run":
        if _config(case)["precision"] == "bf16":
            return {"rel": 0.03, "max": 0.5, "differ": 0.01}
        return {"rel": 0.01, "max": 0.5, "differ": 0.01}
    if kind == "gemm":
        if case["precision"] == "bf16" and case["epi"] in ("store", "gelu"):
            return {"rel": 1e-3, "max": 0.01}
        return {"rel": 5e-6, "max": 1e-4}
    if kind == "attention":
        if case["precision"] == "bf16":
            return {"rel": 5e-3, "max": 0.03}
        return {"rel": 5e-6, "max": 1e-4}
    if kind == "merge":
        return {"rel": 1e-6, "max": 1e-4, "differ": 1e-3}
    return {"rel": 1e-3, "max": 0.01, "differ": 1e-3}


# ------------------------------------------------------------------ exact --
_MATRICES = ("pe_w", "qkv_w", "proj_w", "fc1_w", "fc2_w", "ew", "ew1", "ew2", "head_w")


def _ln(x, g, b):
    mu = x.mean(-1, keepdim=True)
    v = ((x - mu) ** 2).mean(-1, keepdim=True)
    return (x - mu) / torch.sqrt(v + 1e-6) * g + b


def _gelu(x):
    return 0.5 * x * (1 + torch.erf(x / math.sqrt(2)))


def _attend(qkv, size, H):
    """One sample: (rows, CLS probabilities [H, T])."""
    T, d = qkv.shape[0], qkv.shape[1] // 3
    q, k, v = (qkv[:, i * d:(i + 1) * d].reshape(T, H, -1).transpose(0, 1).contiguous()
               for i in range(3))
    S = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(d // H) + size.log()
    P = torch.softmax(S, -1)
    return torch.matmul(P, v).transpose(0, 1).reshape(T, d), P[:, 0]


def _merge_one(x, size, r):
    """Bipartite merge of r pairs of one sample: (x, size, source slots, their
    destination slots); x and size keep every row."""
    P = x[1:] / x[1:].norm(dim=1, keepdim=True).clamp_min(1e-12)
    sim = torch.matmul(P[0::2], P[1::2].t().contiguous())
    val, best = sim.max(1)
    a = torch.sort(-val, stable=True).indices[:r].sort().values
    src, dst = 1 + 2 * a, 2 + 2 * best[a]
    num, den = x * size[:, None], size.clone()
    num = num.index_add(0, dst, num[src])
    den = den.index_add(0, dst, size[src])
    hit = torch.zeros_like(size, dtype=torch.bool)
    hit[dst] = True
    return torch.where(hit[:, None], num / den[:, None], x), den, src, dst


def _top(score, k):
    """Ascending slots of the k highest scores, ties to the lower slot."""
    return torch.sort(-score, stable=True).indices[:k].sort().values


def _exact_run(case, seed):
    cfg = _config(case)
    if case["exits"] and cfg["precision"] == "bf16":
        # a confidence near its threshold sends the sample on to another head,
        # whose logits have nothing to do with the first one's
        return None
    _, W = _served(case)
    W = {k: torch.from_numpy(v).to(GPU).double() for k, v in W.items()}
    img = _images(cfg, case["batch"], seed).double()
    B, p, g = case["batch"], cfg["patch"], cfg["img"] // cfg["patch"]
    rho, L, H = case["rho"], cfg["L"], cfg["H"]
    delta = dict(zip(cfg["exits"], _deltas(case, cfg)))
    kinds = dict(zip(cfg["exits"], cfg["exit_kind"]))
    pat = img.view(B, cfg["in_ch"], g, p, g, p).permute(0, 2, 4, 1, 3, 5).reshape(B, g * g, -1)
    logits = torch.zeros(B, cfg["C"], dtype=torch.float64, device=GPU)
    for i in range(B):
        x = torch.cat([W["cls"][None], pat[i] @ W["pe_w"].t() + W["pe_b"]]) + W["pos"]
        size = torch.ones(x.shape[0], dtype=torch.float64, device=GPU)
        done = False
        for b in range(1, L + 1):
            w = {k[len("blk%d." % b):]: v for k, v in W.items() if k.startswith("blk%d." % b)}
            h, cls = _attend(_ln(x, w["ln1_g"], w["ln1_b"]) @ w["qkv_w"].t() + w["qkv_b"], size, H)
            x = x + h @ w["proj_w"].t() + w["proj_b"]
            h = _gelu(_ln(x, w["ln2_g"], w["ln2_b"]) @ w["fc1_w"].t() + w["fc1_b"])
            x = x + h @ w["fc2_w"].t() + w["fc2_b"]
            score, N = cls.mean(0), x.shape[0] - 1
            if b in cfg["merges"]:
                m = float(torch.sigmoid(w["router_w"] @ x[0] + w["router_b"][0]))
                t = rho * m * N * 0.5 if cfg["merge_rule"] == "fraction" else \
                    2.0 * rho * m * cfg["r_b"][b - 1] + 0.5
                r = min(max(int(math.floor(t)), 0), N // 2)
                if r:
                    x, size, src, dst = _merge_one(x, size, r)
                    score = score.index_add(0, dst, score[src])
                    keep = torch.ones(N + 1, dtype=torch.bool, device=GPU)
                    keep[src] = False
                    x, size, score = x[keep], size[keep], score[keep]
            if b in cfg["exits"]:
                v = x[0]
                if kinds[b] == "pool_mlp":
                    v = (size[1:, None] * x[1:]).sum(0) / size[1:].sum()
                y = _ln(v, w["eln_g"], w["eln_b"])
                lg = w["ew"] @ y + w["eb"] if kinds[b] == "linear" else \
                    w["ew2"] @ _gelu(w["ew1"] @ y + w["eb1"]) + w["eb2"]
                if delta[b] < 1 and float(torch.softmax(lg, 0).max()) >= delta[b]:
                    logits[i], done = lg, True
                    break
            if b in cfg["prunes"]:
                if cfg["prune_rule"] == "learned":
                    score = x @ w["prune_w"] + w["prune_b"][0]
                N = x.shape[0] - 1
                k = int(math.floor(min(1.0, max(0.0, 1 - rho * (1 - cfg["tau_b"][b - 1]))) * N))
                idx = torch.cat([torch.zeros(1, dtype=torch.long, device=GPU),
                                 1 + _top(score[1:], k)])
                x, size = x[idx], size[idx]
        if not done:
            logits[i] = W["head_w"] @ _ln(x[0], W["norm_g"], W["norm_b"]) + W["head_b"]
    return {"logits": logits, "exit_block": None, "counts": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "run":
        return _exact_run(case, seed)
    st = prepare(case, seed)
    if kind == "gemm":
        y = st["A"].double() @ st["W"].double().t() + st["bias"].double()
        if case["epi"] in ("store", "gelu"):
            return _gelu(y) if case["epi"] == "gelu" else y
        out = st["out"].double()
        rows = st["rows"].long() if case["mapped"] else torch.arange(case["rows"], device=GPU)
        out[rows] = out[rows] + y if case["epi"] == "resid" else y
        return out
    cu, B = st["cu"], case["batch"]
    size = st["size"].double()
    if kind == "attention":
        qkv = st["qkv"].double()
        cls = torch.full((B, case["heads"], case["tokens"]), -1.0, dtype=torch.float64, device=GPU)
        out = []
        for i in range(B):
            a, b = cu[i], cu[i + 1]
            h, c = _attend(qkv[a:b], size[a:b], case["heads"])
            out.append(h)
            cls[i, :, :b - a] = c
        return {"out": torch.cat(out), "cls": cls if case["cls"] else None}
    x = st["x"].double()
    if kind == "merge":
        packed = torch.full_like(size, -1.0)
        at = 0
        for i in range(B):
            a, b = cu[i], cu[i + 1]
            s = size[a:b]
            keep = torch.ones(b - a, dtype=torch.bool, device=GPU)
            if st["r"][i]:
                x[a:b], s, src, _ = _merge_one(x[a:b], s, st["r"][i])
                keep[src] = False
            n = int(keep.sum())
            packed[at:at + n] = s[keep]
            at += n
        return {"rows": None, "size": packed, "origin": None, "cu": None, "live": None,
                "counts": None, "x": x, "dst": None}
    packed = torch.full_like(size, -1.0)
    ln = torch.zeros_like(x)
    at = 0
    for i in range(B):
        a, b = cu[i], cu[i + 1]
        if case["exits"]:
            if float(torch.softmax(st["logits"][i].double(), 0).max()) >= CONFIDENCE:
                continue
        n = b - a - 1
        idx = 1 + _top(st["scores"][i, :, 1:b - a].double().mean(0),
                       int(math.floor(case["keep"] * n)))
        idx = torch.cat([torch.zeros(1, dtype=torch.long, device=GPU), idx]) + a
        ln[at:at + len(idx)] = _ln(x[idx], st["ln"][0].double(), st["ln"][1].double())
        packed[at:at + len(idx)] = size[idx]
        at += len(idx)
    return {"rows": None, "size": packed, "origin": None, "cu": None, "live": None,
            "counts": None, "logits": None, "exit_block": None, "ln": ln}
