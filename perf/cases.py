"""Workloads of the relay-boundary compression library, for timing and comparing its public entry points.

Five kinds of work, each through `paper_2604_13349_amd.binding` as a program calls it, on caches resident on the GPU, with the
outputs and the workspace that such a program keeps from call to call:

  relay      one agent's hand-off: score, select, gather and back-fill one sample's cache (plain, or with a sink in right-padded
             storage, headwise or layerwise, exact directions or the Gram subspace iteration)
  batch      the same for a batch of right-padded samples with their own lengths, in one call
  merge      the cache-merging comparison system on the same caches
  transport  the outgoing message [sink; retained rows; reasoning rows], its int8 / int4 row codes, and the rows decoded again

Keys, values and queries are drawn as the benchmark's synthetic caches are: a low-rank part plus noise under a log-normal scale
per channel, a hundredth of a layer's tokens eight times as large, queries i.i.d. normal.
"""
import math

import numpy as np
import torch

from paper_2604_13349_amd import binding as B

LOWRANK, OUTLIER_FRAC, OUTLIER_SCALE = 16, 0.01, 8.0
EPS = 1e-12                  # of Eq. 4 and Eq. 6
RANK_EPS = 2.0 ** -23        # of the rank rule
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _relay(name, dtype, d, layers, heads, group, tokens, window, budget, rank, **more):
    """A relay case; budget_hi > budget: per-head budgets uniform in [budget, budget_hi]."""
    c = {"name": name, "kind": "relay", "dtype": dtype, "d": d, "layers": layers, "heads": heads, "group": group, "tokens": tokens,
         "window": window, "budget": budget, "budget_hi": budget, "rank": rank, "sink": -1, "pad": 0, "layerwise": False, "iters": 0}
    c.update(more)
    return c


def listed():
    batch = _relay("batch_short_prompts", "bf16", 128, 36, 8, 4, 340, 32, 32, 2, kind="batch", samples=12, sink=4)
    merge = _relay("cache_merging", "bf16", 128, 36, 8, 4, 2048, 32, 205, 0, kind="merge")
    transport = _relay("message_int8", "bf16", 128, 36, 8, 4, 1300, 1, 1229, 0, kind="transport", sink=4, gen=40, bits=8)
    return [
        # the smallest call: two fp32 heads of 512 tokens, budget under head_dim; launches and latency are all there is
        _relay("tiny_fp32", "f32", 64, 1, 2, 2, 512, 16, 32, 1),
        # fp32 caches at head_dim 64 with a tenth of a medium prompt kept
        _relay("fp32_prompt", "f32", 64, 12, 8, 4, 2048, 32, 205, 4),
        # the method's own setting: a few hundred prompt tokens, 32 kept, two directions, every layer of an 8B-shaped model
        _relay("short_prompt", "bf16", 128, 36, 8, 4, 256, 32, 32, 2),
        # the same with one index set per layer, four directions from three subspace iterations, a sink and right padding,
        # at an odd length
        _relay("short_prompt_layerwise", "bf16", 128, 36, 8, 4, 333, 32, 32, 4, layerwise=True, iters=3, sink=4, pad=7),
        # twelve samples of the method's own setting with lengths of 165 to 340 tokens in one call
        batch,
        # an ordinary prompt, a tenth kept: more retained rows than head_dim, the back-fill has nothing to add
        _relay("prompt_2k", "bf16", 128, 36, 8, 4, 2048, 32, 205, 4),
        # the headline workload: 8192 tokens, 15 % kept
        _relay("prompt_8k", "bf16", 128, 36, 8, 4, 8192, 32, 1229, 8),
        # the headline cache with a budget under head_dim: every head runs the whole back-fill
        _relay("prompt_8k_backfill", "bf16", 128, 36, 8, 4, 8192, 32, 96, 8),
        # a larger model and a longer prompt: five query heads per KV head, 64 window queries
        _relay("prompt_16k_group5", "bf16", 128, 40, 8, 5, 16384, 64, 3277, 8),
        # the longest prompts, with a budget per head between 10 and 20 %
        _relay("prompt_32k_ragged", "bf16", 128, 36, 8, 4, 32768, 64, 3244, 16, budget_hi=6619),
        # the comparison system on an ordinary prompt
        merge,
        # what leaves after an 8192-token prompt: the message, its int8 codes, and the receiver's rows
        transport,
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["short", "short", "batch", "prompt", "prompt", "backfill", "long", "fp32", "half_dim", "merge", "transport"])
    if kind in ("short", "batch"):
        n = rng.randint(70, 700)
        c = _relay("", "bf16", 128, rng.randint(4, 40), rng.choice([2, 4, 8]), rng.choice([1, 2, 4]), n, 32, rng.randint(16, 64), rng.randint(1, 8),
                   sink=rng.choice([-1, 0, 4]), layerwise=rng.random() < 0.4, iters=rng.choice([0, 0, 3]))
        if kind == "batch":
            c.update(kind="batch", samples=rng.randint(2, 12), tokens=min(n, 500), sink=max(0, c["sink"]), layerwise=False, iters=0)
        elif c["sink"] >= 0:
            c["pad"] = rng.randint(0, 40)
    elif kind in ("prompt", "backfill", "merge"):
        n = _log_int(rng, 700, 4000 if kind == "merge" else 9000)
        b = rng.randint(40, 120) if kind == "backfill" else max(130, int(n * rng.uniform(0.08, 0.2)))
        c = _relay("", "bf16", 128, rng.randint(4, 36), rng.choice([4, 8]), rng.choice([2, 4]), n, 32, b, rng.randint(1, 12))
        if kind == "merge":
            c.update(kind="merge", rank=0)
        else:
            c.update(sink=rng.choice([-1, -1, 4]), layerwise=rng.random() < 0.25)
    elif kind == "long":
        n = _log_int(rng, 9000, 32768)
        b = int(n * 0.099)
        c = _relay("", "bf16", 128, max(1, int(rng.uniform(0.3, 1.0) * 36 * 32768 / max(n, 24000))), 8, 4, n, rng.choice([32, 64]), b, rng.randint(4, 16),
                   budget_hi=rng.choice([b, int(n * 0.202)]))
    elif kind in ("fp32", "half_dim"):
        n = _log_int(rng, 100, 2048)
        c = _relay("", "f32" if kind == "fp32" else "bf16", rng.choice([64, 128]) if kind == "fp32" else 64, rng.randint(1, 5), rng.choice([2, 4, 8]),
                   rng.choice([1, 2, 4]), n, rng.choice([8, 16, 32]), rng.randint(10, 60), rng.randint(1, 4))
        if n > 1200 and rng.random() < 0.5:
            c["budget"] = c["budget_hi"] = n // 8
    else:
        keep = _log_int(rng, 30, 3277)
        layers = max(2, min(40, int(40 * 1229 / max(1229, keep))))
        c = _relay("", rng.choice(["bf16", "bf16", "f32"]), rng.choice([64, 128]), layers, 8, 4, keep + 71, 1, keep, 0,
                   kind="transport", sink=rng.choice([0, 4]), gen=rng.randint(0, 60), bits=rng.choice([4, 8]))
        if c["dtype"] == "f32":
            c["layers"] = max(1, layers // 2)
    c["budget"] = min(c["budget"], c["tokens"] - max(0, c["sink"]) - 1)
    c["budget_hi"] = max(c["budget"], c["budget_hi"] if c["budget_hi"] < c["tokens"] else 0)
    if c["budget_hi"] < c["budget"] + 2:
        c["budget_hi"] = c["budget"]
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ inputs
def _structured(gen, heads, n, d, outliers):
    """[heads, n, d] float32: (noise + rank-16 part) under a scale per head and channel, outlier tokens larger."""
    x = torch.randn((heads, n, d), generator=gen, device="cuda")
    f = torch.randn((heads, n, LOWRANK), generator=gen, device="cuda")
    g = torch.randn((heads, LOWRANK, d), generator=gen, device="cuda")
    x.mul_(math.sqrt(0.5)).add_(torch.matmul(f, g), alpha=math.sqrt(0.5 / LOWRANK))
    x.mul_(torch.exp(0.5 * torch.randn((heads, 1, d), generator=gen, device="cuda")))
    if outliers.numel():
        x[:, outliers] *= OUTLIER_SCALE
    return x


def _cache(case, seed, tokens):
    """K, V [layers, heads, stride, d] and the window queries [layers, heads * group, window, d]; rows past `tokens` are padding."""
    L, H, d, stride = case["layers"], case["heads"], case["d"], tokens + case["pad"]
    dt = DTYPES[case["dtype"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    K = torch.zeros((L, H, stride, d), dtype=dt, device="cuda")
    V = torch.zeros_like(K)
    for l in range(L):
        out = torch.randperm(tokens, generator=gen, device="cuda")[: int(round(OUTLIER_FRAC * tokens))]
        K[l, :, :tokens] = _structured(gen, H, tokens, d, out)
        V[l, :, :tokens] = _structured(gen, H, tokens, d, out)
    Q = torch.randn((L, H * case["group"], case["window"], d), generator=gen, device="cuda").to(dt)
    return K, V, Q


def _lengths(case):
    """Real tokens of the samples of a batch: spread between a half and the whole of the longest."""
    n, s = case["tokens"], case["samples"]
    return [n - (i * 5 % s) * ((n + 1) // 2) // s for i in range(s)]


def _budgets(case, seed):
    if case["budget_hi"] == case["budget"]:
        return None
    r = np.random.RandomState(seed & 0x7FFFFFFF)
    return r.randint(case["budget"], case["budget_hi"] + 1, size=case["layers"] * case["heads"]).astype(np.int32)


def prepare(case, seed):
    s = {"case": case}
    kind = case["kind"]
    if kind == "batch":
        s["lens"] = _lengths(case)
        parts = [_cache(case, seed * 64 + i, n) for i, n in enumerate(s["lens"])]
        shape = (len(parts),) + tuple(parts[0][0].shape[:2]) + (max(s["lens"]), case["d"])
        s["K"] = torch.zeros(shape, dtype=parts[0][0].dtype, device="cuda")
        s["V"] = torch.zeros_like(s["K"])
        for i, (K, V, _) in enumerate(parts):
            s["K"][i, :, :, : s["lens"][i]] = K
            s["V"][i, :, :, : s["lens"][i]] = V
        s["Q"] = torch.stack([q for _, _, q in parts])
        s["out"] = None
    elif kind == "transport":
        # what the compression of a prompt left behind: gathered rows with a length per head, and the reasoning rows
        L, H, d, keep = case["layers"], case["heads"], case["d"], case["budget"]
        s["K"], s["V"], _ = _cache(case, seed, case["tokens"])
        s["keep_K"], s["keep_V"] = (x[:, :, -keep:].contiguous() for x in (s["K"], s["V"]))
        s["gen_K"], s["gen_V"] = (x[:, :, : case["gen"]].contiguous() * 0.5 for x in (s["K"], s["V"]))
        s["n_keep"] = torch.from_numpy(np.random.RandomState(seed & 0x7FFFFFFF).randint(max(1, keep - keep // 8), keep + 1, size=L * H).astype(np.int32)).cuda()
    else:
        s["K"], s["V"], s["Q"] = _cache(case, seed, case["tokens"])
        s["budgets"] = _budgets(case, seed)
        s["variant"] = B.make_variant(subspace_iters=case["iters"]) if case["iters"] else None
        s["out"] = None
        s["ws"] = None
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "batch":
        s["out"] = B.compress_relay_batch(s["K"], s["V"], s["Q"], s["lens"], budget=case["budget"], rank=case["rank"], sink=case["sink"], out=s["out"])
        o = s["out"]
    elif kind == "merge":
        o = B.compress_relay_merge(s["K"], s["V"], s["Q"], budget=case["budget"], ws=s["ws"])
        s["ws"] = o["ws"]
    elif kind == "transport":
        d, dt, bits = case["d"], DTYPES[case["dtype"]], case["bits"]
        gen = case["gen"] > 0
        mk, mv, n = B.append_message(s["K"], s["V"], None, s["keep_K"], s["keep_V"], s["n_keep"], s["gen_K"] if gen else None, s["gen_V"] if gen else None,
                                     case["sink"] + case["budget"] + case["gen"], prev_len_all=case["sink"])
        ck, cv = B.quantize_rows(mk, bits), B.quantize_rows(mv, bits)
        return {"msg_K": mk, "msg_V": mv, "msg_len": n, "codes_K": ck, "codes_V": cv, "rows_K": B.dequantize_rows(*ck, d, dt, bits), "rows_V": B.dequantize_rows(*cv, d, dt, bits)}
    else:
        kw = {}
        if case["sink"] >= 0 or case["pad"]:
            kw = {"n_tokens": case["tokens"], "sink": max(0, case["sink"])}
        if s["budgets"] is not None:
            kw["budgets"] = s["budgets"]
        else:
            kw["budget"] = case["budget"]
        s["out"] = B.compress_relay(s["K"], s["V"], s["Q"], rank=case["rank"], max_budget=case["budget_hi"], out=s["out"], ws=s["ws"],
                                    layerwise=case["layerwise"], variant=s["variant"], **kw)
        o = s["out"]
        s["ws"] = o["ws"]
    return {k: o[k] for k in ("K_out", "V_out", "idx", "n_keep")}


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind, d, es = case["kind"], case["d"], 2 if case["dtype"] == "bf16" else 4
    heads, R = case["layers"] * case["heads"], case["group"] * case["window"]
    keep = 0.5 * (case["budget"] + case["budget_hi"])
    row = d * es
    if kind == "transport":
        rows = heads * (case["sink"] + case["gen"] + 15 * keep / 16)
        padded = heads * (case["sink"] + case["gen"] + case["budget"])
        codes = padded * (d * case["bits"] // 8 + 4)
        return {"bytes": 2 * (rows * row + padded * row + codes + padded * row), "flops": 2 * 6 * padded * d}
    lens = _lengths(case) if kind == "batch" else [case["tokens"]]
    byts = flops = 0.0
    for n in lens:
        byts += heads * (n * row + R * row + 4 * keep * row + 4 * keep + 4)
        flops += 2.0 * heads * R * n * d
        if kind == "merge":
            byts += heads * (n - keep) * row
            flops += 2.0 * heads * (n - keep) * keep * d
        elif case["rank"] > 0 and case["budget"] < d:         # the back-fill reads every value; its Gram matrix is symmetric
            byts += heads * (n - keep) * row
            flops += 1.0 * heads * n * d * d
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    if case["kind"] == "transport":
        return "exact"
    if case["dtype"] == "bf16":
        # values are rounded once to bf16: about 0.9e-3 to 1.5e-3 off the unrounded sum, 2^-8 of a value at most
        return {"rel": 5e-3, "max": 1.6e-2}
    # the offset is formed in single precision (about 2e-5 of itself) and is a small part of a value: 2.5e-8 off at the tiny case
    return {"rel": 1e-5, "max": 4e-4}


# ------------------------------------------------------------------------------------------------ the same in 64 bits
def _masses(K, Q, group):
    """Attention mass of one layer: K [H, n, d], Q [H * group, W, d] double -> [H, n]."""
    H, n, d = K.shape
    q = Q.reshape(H, -1, d)
    out = torch.empty((H, n), dtype=torch.float64, device=K.device)
    for h in range(H):
        out[h] = torch.softmax(torch.matmul(q[h], K[h].t().contiguous()) / math.sqrt(d), dim=1).sum(0)
    return out


def _top(A, b):
    return torch.sort(torch.sort(A, descending=True, stable=True)[1][:b])[0]


def _orth_rows(Y):
    rows, first = [], None
    for y in Y:
        v = y.copy()
        for _ in range(2):
            for q in rows:
                v = v - (v @ q) * q
        n = float(np.linalg.norm(v))
        first = n if first is None else first
        if first > 0 and n > 1e-5 * first:
            rows.append(v / n)
    return np.array(rows).reshape(len(rows), Y.shape[1])


def _delta(V, A, idx, rank, iters):
    """Eq. 2 - 6 for one head, from the sums that the back-fill needs (double, on the host): None where nothing is injected."""
    n, d = V.shape
    keep = torch.zeros(n, dtype=torch.bool, device=V.device)
    keep[idx] = True
    if rank <= 0 or idx.numel() == 0 or idx.numel() == n:
        return None
    Vk, Vd, w = V[idx], V[~keep], A[~keep]
    a_keep, a_del = float(A[idx].sum()), float(w.sum())
    if idx.numel() > d:
        s2 = np.linalg.eigvalsh(torch.matmul(Vk.t().contiguous(), Vk).cpu().numpy())
        if s2[0] > s2[-1] * (idx.numel() * RANK_EPS) ** 2:
            return None
    _, s, Vt = np.linalg.svd(Vk.cpu().numpy(), full_matrices=False)
    r = int((s > s[0] * max(Vk.shape) * RANK_EPS).sum())
    if r == d:
        return None
    P = np.eye(d) - Vt[:r].T @ Vt[:r]
    G = P @ torch.matmul(Vd.t().contiguous(), Vd).cpu().numpy() @ P
    G = 0.5 * (G + G.T)
    rbar = P @ (torch.mv(Vd.t().contiguous(), w).cpu().numpy() / (a_del + EPS))
    k = min(rank, d - r, n - idx.numel())
    if iters:
        i, c = np.arange(k)[:, None] + 0.5, np.arange(d)[None, :] + 0.5
        C = math.sqrt(2.0 / d) * np.cos(np.pi / d * i * c)
        for _ in range(iters):
            C = _orth_rows(C @ G)
    else:
        C = np.linalg.eigh(G)[1][:, -k:].T
    return a_del / (a_keep + EPS) * ((rbar @ C.T) @ C)


def _exact_sample(case, K, V, Q, n, budgets, rows, stride0):
    """K_out and V_out [L, H, rows, d] in double for one sample of n tokens; its first stride0 tokens are the sink."""
    L, H, d = K.shape[0], K.shape[1], K.shape[3]
    Ko = torch.zeros((L, H, rows, d), dtype=torch.float64, device="cuda")
    Vo = torch.zeros_like(Ko)
    for l in range(L):
        A = _masses(K[l, :, :n].double(), Q[l].double(), case["group"])[:, stride0:]
        shared = _top(A.sum(0), budgets[l * H]) if case["layerwise"] else None
        for h in range(H):
            k, v = K[l, h, stride0:n].double(), V[l, h, stride0:n].double()
            idx = shared if shared is not None else _top(A[h], budgets[l * H + h])
            m = idx.numel()
            Ko[l, h, :m], Vo[l, h, :m] = k[idx], v[idx]
            if case["kind"] == "merge":
                keep = torch.zeros(k.shape[0], dtype=torch.bool, device="cuda")
                keep[idx] = True
                kd, kk = k[~keep], k[idx]
                route = torch.argmax(torch.matmul(kd, (kk / kk.norm(dim=1, keepdim=True)).t().contiguous()), dim=1)
                Vo[l, h, :m].index_add_(0, route, v[~keep] * (A[h][~keep] / (A[h][idx][route] + EPS))[:, None])
            else:
                delta = _delta(v, A[h], idx, case["rank"], case["iters"])
                if delta is not None:
                    Vo[l, h, :m] += torch.from_numpy(delta).cuda()
    return Ko, Vo


def _codes(x, bits):
    """zero, scale and the decoded rows of [rows, d] double."""
    top = float(2 ** bits - 1)
    lo, hi = x.min(dim=1)[0], x.max(dim=1)[0]
    zero, scale = lo.half().double(), ((hi - lo) / top).half().double()
    q = torch.where(scale[:, None] > 0, torch.round((x - zero[:, None]) / torch.where(scale > 0, scale, torch.ones_like(scale))[:, None]).clamp(0, top), torch.zeros_like(x))
    return scale, zero, zero[:, None] + scale[:, None] * q


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind == "transport":
        d, keep, stride = case["d"], case["budget"], case["sink"] + case["budget"] + case["gen"]
        out = {}
        for t in "KV":
            rows = torch.zeros((case["layers"] * case["heads"], stride, d), dtype=torch.float64, device="cuda")
            full, kept, gen = (s[x + t].reshape(rows.shape[0], -1, d).double() for x in ("", "keep_", "gen_"))
            for h, n in enumerate(s["n_keep"].tolist()):
                rows[h, : case["sink"]] = full[h, : case["sink"]]
                rows[h, case["sink"] : case["sink"] + n] = kept[h, :n]
                rows[h, case["sink"] + n : case["sink"] + n + case["gen"]] = gen[h]
            scale, zero, back = _codes(rows.reshape(-1, d), case["bits"])
            out.update({"msg_" + t: rows, "codes_" + t: (None, scale, zero), "rows_" + t: back})
        out["msg_len"] = None
        return out
    if kind == "batch":
        rows = max(min(case["budget"], n - case["sink"]) for n in s["lens"])
        one = [case["budget"]] * (case["layers"] * case["heads"])
        parts = [_exact_sample(case, s["K"][i], s["V"][i], s["Q"][i], n, one, rows, case["sink"]) for i, n in enumerate(s["lens"])]
        Ko, Vo = (torch.stack([p[j] for p in parts]) for j in (0, 1))
    else:
        b = s["budgets"].tolist() if s["budgets"] is not None else [case["budget"]] * (case["layers"] * case["heads"])
        Ko, Vo = _exact_sample(case, s["K"], s["V"], s["Q"], case["tokens"], b, case["budget_hi"], max(0, case["sink"]))
    return {"K_out": Ko, "V_out": Vo, "idx": None, "n_keep": None}
