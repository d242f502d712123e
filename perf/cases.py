"""The work that users of this library have it do, as measurable cases: sizes, inputs, one pass, and what to expect of it.

Every case goes through the public entry points of the package.  A case is a dict of plain values; its "op" says
which of the library's uses it stands for:

  layer    one layer of a context arrives: score it, store it compressed, load it back (small, launch-bound calls)
  store    K and V of a whole context are compressed
  load     K and V of a whole context are restored into the serving engine's pages
  kivi     per-channel asymmetric K, per-token asymmetric V (the KIVI-style codec), both directions
  drop     token dropping joined with quantization: the kept tokens are gathered and quantized, then restored to
           their own positions of a paged pool
  score    snapkv importance of every token of a context
  keys     knorm / keydiff importance of every token of a context
  select   (smoothing and) the per-head keep-set from given scores
  eval     quality-loss proxy of every candidate configuration of a context (utility table of the policy)

The shapes are those of the library's benchmark: an 8B-shaped cache (32 layers x 8 KV heads), a 70B-shaped one (80 x 8,
8 query heads per KV head), a long-context one (28 x 4, 7 query heads per KV head), head_dim 128, 16-token pages.
"""
from __future__ import annotations

import math

import torch

import paper_2512_14946_amd as kvp

D = 128
PAGE = 16
DEV = "cuda"


# ---------------------------------------------------------------------------------------------- the listed cases

def listed():
    return [
        # A chunk's layer is scored, stored and loaded back during prefill: five short calls, the library's smallest work.
        dict(name="layer_int8", op="layer", L=1, H=8, T=4096, G=4, W=32, bits=8, group=128),
        # Compression of a whole 32K-token context of an 8B-shaped model: the headline workload, first half.
        dict(name="store_int4_8b", op="store", L=32, H=8, T=32768, bits=4, group=64, asym=False),
        # ... and its restore on a cache hit, into the scattered pages of a live server: second half.
        dict(name="load_int4_8b", op="load", L=32, H=8, T=32768, bits=4, group=64, asym=False),
        # The 2-bit codec family with a zero point, K per channel and V per token; a context length nobody rounded.
        dict(name="kivi_int2_ragged", op="kivi", L=28, H=4, T=30011, bits=2, group=32),
        # Keep-set + int4 of a 70B-shaped context at keep ratio 0.3, and its restore at the original positions.
        dict(name="drop_int4_70b", op="drop", L=80, H=8, T=16384, k=4916, bits=4, group=32),
        # Importance scores of a 70B-shaped context: 64 window queries x 8 query heads per KV head.
        dict(name="score_70b", op="score", L=80, H=8, T=16384, G=8, W=64, causal=True, force_window=True),
        # Importance scores of a 128K-token context with 7 query heads per KV head (a row count that fills no power of two).
        dict(name="score_long", op="score", L=28, H=4, T=131072, G=7, W=32, causal=True, force_window=True),
        # keydiff importance of an 8B-shaped context (the paper's key-only dropping method).
        dict(name="keydiff_8b", op="keys", L=32, H=8, T=32768, method="keydiff"),
        # Smoothing and keep-sets of a 70B-shaped context: many rows of moderate length.
        dict(name="select_70b", op="select", rows=640, T=16384, k=4916, window=64, kernel=7, mode="max"),
        # Keep-sets of a 128K-token context: few long rows, keep ratio 0.1.
        dict(name="select_long", op="select", rows=112, T=131072, k=13108, window=32, kernel=0, mode="max"),
        # One context of the policy's utility sweep: 9 codecs and 4 keep levels, and dropping alone, 40 candidates.
        dict(name="eval_sweep", op="eval", L=32, H=8, T=8192, G=4, W=32, bits="16,8,4,2", groups="32,64,128",
             keeps="0.25,0.5,0.75,1.0", pv="default"),
        # Re-profiling of a short context with the matrix-core option of the same call.
        dict(name="eval_matrix_ragged", op="eval", L=8, H=4, T=5003, G=7, W=32, bits="16,8,4,2", groups="32,64,128",
             keeps="0.25,0.5,0.75,1.0", pv="matrix"),
    ]


# ---------------------------------------------------------------------------------------------- drawn cases

def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["layer", "store", "load", "kivi", "drop", "score", "score", "keys", "select", "select", "eval", "eval"])
    H = rng.choice([1, 2, 4, 8, 8, 5])
    if op == "layer":
        G = rng.choice([1, 4, 7, 8])
        return dict(op=op, L=rng.choice([1, 1, 2]), H=H, T=_log_int(rng, 200, 8192), G=G,
                    W=rng.choice([8, 16, 32]), bits=rng.choice([8, 4, 2]), group=rng.choice([32, 64, 128]))
    if op in ("store", "load", "kivi", "drop", "keys"):
        rows = 32 * 8 * 32768                       # (layer, token, head) rows of the largest listed cache
        L = _log_int(rng, 1, 80)
        T = _log_int(rng, 256, max(257, min(131072, rows // (L * H))))
        if op == "keys":
            return dict(op=op, L=L, H=H, T=T, method=rng.choice(["knorm", "keydiff"]))
        c = dict(op=op, L=L, H=H, T=T, bits=rng.choice([8, 4, 2]), group=rng.choice([32, 64, 128]))
        if op == "drop":
            c["k"] = max(1, int(math.ceil(rng.uniform(0.1, 0.9) * T)))
        elif op in ("store", "load"):
            c["asym"] = rng.random() < 0.3
        return c
    if op == "score":
        G, W = rng.choice([1, 4, 7, 8]), rng.choice([1, 16, 32, 50, 64])
        L = _log_int(rng, 1, 80)
        cells = 80 * 8 * 16384 * 512 // (L * H * max(32, G * W))
        return dict(op=op, L=L, H=H, T=_log_int(rng, 256, max(257, min(131072, cells))), G=G, W=W,
                    causal=rng.random() < 0.9, force_window=rng.random() < 0.9)
    if op == "select":
        rows = _log_int(rng, 8, 640)
        T = _log_int(rng, 512, min(131072, 112 * 131072 // rows))
        k = max(1, int(math.ceil(rng.uniform(0.05, 0.9) * T)))
        return dict(op=op, rows=rows, T=T, k=k, window=rng.choice([8, 32, 64]), kernel=rng.choice([0, 5, 7]), mode="max")
    G, W = rng.choice([1, 4, 7, 8]), rng.choice([16, 32])
    L = _log_int(rng, 1, 32)
    blocks = 32 * 8 * 8192 // (L * H * -(-G * W // 128))
    return dict(op=op, L=L, H=H, T=_log_int(rng, 300, max(301, min(16384, blocks))), G=G, W=W,
                bits=rng.choice(["16,8,4,2", "16,4", "8,4,2"]), groups=rng.choice(["32,64,128", "64"]),
                keeps=rng.choice(["0.25,0.5,0.75,1.0", "0.3,1.0", "0.5"]), pv=rng.choice(["default", "default", "matrix", "fp32"]))


# ---------------------------------------------------------------------------------------------- inputs

def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 16 + salt)
    return g


def _plane(L, T, H, seed, salt, outliers):
    """bf16 [L][T][H][128]: normal values; K has 4 fixed outlier channels per head, 8 times as large."""
    g = _gen(seed, salt)
    x = torch.empty(L, T, H, D, dtype=torch.bfloat16, device=DEV)
    mult = torch.ones(L, H, D, device=DEV)
    if outliers:
        mult.scatter_(-1, torch.rand(L, H, D, generator=g, device=DEV).argsort(dim=-1)[..., :4], 8.0)
    for l in range(L):
        x[l] = torch.randn(T, H, D, generator=g, device=DEV).mul_(mult[l])
    return x


def _queries(L, W, Hq, seed):
    return torch.randn(L, W, Hq, D, generator=_gen(seed, 3), device=DEV).to(torch.bfloat16)


def _keep_lists(L, T, H, k, seed):
    """Sorted random keep-sets int32 [L][H][k] that always hold the last tokens, as a score-based selection gives."""
    s = torch.rand(L, H, T, generator=_gen(seed, 5), device=DEV)
    s[..., max(0, T - 64):] = 2.0
    return s.topk(k, dim=-1).indices.sort(dim=-1).values.to(torch.int32).contiguous()


def _pages(L, T, H, seed, salt):
    """A paged pool of a live server: pages in random order, a few of them not this context's."""
    n = (T + PAGE - 1) // PAGE
    table = torch.randperm(n + n // 8, generator=_gen(seed, salt), device=DEV)[:n].to(torch.int32)
    pool = torch.zeros(L, n + n // 8, PAGE, H, D, dtype=torch.bfloat16, device=DEV)
    return kvp.PagedKV(pool, table, T)


def _configs(case):
    T = case["T"]
    keeps = [kvp.kvp_keep_count(float(r), T) for r in case["keeps"].split(",")]
    cfgs = []
    for b in case["bits"].split(","):
        for g in ["0"] if b == "16" else case["groups"].split(","):
            cfgs += [(int(b), int(g), k) for k in keeps]
    return cfgs


def _qplanes(c, T, n_slots=None):
    asym = c["op"] == "kivi" or bool(c.get("asym"))
    n = T if n_slots is None else n_slots
    make = lambda per_channel: kvp.alloc_qplane(c["L"], n, c["H"], D, c["bits"], c["group"], DEV, page=PAGE,  # noqa: E731
                                                asymmetric=asym, per_channel=per_channel)
    return make(c["op"] == "kivi"), make(False)


def _workspace(nbytes):
    return torch.empty(max(16, nbytes), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    c, s = case, {"case": case}
    op, L, H, T = c["op"], c.get("L"), c.get("H"), c["T"]
    if op in ("layer", "store", "load", "kivi", "drop"):
        s["K"], s["V"] = _plane(L, T, H, seed, 1, True), _plane(L, T, H, seed, 2, False)
        s["qk"], s["qv"] = _qplanes(c, T, c.get("k"))
    if op in ("layer", "load", "kivi", "drop"):
        s["pk"], s["pv"] = _pages(L, T, H, seed, 6), _pages(L, T, H, seed, 7)
    if op == "load":          # the context was stored earlier; only its compressed form is at hand
        kvp.kvp_quantize(s.pop("K"), s["qk"])
        kvp.kvp_quantize(s.pop("V"), s["qv"])
    if op == "drop":
        s["keep"] = _keep_lists(L, T, H, c["k"], seed)
    if op in ("score", "eval", "layer"):
        Hq, W = c["G"] * H, c["W"]
        s["Q"] = _queries(L, W, Hq, seed)
        s.setdefault("K", _plane(L, T, H, seed, 1, True) if op != "layer" else s.get("K"))
        if op == "eval":
            s["V"] = _plane(L, T, H, seed, 2, False)
            s["cfgs"] = _configs(c)
            n = len(s["cfgs"])
            s["loss"] = torch.zeros(n, device=DEV)
            s["partial"] = torch.zeros(L, n, 2, device=DEV)
            s["ws"] = _workspace(kvp.kvp_eval_workspace_bytes(L, H, Hq, W, T, n))
        else:
            s["scores"] = torch.zeros(L, H, T, device=DEV)
            s["ws"] = _workspace(kvp.kvp_score_workspace_bytes(L, H, Hq, W, T))
    if op == "keys":
        s["K"] = _plane(L, T, H, seed, 1, True)
        s["method"] = kvp.KVP_SCORE_KEYDIFF if c["method"] == "keydiff" else kvp.KVP_SCORE_KNORM
        s["scores"] = torch.zeros(L, H, T, device=DEV)
        s["ws"] = _workspace(kvp.kvp_score_keys_workspace_bytes(L, H, T, s["method"]))
    if op == "select":
        # summed attention of window queries is close to log-normal; the window itself is always kept
        s["scores"] = torch.randn(c["rows"], T, generator=_gen(seed, 4), device=DEV).mul_(0.6).exp_().mul_(0.01)
        s["scores"][:, T - min(c["window"], T):] = math.inf
        s["smooth"] = torch.zeros(c["rows"], T, device=DEV) if c["kernel"] else None
        s["idx"] = torch.zeros(c["rows"], c["k"], dtype=torch.int32, device=DEV)
        s["ws"] = _workspace(kvp.kvp_select_workspace_bytes(c["rows"], T, c["k"]))
    return s


# ---------------------------------------------------------------------------------------------- one pass

def _plane_out(q):
    out = {"codes": q.codes, "scales": q.scales}
    if q.mins is not None:
        out["mins"] = q.mins
    return out


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "layer":
        kvp.kvp_score_tokens(s["Q"], s["K"], s["scores"], ws=s["ws"])
    if op in ("layer", "store", "kivi", "drop"):
        kvp.kvp_quantize(s["K"], s["qk"], s.get("keep"))
        kvp.kvp_quantize(s["V"], s["qv"], s.get("keep"))
    if op in ("layer", "load", "kivi"):
        kvp.kvp_dequantize_paged(s["qk"], s["pk"])
        kvp.kvp_dequantize_paged(s["qv"], s["pv"])
    if op == "drop":
        kvp.kvp_dequantize_paged_scatter(s["qk"], s["keep"], s["pk"])
        kvp.kvp_dequantize_paged_scatter(s["qv"], s["keep"], s["pv"])
    if op == "score":
        return kvp.kvp_score_tokens(s["Q"], s["K"], s["scores"], causal=c["causal"], force_window=c["force_window"], ws=s["ws"])
    if op == "keys":
        return kvp.kvp_score_keys(s["K"], s["method"], s["scores"], ws=s["ws"])
    if op == "select":
        rows = s["scores"]
        if c["kernel"]:
            rows = kvp.kvp_smooth_scores(rows, min(c["window"], c["T"]), c["kernel"], c["mode"], out=s["smooth"])
        idx = kvp.kvp_select_topk(rows, c["k"], s["idx"], ws=s["ws"])
        return {"idx": idx, "smooth": s["smooth"]} if c["kernel"] else {"idx": idx}
    if op == "eval":
        loss, partial = kvp.kvp_eval_configs(s["Q"], s["K"], s["V"], s["cfgs"], s["loss"], s["partial"], ws=s["ws"],
                                             pv_matrix_cores=c["pv"] == "matrix", pv_fp32=c["pv"] == "fp32")
        return {"loss": loss, "partial": partial}
    out = {}
    if op != "load":
        out.update(k=_plane_out(s["qk"]), v=_plane_out(s["qv"]))
    if "pk" in s:
        out.update(pool_k=s["pk"].pool, pool_v=s["pv"].pool)
    if op == "layer":
        out["scores"] = s["scores"]
    return out


# ---------------------------------------------------------------------------------------------- what a pass needs

def _qplane_bytes(c, n, per_channel, asym):
    elems = c["L"] * n * c["H"] * D
    return elems * c["bits"] / 8 + elems / c["group"] * (8 if asym else 4)


def work(case):
    c, op, T = case, case["op"], case["T"]
    if op == "select":
        one = 4.0 * c["rows"] * T
        return {"bytes": one + 4.0 * c["rows"] * c["k"] + (one if c["kernel"] else 0.0), "flops": 0.0}
    L, H = c["L"], c["H"]
    plane = 2.0 * L * T * H * D
    if op == "keys":
        return {"bytes": plane + 4.0 * L * T * H, "flops": (2.0 if c["method"] == "knorm" else 6.0) * L * T * H * D}
    if op == "score":
        M = c["G"] * c["W"]
        return {"bytes": plane + 2.0 * L * H * M * D + 4.0 * L * T * H, "flops": 2.0 * L * H * M * T * D}
    if op == "eval":
        M, cfgs = c["G"] * c["W"], _configs(c)
        most = {}
        for b, g, k in cfgs:
            most[(b, g)] = max(k, most.get((b, g), 0))
        most[(16, 0)] = T                       # the uncompressed outputs every candidate is compared with
        return {"bytes": 2 * plane + 2.0 * L * H * M * D + 4.0 * len(cfgs) * (1 + 2 * L),
                "flops": 4.0 * L * H * M * D * sum(most.values())}
    asym = op == "kivi" or bool(c.get("asym"))
    n = c.get("k", T)
    q = _qplane_bytes(c, n, op == "kivi", asym) + _qplane_bytes(c, n, False, asym)
    rows = 2 * 2.0 * L * n * H * D              # K and V rows in bf16, as read or as written
    if op in ("store", "load"):
        return {"bytes": rows + q, "flops": 0.0}
    total = 2 * rows + 2 * q
    flops = 0.0
    if op == "drop":
        total += 4 * 4.0 * L * H * n
    if op == "layer":
        M = c["G"] * c["W"]
        total += plane + 2.0 * L * H * M * D + 4.0 * L * T * H
        flops = 2.0 * L * H * M * T * D
    return {"bytes": total, "flops": flops}


# ---------------------------------------------------------------------------------------------- tolerances

def tolerance(case):
    op = case["op"]
    # Codes, scales, minima, restored bf16 values and keep-sets have one right answer, bit for bit.
    if op in ("store", "load", "kivi", "drop", "select"):
        return "exact"
    # Each figure is about four times what the path was seen to differ from 64-bit results over listed and drawn cases.
    # Scores: logits of a few tens in 32 bits, exponentials, sums over up to 512 rows and 131072 keys (5e-7 seen).
    if op in ("score", "layer"):
        return {"rel": 2e-6, "max": 5e-5}
    # Key norms: one 32-bit sum of 128 squares (4e-8 seen).  keydiff: a mean over all keys is taken from a sum of
    # cosines near its own size, so the 32-bit error of that sum counts (3e-7 seen).
    if op == "keys":
        return {"rel": 2e-7, "max": 2e-6} if case["method"] == "knorm" else {"rel": 2e-6, "max": 5e-5}
    # Losses and their per-layer sums, differences of nearly equal outputs: the default form rounds probabilities to
    # 16 bits (4e-6 seen), the other two do not (1e-7 seen; a token at the edge of a keep-set may change sides).
    return {"rel": 2e-5, "max": 2e-4} if case["pv"] == "default" else {"rel": 2e-6, "max": 5e-5}


# ---------------------------------------------------------------------------------------------- 64-bit results

def _exact_plane(q, x, keep):
    """Scales (and minima) of the groups of x in 64 bits."""
    if keep is not None:
        x = torch.gather(x, 1, keep.permute(0, 2, 1).long()[..., None].expand(-1, -1, -1, D))
    L, T, H, _ = x.shape
    g, Tp = q.group, q.codes.shape[1]
    sc = torch.zeros(q.scales.shape, dtype=torch.float64, device=DEV)
    mn = torch.zeros_like(sc) if q.mins is not None else None
    levels = 2 ** q.bits - 1 if mn is not None else 2 ** (q.bits - 1) - 1
    for l in range(L):
        y = x[l].double()
        if q.group_axis:
            for lo in range(0, T, g):
                part = y[lo:lo + g]
                hi_, lo_ = part.amax(0), part.amin(0)
                sc[l, lo // g] = (hi_ - lo_) / levels if mn is not None else part.abs().amax(0) / levels
                if mn is not None:
                    mn[l, lo // g] = lo_
        else:
            part = y.view(T, H, D // g, g)
            hi_, lo_ = part.amax(-1), part.amin(-1)
            sc[l, :T] = (hi_ - lo_) / levels if mn is not None else part.abs().amax(-1) / levels
            if mn is not None:
                mn[l, :T] = lo_
    out = {"codes": None, "scales": sc}
    if mn is not None:
        out["mins"] = mn
    return out


def _exact_pool(q, paged, keep):
    """The restored plane in 64 bits (before rounding to bf16), from the stored codes, scales and minima."""
    L, Tp, H, cb = q.codes.shape
    n = q.T
    pool = torch.zeros(paged.pool.shape, dtype=torch.float64, device=DEV)
    per = 8 // q.bits
    for l in range(L):
        b = q.codes[l, :n].to(torch.int32)
        f = torch.stack([(b >> (q.bits * i)) & (2 ** q.bits - 1) for i in range(per)], dim=-1).reshape(n, H, D)
        if q.mins is None:
            f = torch.where(f >= 2 ** (q.bits - 1), f - 2 ** q.bits, f)
        def spread(p):
            if q.group_axis:
                return p[l].double().repeat_interleave(q.group, 0)[:n]
            return p[l, :n].double().repeat_interleave(q.group, -1)
        v = f.double() * spread(q.scales)
        if q.mins is not None:
            v = v + spread(q.mins)
        if keep is None:
            t = torch.arange(n, device=DEV)
            pool[l, paged.block_table[t // PAGE].long(), t % PAGE] = v
        else:
            t = keep[l].long().t()                                   # [k][H]
            h = torch.arange(H, device=DEV).expand_as(t)
            pool[l, paged.block_table[t // PAGE].long(), t % PAGE, h] = v
    return pool


def _exact_scores(Q, K, causal, force_window):
    L, T, H, _ = K.shape
    W, Hq = Q.shape[1:3]
    G = Hq // H
    pos = torch.arange(T - W, T, device=DEV)
    masked = torch.arange(T, device=DEV)[None, :] > pos[:, None]     # [W][T]
    out = torch.empty(L, H, T, dtype=torch.float64, device=DEV)
    for l in range(L):
        for h in range(H):
            q = Q[l, :, h * G:(h + 1) * G].double().transpose(0, 1).reshape(G * W, D)
            s = (q @ K[l, :, h].double().t().contiguous()) / math.sqrt(D)
            if causal:
                s = s.view(G, W, T).masked_fill(masked, -math.inf).view(G * W, T)
            out[l, h] = torch.softmax(s, dim=-1).sum(0)
    if force_window:
        out[..., T - W:] = math.inf
    return out


def _exact_codec(x, bits, group):
    """bf16 rows through the symmetric quantizer and back, as fp64 holding the bf16 values a decode would read."""
    if bits == 16:
        return x.double()
    qmax = 2 ** (bits - 1) - 1
    f = x.float().view(*x.shape[:-1], D // group, group)
    amax = f.abs().amax(-1, keepdim=True)
    scale = amax / torch.full_like(amax, float(qmax))   # a Python number as divisor becomes a product with its reciprocal
    q = torch.where(scale > 0, torch.round(f / torch.where(scale > 0, scale, 1.0)), 0.0).clamp(-qmax, qmax)
    return (q * scale).view(x.shape).to(torch.bfloat16).double()


def _exact_eval(c, s):
    Q, K, V, cfgs = s["Q"], s["K"], s["V"], s["cfgs"]
    L, T, H, _ = K.shape
    G, W = c["G"], c["W"]
    levels = sorted({k for _, _, k in cfgs})
    rank = torch.empty(H, T, dtype=torch.int64, device=DEV)
    masked = (torch.arange(T, device=DEV)[None, :] > torch.arange(T - W, T, device=DEV)[:, None]).repeat(G, 1)  # [G*W][T]
    partial = torch.zeros(L, len(cfgs), 2, dtype=torch.float64, device=DEV)
    for l in range(L):
        order = torch.sort(_exact_scores(Q[l:l + 1], K[l:l + 1], True, True)[0], dim=-1, descending=True, stable=True).indices
        rank.scatter_(1, order, torch.arange(T, device=DEV).expand(H, T))
        q = Q[l].double().view(W, H, G, D).permute(1, 2, 0, 3).reshape(H, G * W, D)

        def outputs(bits, group, keeps):
            k, v = (_exact_codec(x[l].transpose(0, 1).contiguous(), bits, group) for x in (K, V))
            e = torch.matmul(q, k.transpose(1, 2).contiguous()).div_(math.sqrt(D)).masked_fill_(masked, -math.inf)
            for keep in keeps:
                p = torch.softmax(e.masked_fill((rank >= keep)[:, None, :], -math.inf), dim=-1)
                yield keep, torch.matmul(p, v)
        full = dict(outputs(16, 0, [T]))[T]
        for b, g in sorted({(b, g) for b, g, _ in cfgs}):
            for keep, o in outputs(b, g, levels):
                num = (o - full).square().sum()
                for i, cf in enumerate(cfgs):
                    if cf == (b, g, keep):
                        partial[l, i, 0], partial[l, i, 1] = num, full.square().sum()
    total = partial.sum(0)
    return {"loss": (total[:, 0] / total[:, 1]).sqrt(), "partial": partial}


def exact(case, seed):
    c, op = case, case["op"]
    s = prepare(case, seed)
    if op == "score":
        return _exact_scores(s["Q"], s["K"], c["causal"], c["force_window"])
    if op == "keys":
        K, out = s["K"], s["scores"].double()
        for l in range(c["L"]):
            x = K[l].double().transpose(0, 1)                        # [H][T][D]
            n = x.norm(dim=-1)
            if c["method"] == "knorm":
                out[l] = n
            else:
                u = x / n.clamp_min(1e-300)[..., None]
                out[l] = -((u * u.sum(1, keepdim=True)).sum(-1) - 1.0) / max(1, c["T"] - 1)
        return out
    if op == "select":
        if not c["kernel"]:
            return None                                              # whole numbers only
        P, r = c["T"] - min(c["window"], c["T"]), c["kernel"] // 2
        sm = s["scores"].double()
        if P > 0:
            pad = torch.nn.functional.pad(sm[:, :P], (r, r), value=-math.inf)
            sm = torch.cat([pad.unfold(1, c["kernel"], 1).amax(-1), sm[:, P:]], dim=1)
        return {"idx": None, "smooth": sm}
    if op == "eval":
        return _exact_eval(c, s)
    keep, out = s.get("keep"), {}
    if op != "load":
        out.update(k=_exact_plane(s["qk"], s["K"], keep), v=_exact_plane(s["qv"], s["V"], keep))
    if "pk" in s:
        if op != "load":
            run(s)                                                   # the codes that are restored are whole numbers
        out.update(pool_k=_exact_pool(s["qk"], s["pk"], keep), pool_v=_exact_pool(s["qv"], s["pv"], keep))
    if op == "layer":
        out["scores"] = _exact_scores(s["Q"], s["K"], True, True)
    return out
