"""Performance cases of the KV reduction pass: what a serving program has the library do.

A prefill hands over one layer's cache (or a stack of layers folded into the batch): deep layers are
evicted, shallow layers get codebooks; later the codebooks are expanded again (Eq. 14) and every
decode step merges its new tokens.  Head shapes are those of the benchmark configurations (8 KV heads
x 4 query heads, head_dim 128), lengths run from 512 to 32768 tokens.  Inputs follow the recipes of
``paper_2507_06517_amd.workloads``, drawn on the GPU: clustered keys and values, a drift along the
sequence, a share of isolated noise, a few heavy tokens, window queries near the clusters.

Programs keep plans (outputs and workspace of one shape) between calls, so ``prepare`` makes them.
"""
import math

import torch

from paper_2507_06517_amd import binding as sb

D = 128
THETA_K, THETA_V = 0.98, 0.95


def _layer(name, dtype, batch, heads, length, clusters, drift=0.0, noise=0.0, window=32, pool=7, budget=1024,
           cap=1024, mode="serial", token_major=False, group=4):
    c = dict(kind="layer", dtype=dtype, batch=batch, heads=heads, length=length, clusters=clusters, drift=drift,
             noise=noise, window=window, pool=pool, budget=budget, cap=cap, mode=mode, token_major=token_major,
             group=group)
    return dict(c, name=name) if name else c


def _evict(name, dtype, batch, heads, length, clusters, drift=0.0, noise=0.0, window=32, pool=7, budget=1024,
           taper_to=0, scores=True, token_major=False, group=4):
    c = dict(kind="evict", dtype=dtype, batch=batch, heads=heads, length=length, clusters=clusters, drift=drift,
             noise=noise, window=window, pool=pool, budget=budget, taper_to=taper_to, scores=scores,
             token_major=token_major, group=group)
    return dict(c, name=name) if name else c


def _codebook(name, dtype, batch, heads, length, clusters, drift=0.0, noise=0.0, cap=512, token_major=False):
    c = dict(kind="codebook", dtype=dtype, batch=batch, heads=heads, length=length, clusters=clusters, drift=drift,
             noise=noise, cap=cap, token_major=token_major)
    return dict(c, name=name) if name else c


def _whole_layer(name, dtype, heads, kept, group, clusters, cap):
    c = dict(kind="whole_layer", dtype=dtype, heads=heads, kept=kept, group=group, clusters=clusters, cap=cap)
    return dict(c, name=name) if name else c


def _rebuild(name, dtype, units, length, cap):
    c = dict(kind="rebuild", dtype=dtype, units=units, length=length, cap=cap)
    return dict(c, name=name) if name else c


def _decode(name, dtype, heads, new, stored, layers, fixed_scratch):
    c = dict(kind="decode", dtype=dtype, heads=heads, new=new, stored=stored, layers=layers,
             fixed_scratch=fixed_scratch)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest use of both paths, launches and latency: one head of a short fp32 prompt
        _layer("head_512_f32", "f32", 1, 1, 512, 380, noise=0.0, budget=128, cap=128),
        # an ordinary prompt: both paths on one layer of an 8B-shaped model
        _layer("layer_4k_f16", "f16", 1, 8, 4096, 64),
        # the shallow quarter and the deep three quarters of a 32-layer stack at 8k, each folded into one
        # call; the budgets of the deep layers taper
        _codebook("codebook_8k_8layers_f16", "f16", 8, 8, 8192, 64, cap=512),
        _evict("evict_8k_24layers_f16", "f16", 24, 8, 8192, 64, budget=2048, taper_to=256, scores=False),
        # an odd prompt length from a cache kept token-major [batch, length, heads, d], both calls overlapped
        _layer("ragged_11k_bf16", "bf16", 1, 8, 11003, 150, drift=0.003, noise=0.1, budget=1100, cap=900,
               mode="overlapped", token_major=True),
        # long context: eviction of one layer, with the scores
        _evict("evict_32k_f16", "f16", 1, 8, 32768, 256, drift=0.0026, window=64, budget=2048),
        # long context, the benchmark's configuration: three layers through the layer pipeline
        _layer("pipeline_32k_f16", "f16", 1, 8, 32768, 256, drift=0.0026, window=64, budget=2048, cap=2048,
               mode="pipelined"),
        # the largest: a batch of four long prompts, half of the tokens isolated, the codebook cut at 4096
        _layer("batch4_32k_bf16", "bf16", 4, 8, 32768, 256, noise=0.5, window=64, pool=15, budget=4096, cap=4096,
               mode="overlapped"),
        # one codebook per layer over the kept rows of all query heads (grouped heads repeated)
        _whole_layer("whole_layer_32x1024_f16", "f16", 32, 1024, 4, 96, 2048),
        # expanding a long layer's K and V again before attention
        _rebuild("rebuild_32k_f16", "f16", 8, 32768, 2048),
        # a decode step: one new token per head, K and V of eight codebook layers, no allocation allowed
        _decode("decode_step_8layers_f16", "f16", 8, 1, 1650, 8, True),
        # a turn's worth of later tokens merged at once into one layer's codebooks
        _decode("decode_256_f16", "f16", 8, 256, 1650, 1, False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng):
    """Sizes of a prefill call, at most the work of a batch of four 32k prompts."""
    length = _log_int(rng, 512, 32768)
    heads = rng.choice([1, 2, 4, 8, 8, 8])
    room = 3.0 * 32768.0 ** 2 / float(length) ** 2
    room = min(room, 3.0 * 32768.0 / length, 32.0)
    batch = _log_int(rng, 1, max(1.0, room * 8 / heads)) if rng.random() < 0.5 else 1
    dtype = rng.choice(["f16", "f16", "bf16", "bf16", "f32"])
    recipe = rng.choice(["plain", "drift", "noise"])
    clusters = max(8, min(length // 8, _log_int(rng, 48, 400)))
    if dtype == "f32":
        batch = max(1, batch // 2)
    return dict(dtype=dtype, batch=min(batch, 24), heads=heads, length=length, clusters=clusters,
                drift=0.0026 * math.sqrt(32768.0 / length) if recipe == "drift" else 0.0,
                noise=round(rng.uniform(0.05, 0.5), 3) if recipe == "noise" else 0.0,
                token_major=rng.random() < 0.3)


def draw(rng):
    kind = rng.choice(["layer", "layer", "evict", "codebook", "codebook", "whole_layer", "rebuild", "decode"])
    if kind == "rebuild":
        length = _log_int(rng, 512, 32768)
        return _rebuild(None, rng.choice(["f16", "bf16", "f32"]), rng.choice([1, 8, 8, 16, 32]), length,
                        _log_int(rng, 128, 4096))
    if kind == "decode":
        new = rng.choice([1, 1, 2, 4, _log_int(rng, 5, 1024), _log_int(rng, 5, 1024)])
        return _decode(None, rng.choice(["f16", "bf16", "f32"]), rng.choice([1, 4, 8, 8, 32]), new,
                       _log_int(rng, 100, 4096), _log_int(rng, 1, 16) if new <= 4 else 1, new <= 4)
    if kind == "whole_layer":
        group = rng.choice([2, 4])
        return _whole_layer(None, rng.choice(["f16", "bf16"]), group * rng.choice([1, 4, 8]),
                            _log_int(rng, 128, 1600), group, _log_int(rng, 24, 200), _log_int(rng, 256, 4096))
    s = _shape(rng)
    if kind == "codebook":
        return _codebook(None, cap=_log_int(rng, max(64, s["length"] // 16), max(128, s["length"] // 4)), **s)
    window = rng.choice([16, 32, 32, 64])
    more = dict(window=window, pool=rng.choice([1, 7, 7, 15]), group=rng.choice([1, 4, 4]),
                budget=window + _log_int(rng, max(32, s["length"] // 32), max(64, s["length"] // 3)))
    if kind == "evict":
        return _evict(None, taper_to=window + 16 if s["batch"] > 1 and rng.random() < 0.5 else 0,
                      scores=rng.random() < 0.5, **more, **s)
    s["batch"] = min(s["batch"], 8)
    return _layer(None, cap=_log_int(rng, max(64, s["length"] // 16), max(128, s["length"] // 4)),
                  mode=rng.choice(["serial", "overlapped"]), **more, **s)


# ---------------------------------------------------------------- inputs

def _gen(seed, *more):
    g = torch.Generator(device="cuda")
    for x in more:
        seed = seed * 1000003 + x
    g.manual_seed(seed % (1 << 62))
    return g


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _pick(centres, assign):
    """centres [B, H, C, d] at assign [B, H, n] -> [B, H, n, d]"""
    B, H, C, d = centres.shape
    at = assign + (torch.arange(B * H, device="cuda") * C).view(B, H, 1)
    return centres.reshape(-1, d)[at.reshape(-1)].view(B, H, -1, d)


def _stored(x, dtype, token_major):
    """Cast to the cache type; token_major: the same tensor as a view of a [B, l, H, d] cache."""
    x = x.to(sb.torch_dtype(dtype))
    return x.transpose(1, 2).contiguous().transpose(1, 2) if token_major else x


def _cache(case, seed):
    """K, V [B, H, l, d] and the key clusters' centres: K and V share the assignment, K has 5 % heavy tokens."""
    B, H, n, C = case["batch"], case["heads"], case["length"], case["clusters"]
    g = _gen(seed, 1)
    assign = torch.randint(0, C, (B, H, n), generator=g, device="cuda")
    isolated = torch.rand((B, H, n, 1), generator=g, device="cuda") < case["noise"] if case["noise"] > 0 else None
    out, centres = [], None
    for k in range(2):
        c = _normal(g, B, H, C, D)
        centres = c if k == 0 else centres
        x = _pick(c, assign)
        x += 0.1 * _normal(g, B, H, n, D)
        if case["drift"] > 0:
            x += torch.cumsum(case["drift"] * _normal(g, B, H, n, D), dim=2)
        if k == 0:
            heavy = torch.rand((B, H, n, 1), generator=g, device="cuda") < 0.05
            x = torch.where(heavy, 4.0 * x, x)
        if isolated is not None:
            u = torch.rand(x.shape, generator=g, device="cuda")
            x = torch.where(isolated, (2.0 * u - 1.0) * math.sqrt(3.0), x)
        out.append(_stored(x, case["dtype"], case.get("token_major", False)))
        del x
    return out[0], out[1], centres


def _queries(case, seed, centres):
    """The window queries of every query head, each near a random centre of its KV head's keys."""
    B, H, C, _ = centres.shape
    g = _gen(seed, 2)
    at = torch.randint(0, C, (B, H, case["group"] * case["window"]), generator=g, device="cuda")
    q = _pick(centres, at)
    q += 0.1 * _normal(g, *q.shape)
    return q.view(B, H * case["group"], case["window"], D).to(sb.torch_dtype(case["dtype"])).contiguous()


def _plan_deep(case, K):
    budgets = None
    if case.get("taper_to"):
        B = case["batch"]
        per = [round(case["budget"] + (case["taper_to"] - case["budget"]) * i / (B - 1)) for i in range(B)]
        budgets = torch.tensor([b for b in per for _ in range(case["heads"])], dtype=torch.int32, device="cuda")
    return sb.plan_deep(K, case["group"], case["dtype"], case["window"], case["pool"], case["budget"],
                        want_scores=case.get("scores", True), budgets=budgets)


def _plan_shallow(case, K):
    return sb.plan_shallow(K, case["dtype"], THETA_K, THETA_V, case["cap"])


def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind)
    if kind in ("layer", "evict", "codebook"):
        K, V, centres = _cache(case, seed)
        s.update(K=K, V=V)
        if kind != "codebook":
            s["Q"] = _queries(case, seed, centres)
        if kind == "evict":
            s["deep"] = _plan_deep(case, K)
        elif kind == "codebook":
            s["shallow"] = _plan_shallow(case, K)
        else:
            s["mode"] = case["mode"]
            if case["mode"] == "pipelined":
                s["layers"] = [(K, V, s["Q"])]
                for i in (1, 2):
                    k, v, c = _cache(case, seed + 7919 * i)
                    s["layers"].append((k, v, _queries(case, seed + 7919 * i, c)))
                s["pipe"] = sb.PipelinedLayers(lambda: (_plan_deep(case, K), _plan_shallow(case, K)), depth=3)
            else:
                s["deep"], s["shallow"] = _plan_deep(case, K), _plan_shallow(case, K)
                if case["mode"] == "overlapped":
                    s["both"] = sb.OverlappedLayer(s["deep"], s["shallow"])
    elif kind == "whole_layer":
        # what an eviction with repeated heads leaves: the query heads of a group keep overlapping, ascending
        # choices of the same KV head's tokens, so the same row turns up under several heads
        H, kept, group = case["heads"], case["kept"], case["group"]
        pool = 2 * kept
        K, V, _ = _cache(dict(case, batch=1, heads=H // group, length=pool, drift=0.0, noise=0.2), seed)
        g = _gen(seed, 3)
        at = torch.rand((1, H, pool), generator=g, device="cuda").argsort(dim=2)[:, :, :kept].sort(dim=2).values
        at = at.unsqueeze(3).expand(1, H, kept, D)
        s.update(K=K.repeat_interleave(group, dim=1).gather(2, at).contiguous(),
                 V=V.repeat_interleave(group, dim=1).gather(2, at).contiguous(), dtype=case["dtype"], cap=case["cap"])
    elif kind == "rebuild":
        u, n, cap = case["units"], case["length"], case["cap"]
        g = _gen(seed, 4)
        s["dtype"] = case["dtype"]
        for t in ("k", "v"):
            s["C_" + t] = torch.nn.functional.normalize(_normal(g, 1, u, cap, D), dim=3).to(sb.torch_dtype(case["dtype"]))
            # few entries serve many tokens, many entries few
            r = torch.rand((1, u, n), generator=g, device="cuda")
            s["ref_" + t] = (r * r * cap).to(torch.int32).clamp_(max=cap - 1)
            s["mag_" + t] = 11.3 + 0.7 * _normal(g, 1, u, n)
    else:
        # stored codebooks of K and V per layer; three new tokens of four near a stored entry, one elsewhere
        H, m, k = case["heads"], case["new"], case["stored"]
        cap, n = k + 2 * m + 16, 2 * case["layers"]
        dt = sb.torch_dtype(case["dtype"])
        g = _gen(seed, 5)
        entries = torch.nn.functional.normalize(_normal(g, n, H, k, D), dim=3)
        at = torch.randint(0, k, (n, H, m), generator=g, device="cuda")
        near = 11.3 * _pick(entries, at) + 0.1 * _normal(g, n, H, m, D)
        few = _normal(g, n, H, max(1, m // 12), D)
        far = _pick(few, torch.randint(0, few.shape[2], (n, H, m), generator=g, device="cuda"))
        far += 0.1 * _normal(g, n, H, m, D)
        novel = torch.rand((n, H, m, 1), generator=g, device="cuda") < 0.25
        s.update(dtype=case["dtype"], fixed=case["fixed_scratch"], cap=cap, n=n,
                 X=torch.where(novel, far, near).to(dt).unsqueeze(1).contiguous(),
                 C=torch.zeros((n, 1, H, cap, D), dtype=dt, device="cuda"),
                 stored=torch.full((n, 1, H), k, dtype=torch.int32, device="cuda"))
        s["C"][:, 0, :, :k] = entries.to(dt)
        s["n_codes"] = s["stored"].clone()
        if case["fixed_scratch"]:
            s["ref"] = torch.empty((n, 1, H, m), dtype=torch.int32, device="cuda")
            s["mag"] = torch.empty((n, 1, H, m), dtype=torch.float32, device="cuda")
            s["n_found"] = torch.empty((n, 1, H), dtype=torch.int32, device="cuda")
            s["n_matched"] = torch.empty((n, 1, H), dtype=torch.int32, device="cuda")
        s["desc"] = sb.KvDesc(1, H, 1, m, D, sb._DT[case["dtype"]])
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    kind = s["kind"]
    if kind == "evict":
        return s["deep"].run(s["K"], s["V"], s["Q"])
    if kind == "codebook":
        return s["shallow"].run(s["K"], s["V"])
    if kind == "layer":
        if s["mode"] == "pipelined":
            sets = [s["pipe"].run(*x) for x in s["layers"]]
            s["pipe"].finish()
            return [((x["deep"].kept, x["deep"].K_out, x["deep"].V_out, x["deep"].scores), x["shallow"].out)
                    for x in sets]
        if s["mode"] == "overlapped":
            return s["both"].run(s["K"], s["V"], s["Q"])
        return s["deep"].run(s["K"], s["V"], s["Q"]), s["shallow"].run(s["K"], s["V"])
    if kind == "whole_layer":
        out = sb.compress_shallow_layer(s["K"], s["V"], s["dtype"], THETA_K, THETA_V, s["cap"])
        return {k: v for k, v in out.items() if k != "workspace"}
    if kind == "rebuild":
        return [sb.reconstruct(s["C_" + t], s["ref_" + t], s["mag_" + t], s["dtype"]) for t in ("k", "v")]
    # a decode step ends with longer codebooks; the counts are put back first, so that every pass extends the
    # same ones
    s["n_codes"].copy_(s["stored"])
    if s["fixed"]:
        for i in range(s["n"]):                         # K, V of layer 0, K, V of layer 1, ...
            sb.spindle_decode_merge_static(s["desc"], s["X"][i], THETA_V if i % 2 else THETA_K, s["cap"], s["C"][i],
                                           s["n_codes"][i], s["n_found"][i], s["n_matched"][i], s["ref"][i],
                                           s["mag"][i])
        return s["ref"], s["mag"], s["n_found"], s["n_matched"], s["C"], s["n_codes"]
    outs = [sb.decode_merge(s["X"][i], s["dtype"], THETA_V if i % 2 else THETA_K, s["C"][i], s["n_codes"][i])
            for i in range(s["n"])]
    return [(o["ref"], o["mag"], o["n_found"], o["n_matched"]) for o in outs], s["C"], s["n_codes"]


# ---------------------------------------------------------------- what a pass cannot do without

def _size(dtype):
    return 4 if dtype == "f32" else 2


def _evict_work(case):
    u, n, e = case["batch"] * case["heads"], case["length"], _size(case["dtype"])
    kept = (case["budget"] + case["taper_to"]) / 2 if case.get("taper_to") else case["budget"]
    kept = min(kept, n)
    # keys and queries read, kept rows of V read, kept rows of both written with their positions, scores
    nbytes = u * (n * D * e + case["group"] * case["window"] * D * e + 3 * kept * D * e + 4 * kept)
    nbytes += 4 * u * n if case.get("scores", True) else 0
    return nbytes, 2.0 * u * case["group"] * case["window"] * n * D


def _codebook_work(problems, n, cap, dtype):
    """Keys or values read, codebook, references and magnitudes written.  Products: every token against every
    entry once; comparing all pairs of tokens is one way to find the entries, not what the result needs."""
    cap = min(cap, n)
    return problems * (n * D * _size(dtype) + cap * D * _size(dtype) + 8 * n), 2.0 * problems * n * cap * D


def work(case):
    kind = case["kind"]
    if kind == "evict":
        b, f = _evict_work(case)
    elif kind == "codebook":
        b, f = _codebook_work(2 * case["batch"] * case["heads"], case["length"], case["cap"], case["dtype"])
    elif kind == "layer":
        b, f = _evict_work(case)
        b2, f2 = _codebook_work(2 * case["batch"] * case["heads"], case["length"], case["cap"], case["dtype"])
        b, f = b + b2, f + f2
        if case["mode"] == "pipelined":
            b, f = 3 * b, 3 * f
    elif kind == "whole_layer":
        b, f = _codebook_work(2, case["heads"] * case["kept"], case["cap"], case["dtype"])
    elif kind == "rebuild":
        b = 2 * case["units"] * (case["length"] * (D * _size(case["dtype"]) + 8) + case["cap"] * D * _size(case["dtype"]))
        f = 2.0 * case["units"] * case["length"] * D
    else:
        H, m, e = case["heads"], case["new"], _size(case["dtype"])
        b = 2 * case["layers"] * H * ((case["stored"] + 2 * m) * D * e + 8 * m)
        f = 2.0 * 2 * case["layers"] * H * m * case["stored"] * D
    return {"bytes": b, "flops": f}


def tolerance(case):
    """References, counts and kept positions are whole numbers that the method fixes: none may differ.  Against a
    64-bit evaluation the scores (32-bit sums over up to 256 rows of exponentials) are off by 0.4e-6 to 2e-6, at most
    8e-6 of one value; copied rows and float32 magnitudes are the same bits; a stored entry is a quotient rounded to
    the cache type, of which a few are another unit in the last place (8e-6 over a float16 codebook)."""
    rel = {"f32": 2e-6, "f16": 4e-5, "bf16": 3e-4}[case["dtype"]]
    return {"rel": rel, "max": {"f32": 1e-5, "f16": 2e-3, "bf16": 1.6e-2}[case["dtype"]], "differ": 0.0}
