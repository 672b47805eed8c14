"""The calls whose speed this framework is judged by, over the range its users call it in.

A "layer" case is one scheduler step of `layers` model layers on a varlen batch, as a serving
program runs it: each layer appends the chunk's K/V to its own page pool and attends to the
cached prefix and, causally, to the chunk.  Where `plan` is true the step's work partition is
made in the pass (once for all its layers); where it is false the pass is a layer of a step
whose plan is there already.  A "swap" case moves pages between the device pools and the
pinned host pools, out and back in, as the scheduler's preemptions ask for.

Scores are drawn with a standard deviation of 1.5 after scaling, so that the softmax weighs
keys as unevenly as a trained model's does.
"""
import math
import random

import torch

import paper_2604_16395_amd as s2l

DEV = "cuda"
HEAD_DIM, PAGE = 128, 16
SCALE = HEAD_DIM ** -0.5
Q_STD = 1.5


def _layer(name, **kw):
    case = dict(what="layer", reqs=1, p_lo=0, p_hi=0, c_lo=1, c_hi=1, c_mode="uniform", page_aligned=False, lens=1,
                hq=32, hkv=8, kv="bf16", call="separate", plan=True, layers=1)
    case.update(kw)
    return dict(name=name, **case)


def listed():
    return [
        # the smallest step: a short context of a small model (8 query, 2 kv heads), where
        # launches and latency are all there is
        _layer("small_step", p_lo=256, p_hi=256, c_lo=128, c_hi=128, hq=8, hkv=2),
        # one decoding request: the per-layer call of a step that has its plan
        _layer("decode_one", p_lo=2047, p_hi=2047, plan=False),
        # a decode batch at long ragged contexts: every key of 64 requests is read for one token
        _layer("decode_batch", reqs=64, p_lo=1024, p_hi=32768, plan=False),
        # the same from an e4m3 cache and 70B-like heads, with shorter contexts, plan included
        _layer("decode_batch_fp8", reqs=24, p_lo=1, p_hi=16384, hq=64, kv="fp8", lens=2),
        # the first chunk of a streamed context (nothing cached yet), append fused
        _layer("stream_first", p_lo=0, p_hi=0, c_lo=512, c_hi=512, call="fused", page_aligned=True, layers=4),
        # a streamed context at 8192 cached tokens: a step of eight layers of an 8B model,
        # append fused
        _layer("stream_8k", p_lo=8192, p_hi=8192, c_lo=512, c_hi=512, call="fused", page_aligned=True, layers=8),
        # one GPU's share of the same at tensor parallel 2, with a ragged prefix and chunk
        _layer("ragged_tp2", p_lo=5003, p_hi=5003, c_lo=389, c_hi=389, hq=16, hkv=4, layers=4),
        # several requests' chunks in one step
        _layer("batch8", reqs=8, p_lo=0, p_hi=8192, c_lo=512, c_hi=512, lens=3),
        # a full mixed step: long and short prefixes, chunks from one token to 2048
        _layer("mixed64", reqs=64, p_lo=0, p_hi=32768, c_lo=1, c_hi=2048, c_mode="lognormal", lens=4),
        # a 128K context in an e4m3 cache with 70B-like heads
        _layer("long_fp8", p_lo=131072, p_hi=131072, c_lo=2048, c_hi=2048, hq=64, kv="fp8", plan=False),
        # one GPU's share of it at tensor parallel 8, quantised queries
        _layer("long_fp8_q8_tp8", p_lo=131072, p_hi=131072, c_lo=2048, c_hi=2048, hq=8, hkv=1, kv="fp8", call="q8"),
        # preemption: 512 scattered pages of one 8B layer to host memory and back
        dict(name="swap", what="swap", pages=512, hkv=8, kv="bf16"),
    ]


MAX_FLOPS, MAX_BYTES = 8.5e12, 4.0e9   # about the largest listed case


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.08:
        return dict(what="swap", pages=_log_int(rng, 16, 2048), hkv=rng.choice([1, 2, 4, 8]), kv=rng.choice(["bf16", "fp8"]))
    while True:
        kind = rng.choice(["decode", "stream", "batch", "mixed"])
        hq, hkv = rng.choice([(8, 2), (16, 4), (32, 8), (64, 8), (8, 1)])
        kv = rng.choice(["bf16", "bf16", "fp8"])
        kw = dict(hq=hq, hkv=hkv, kv=kv, lens=rng.randrange(1 << 20), plan=rng.random() < 0.6)
        if kind == "decode":
            hi = _log_int(rng, 64, 32768)
            kw.update(reqs=_log_int(rng, 1, 96), p_lo=rng.choice([hi, max(1, hi // 16)]), p_hi=hi, layers=rng.choice([1, 1, 4]))
        elif kind == "stream":
            p = rng.choice([0, _log_int(rng, 16, 131072), _log_int(rng, 16, 131072)])
            c = _log_int(rng, 17, 2048)
            kw.update(p_lo=p, p_hi=p, c_lo=c, c_hi=c, layers=rng.choice([1, 2, 8]))
        elif kind == "batch":
            hi = _log_int(rng, 64, 32768)
            kw.update(reqs=rng.randint(2, 16), p_lo=0, p_hi=hi, c_lo=_log_int(rng, 17, 512), c_hi=1024)
        else:
            kw.update(reqs=rng.randint(8, 64), p_lo=0, p_hi=_log_int(rng, 512, 32768), c_lo=1, c_hi=2048, c_mode="lognormal")
        if kind != "decode":
            kw["page_aligned"] = rng.random() < 0.5
            calls = ["separate", "separate", "fused"] + (["q8", "q8"] if kv == "fp8" else [])
            kw["call"] = rng.choice(calls)
        case = _layer("", **kw)
        del case["name"]
        P, C = lengths(case)
        if kw.get("call") == "q8" and max(C) * (hq // hkv) <= 16:
            continue   # the quantised-Q call takes chunks, not decode-only batches
        w = work(case)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return case


def lengths(case):
    """Prefix and chunk lengths of the requests."""
    rng = random.Random(1000003 * case["lens"] + case["reqs"])
    P, C = [], []
    for _ in range(case["reqs"]):
        p = rng.randint(case["p_lo"], case["p_hi"])
        if case["c_mode"] == "lognormal":
            c = min(case["c_hi"], max(case["c_lo"], int(rng.lognormvariate(math.log(64.0), 4.118))))
        else:
            c = rng.randint(case["c_lo"], case["c_hi"])
        P.append(p // PAGE * PAGE if case["page_aligned"] else p)
        C.append(c)
    return P, C


def work(case):
    if case["what"] == "swap":
        page = case["hkv"] * PAGE * HEAD_DIM * (1 if case["kv"] == "fp8" else 2)
        return {"bytes": 8 * case["pages"] * page, "flops": 0}   # K and V, out and in, read and written
    P, C = lengths(case)
    hq, hkv, eb = case["hq"], case["hkv"], 1 if case["kv"] == "fp8" else 2
    row = hkv * HEAD_DIM * 2                       # K and V elements of one token
    T = sum(C)
    pages = sum(P) * row * eb + T * row * (2 + eb)  # the prefix read; new rows read, their slots written
    io = T * hq * (HEAD_DIM * 4 + 4)                # Q in, O and log-sum-exp out
    pairs = sum(c * p + c * (c + 1) // 2 for p, c in zip(P, C))
    return {"bytes": case["layers"] * (pages + io), "flops": case["layers"] * 4 * HEAD_DIM * hq * pairs}


def tolerance(case):
    if case["what"] == "swap":
        return "exact"
    # bf16 probabilities and outputs: 2.3e-3 from the exact result; with e4m3 queries, whose codes
    # turn on the last bit of a scale, 4.7e-3
    if case["call"] == "q8":
        return {"rel": 0.02, "max": 0.2, "differ": 0.0}
    return {"rel": 0.01, "max": 0.1, "differ": 0.0}


def _pages(gen, n, hkv, fp8, scale):
    """A pool of pages of N(0, 1) values: bf16, or e4m3 codes of value / scale per kv head."""
    if not fp8:
        return torch.empty((n, hkv, PAGE, HEAD_DIM), dtype=torch.bfloat16, device=DEV).normal_(generator=gen)
    pool = torch.empty((n, hkv, PAGE, HEAD_DIM), dtype=torch.uint8, device=DEV)
    inv = (1.0 / scale).view(1, hkv, 1, 1)
    for i in range(0, n, 8192):
        x = torch.empty((min(8192, n - i), hkv, PAGE, HEAD_DIM), device=DEV).normal_(generator=gen)
        pool[i:i + 8192] = (x * inv).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    return pool


def _inputs(case, seed):
    """Everything a pass reads, made from the seed with plain torch."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    host = torch.Generator().manual_seed(seed)
    fp8 = case["kv"] == "fp8"
    hkv = case["hkv"]
    if case["what"] == "swap":
        n = case["pages"]
        total = 2 * n + 8
        ones = torch.ones(hkv, device=DEV) / 64
        perm = torch.randperm(total, generator=host).to(torch.int32)
        slots = torch.randperm(n, generator=host).to(torch.int32)
        return dict(k=_pages(gen, total, hkv, fp8, ones), v=_pages(gen, total, hkv, fp8, ones), scale=ones if fp8 else None,
                    out=torch.stack([perm[:n], slots], 1).contiguous(), back=torch.stack([slots, perm[n:2 * n]], 1).contiguous())
    P, C = lengths(case)
    T = sum(C)
    need = [(p + c + PAGE - 1) // PAGE for p, c in zip(P, C)]
    total = sum(need) + 8
    perm = torch.randperm(total, generator=host).to(torch.int32)
    tables = torch.zeros((len(P), max(need)), dtype=torch.int32)
    at = 0
    for r, k in enumerate(need):
        tables[r, :k] = perm[at:at + k]
        at += k
    layers = []
    for _ in range(case["layers"]):
        ks = vs = None
        if fp8:   # about max |x| / 448 of each head
            ks, vs = ((4.5 + torch.rand(hkv, generator=gen, device=DEV)) / 448 for _ in range(2))

        def rows(heads, std=1.0):
            x = torch.empty((T, heads, HEAD_DIM), device=DEV).normal_(0.0, std, generator=gen)
            return x.to(torch.bfloat16)

        layers.append(dict(k=_pages(gen, total, hkv, fp8, ks), v=_pages(gen, total, hkv, fp8, vs), ks=ks, vs=vs,
                           k_new=rows(hkv), v_new=rows(hkv), q=rows(case["hq"], Q_STD)))
    return dict(P=P, C=C, tables=tables, layers=layers)


class _State:
    pass


def prepare(case, seed):
    x = _inputs(case, seed)
    st = _State()
    st.case = case
    if case["what"] == "swap":
        st.cache = s2l.PagedKVCache(x["k"], x["v"], *((x["scale"], x["scale"]) if case["kv"] == "fp8" else ()))
        st.out, st.back = x["out"].to(DEV), x["back"].to(DEV)
        shape = (case["pages"],) + tuple(x["k"].shape[1:])
        st.host_k = torch.zeros(shape, dtype=x["k"].dtype, pin_memory=True)
        st.host_v = torch.zeros(shape, dtype=x["k"].dtype, pin_memory=True)
        return st
    hq, hkv, T = case["hq"], case["hkv"], sum(x["C"])
    st.batch = s2l.Batch(x["P"], x["C"], x["tables"].numpy(), device=DEV)
    st.ws = torch.empty(s2l.s2l_attn_workspace_bytes(st.batch, hq, hkv), dtype=torch.uint8, device=DEV)
    st.plan = None if case["plan"] else s2l.s2l_attn_plan(st.batch, hq, hkv, st.ws)
    st.layers = []
    for y in x["layers"]:
        cache = s2l.PagedKVCache(y["k"], y["v"], y["ks"], y["vs"])
        out = torch.empty((T, hq, HEAD_DIM), dtype=torch.bfloat16, device=DEV)
        lse = torch.empty((T, hq), dtype=torch.float32, device=DEV)
        st.layers.append((cache, y["k_new"], y["v_new"], y["q"], out, lse))
    return st


def run(st):
    case = st.case
    if case["what"] == "swap":
        s2l.s2l_kv_swap_out(st.cache, st.out, st.host_k, st.host_v)
        s2l.s2l_kv_swap_in(st.cache, st.back, st.host_k, st.host_v)
        return {"host_k": st.host_k, "host_v": st.host_v, "k": st.cache.k_pages, "v": st.cache.v_pages}
    hq, batch, ws = case["hq"], st.batch, st.ws
    plan = s2l.s2l_attn_plan(batch, hq, case["hkv"], ws) if case["plan"] else st.plan
    results = []
    for cache, k_new, v_new, q, out, lse in st.layers:
        if case["call"] == "fused":
            s2l.s2l_append_chunk_prefill_attn(cache, batch, k_new, v_new, q, hq, SCALE, out, lse, plan, ws)
        else:
            s2l.s2l_kv_append(cache, batch, k_new, v_new)
            attn = s2l.s2l_chunk_prefill_attn_q8 if case["call"] == "q8" else s2l.s2l_chunk_prefill_attn
            attn(cache, batch, q, hq, SCALE, out, lse, plan, ws)
        results.append({"o": out, "lse": lse, "k": cache.k_pages, "v": cache.v_pages})
    return results


def _append(pool, new, scale, case, x):
    """The pool after the chunk's rows joined it."""
    rows = new if scale is None else (new.float() * (1.0 / scale).view(1, -1, 1)).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    pool = pool.clone()
    at = 0
    for r, (p, c) in enumerate(zip(x["P"], x["C"])):
        pos = torch.arange(p, p + c)
        page = x["tables"][r].long()[pos // PAGE].to(DEV)
        pool[page, :, (pos % PAGE).to(DEV)] = rows[at:at + c]
        at += c
    return pool


def exact(case, seed):
    x = _inputs(case, seed)
    if case["what"] == "swap":
        o, b = x["out"].long(), x["back"].long()
        res = {}
        for key, pool in (("k", x["k"]), ("v", x["v"])):
            host = torch.empty((case["pages"],) + tuple(pool.shape[1:]), dtype=pool.dtype, device=DEV)
            host[o[:, 1].to(DEV)] = pool[o[:, 0].to(DEV)]
            pool[b[:, 1].to(DEV)] = host[b[:, 0].to(DEV)]
            res["host_" + key], res[key] = host.cpu(), pool
        return res
    hq, hkv = case["hq"], case["hkv"]
    G = hq // hkv
    results = []
    for y in x["layers"]:
        kp, vp = (_append(y[n], y[n + "_new"], y[n + "s"], case, x) for n in ("k", "v"))
        q = y["q"].double()
        if case["call"] == "q8":   # each (token, head) row as e4m3 codes of row / (max / 448)
            qf = y["q"].float()
            sq = qf.abs().amax(-1, keepdim=True) / 448.0
            sq = torch.where(sq > 0, sq, torch.ones_like(sq))
            q = (qf * (1.0 / sq)).clamp(-448, 448).to(torch.float8_e4m3fn).double() * sq.double()
        out = torch.empty(q.shape, dtype=torch.float64, device=DEV)
        lse = torch.empty(q.shape[:2], dtype=torch.float64, device=DEV)
        row = 0
        for r, (p, c) in enumerate(zip(x["P"], x["C"])):
            n = p + c
            pages = x["tables"][r, :(n + PAGE - 1) // PAGE].long().to(DEV)
            for g in range(hkv):
                def dense(pool, scale):
                    z = pool[pages, g].reshape(-1, HEAD_DIM)[:n]
                    return z.double() if scale is None else z.view(torch.float8_e4m3fn).double() * scale[g].double()

                kd, vd = dense(kp, y["ks"]), dense(vp, y["vs"])
                step = max(1, (1 << 27) // (n * G))
                for i in range(0, c, step):
                    j = min(c, i + step)
                    s = (q[row + i:row + j, g * G:(g + 1) * G].reshape(-1, HEAD_DIM) @ kd.t()).mul_(SCALE)
                    if p + i + 1 < n:
                        tok = torch.arange(p + i, p + j, device=DEV).repeat_interleave(G)
                        s.masked_fill_(torch.arange(n, device=DEV)[None, :] > tok[:, None], -math.inf)
                    m = s.amax(-1, keepdim=True)
                    s.sub_(m).exp_()
                    l = s.sum(-1, keepdim=True)
                    out[row + i:row + j, g * G:(g + 1) * G] = ((s @ vd) / l).view(j - i, G, HEAD_DIM)
                    lse[row + i:row + j, g * G:(g + 1) * G] = (m + l.log()).view(j - i, G)
            row += c
        results.append({"o": out, "lse": lse, "k": kp, "v": vp})
    return results
