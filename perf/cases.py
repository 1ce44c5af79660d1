"""The work that users of this library have it do, as cases that can be timed and checked.

A case is one of six kinds, each a sequence of public calls as a serving program makes them for one
attention layer:

  step     the decode step of one generated token: the token's key joins the codes, the queries are
           coded, the attention scans the codes of the whole context
  tables   the same step with the sample retrieved from hash tables built some tokens earlier
  rebuild  the tables are built anew and a step goes through them
  prefill  the key mean and the codes of a whole cache
  chunk    the codes of a chunk of keys appended behind a frozen mean (a further turn of a conversation)
  prompt   a short prompt from its cache to the first output: key mean, codes, attention

Inputs are drawn on the GPU with the geometry of paper_2410_16179_amd/workloads.py: the keys of a KV
head share a large offset, queries lie along a sum of planted keys plus noise.
"""
from __future__ import annotations

import math

import torch

from paper_2410_16179_amd import binding as mp

D = 128
SINK, LOCAL = 4, 64

_DEFAULT = {"batch": 1, "q_heads": 32, "kv_heads": 8, "K": 10, "L": 150, "dtype": "bf16", "kv": "", "min_hits": 2,
            "planted": 32, "spare": 0, "layout": "head", "live": False, "projector": "prepared", "appended": 0,
            "first": 0, "keys": 0}


def _case(name, kind, n, **more):
    c = {"name": name, "kind": kind, "n": n}
    c.update({k: v for k, v in more.items() if _DEFAULT[k] != v})
    return c


def _full(case):
    return {**_DEFAULT, **case}


def listed():
    return [
        # a short conversation, one user: nothing but latency and launches
        _case("step_2k", "step", 2048),
        # 16k tokens, one user (workload C2)
        _case("step_16k", "step", 16384),
        # the paper's 96k tokens, one user (C3, the benchmark's workload), with room for the tokens to come
        _case("step_96k", "step", 98304, spare=2048),
        # the same through hash tables built up to 2048 tokens earlier
        _case("step_96k_tables", "tables", 98304, appended=1984, spare=2048),
        # a serving batch of 64k contexts, peaked and flat heads (C4)
        _case("step_b16_64k", "step", 65536, batch=16, K=9, L=120, planted=512),
        # a batch of 128k contexts, eight query heads per KV head, through tables (C5)
        _case("step_b8_128k_tables", "tables", 131072, batch=8, q_heads=64, K=10, L=170, appended=512, spare=512),
        # a quantised cache stored token by token, ragged length kept in device memory, odd group of heads
        _case("step_fp8_ragged", "step", 50003, batch=3, q_heads=40, K=10, L=220, kv="fp8", layout="token", live=True,
              spare=1024),
        # every head with keys of its own (no grouping), a table set of the paper's study that is not a
        # configuration of its own
        _case("step_mha", "step", 20011, q_heads=32, kv_heads=32, K=9, L=110),
        # float32 from end to end (C1): a prompt of 4096 tokens and the first step behind it
        _case("prompt_fp32", "prompt", 4096, q_heads=1, kv_heads=1, K=8, L=75, dtype="fp32", planted=16,
              projector="plain"),
        # the codes of a 96k cache (C3), once per conversation
        _case("prefill_96k", "prefill", 98304),
        # four conversations of 32k tokens get 4099 more each, quantised cache
        _case("chunk_fp8", "chunk", 36867, batch=4, first=32768, keys=4099, K=9, L=120, kv="fp8"),
        # new hash tables over 96k tokens and the first step through them
        _case("rebuild_96k", "rebuild", 98304, spare=2048),
    ]


# (K, L) of the paper's tables: its accuracy and system tables, and the sampled fractions of at most
# a few per cent from its study of table shapes
_TABLES = [(10, 150), (10, 150), (9, 120), (10, 170), (8, 75), (10, 220), (11, 300), (9, 110), (8, 90), (10, 300), (9, 75),
           (9, 100), (10, 100), (10, 120), (10, 200), (11, 150), (11, 200)]
_HEADS = [(32, 8), (32, 8), (64, 8), (40, 8), (28, 4), (16, 2), (8, 1), (24, 8), (8, 8), (32, 32)]


def _between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "tables", "tables", "prefill", "chunk", "prompt", "rebuild"])
    hq, hkv = rng.choice(_HEADS)
    K, L = rng.choice(_TABLES)
    dtype, kv = rng.choice([("bf16", ""), ("bf16", ""), ("bf16", ""), ("bf16", "fp8"), ("fp32", "")])
    c = {"q_heads": hq, "kv_heads": hkv, "K": K, "L": L, "dtype": dtype, "kv": kv,
         "min_hits": rng.choice([2, 2, 2, 2, 1, 3]), "planted": rng.choice([8, 32, 32, 512]),
         "layout": rng.choice(["head", "head", "token"])}
    most = {"step": 4 << 20, "tables": 4 << 20, "prefill": 3 << 18, "chunk": 3 << 18, "prompt": 1 << 16,
            "rebuild": 1 << 19}[kind]                        # keys over all heads
    if dtype == "fp32":
        most = min(most, {"prefill": 1 << 14, "chunk": 1 << 14, "prompt": 1 << 14}.get(kind, 1 << 21))
    most = most * 1500 // max(1500, K * L)
    c["batch"] = b = rng.choice([x for x in (1, 1, 1, 2, 3, 4, 8, 16) if x == 1 or (x * hkv <= 128 and x * hkv * 512 <= most)])
    top = min(131072, most // (b * hkv))
    n = _between(rng, min(1024, top // 2), top)
    while work({**c, "kind": kind, "n": n})["bytes"] > 1.5e9:  # (low thresholds sample many rows)
        n //= 2
    if rng.random() < 0.3:
        n -= n % 64
    if kind in ("step", "tables"):
        c["spare"] = rng.choice([0, 0, 256, 2048])
        c["live"] = rng.random() < 0.3
        c["projector"] = rng.choice(["prepared", "prepared", "plain"])
    if kind == "tables":
        c["appended"] = rng.randint(0, min(2048, n // 2))
    if kind in ("tables", "rebuild"):
        c["min_hits"] = rng.choice([2, 2, 2, 1])
    if kind == "chunk":
        c["first"] = rng.randint(0, n // 2)
        c["keys"] = n - c["first"]
    if kind == "prompt":
        c["projector"] = "plain"
    got = _case("", kind, n, **c)
    del got["name"]
    return got


# ---- inputs ------------------------------------------------------------------------------------------
def _store(x, kind):
    if kind == "bf16":
        return x.to(torch.bfloat16)
    if kind == "fp8":
        return x.clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return x


def _inputs(c, seed):
    """K, V [B, Hkv, cap, 128] (views, in the case's layout), q, W, mu (float32, of the frozen mean) and the capacity."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 31) + 17)
    B, Hq, Hkv, n, cap = c["batch"], c["q_heads"], c["kv_heads"], c["n"], c["n"] + c["spare"]
    G = Hq // Hkv
    kind = c["kv"] or c["dtype"]
    at = {"bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn, "fp32": torch.float32}[kind]

    def cache():
        if c["layout"] == "token":
            return torch.empty(B, cap, Hkv, D, dtype=at, device="cuda").permute(0, 2, 1, 3)
        return torch.empty(B, Hkv, cap, D, dtype=at, device="cuda")

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda")

    W = _store(normal(D, c["K"] * c["L"]), c["dtype"])
    Kc, Vc = cache(), cache()
    mu = torch.empty(B, Hkv, D, device="cuda")
    q = torch.empty(B, Hq, D, device="cuda")
    frozen = c["first"] or n                                  # keys that the centering vector was taken from
    P = min(c["planted"], n - SINK - LOCAL)
    for b in range(B):
        for h in range(Hkv):
            k = _store(2.0 * normal(D) + normal(cap, D), kind)
            Kc[b, h] = k
            Vc[b, h] = _store(normal(cap, D), kind)
            mu[b, h] = k[:frozen].double().mean(0)
            pick = torch.randint(SINK, n - LOCAL, (G, P), generator=g, device="cuda")
            s = k.to(torch.float32)[pick].sum(1)
            q[b, h * G:(h + 1) * G] = 0.8 * s / s.norm(dim=1, keepdim=True) + 0.5 * normal(G, D)
    return Kc, Vc, _store(q, c["dtype"]), W, mu, cap


def prepare(case, seed):
    c = _full(case)
    Kc, Vc, q, W, mu, cap = _inputs(c, seed)
    B, Hq, Hkv, n, kind = c["batch"], c["q_heads"], c["kv_heads"], c["n"], c["kind"]
    s = {"kind": kind, "q": q, "W": W, "K": Kc, "V": Vc, "mu": mu, "n": n, "projector": c["projector"]}
    same = dict(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, K=c["K"], L=c["L"], n_cap=cap, dtype=c["dtype"], min_hits=c["min_hits"],
                n_sink=SINK, n_local=LOCAL, k_strides=Kc.stride()[:3], v_strides=Vc.stride()[:3], kv_dtype=c["kv"])
    if c["live"]:                                             # the length of the running conversation, the bound its capacity
        s["n_dev"] = torch.tensor([n], dtype=torch.int64, device="cuda")
        p = mp.make_params(n_ctx=cap, n_ctx_dev=s["n_dev"], **same)
    else:
        p = mp.make_params(n_ctx=n, **same)
    s["params"] = p
    s["key_codes"] = mp.alloc_key_codes(p)
    s["ws"] = mp.alloc_workspace(p)
    if kind in ("prefill", "prompt"):
        s["mu"] = torch.empty_like(mu)
    elif kind == "chunk":
        s["first"], s["keys"] = c["first"], c["keys"]
    else:
        mp.magicpig_hash_keys(p, Kc, mu, W, 0, n, s["key_codes"], s["ws"])
        if c["projector"] == "prepared":
            s["prepared"] = mp.alloc_prepared_projector(p)
            mp.magicpig_prepare_projector(p, W, s["prepared"])
            s["centering"] = mp.alloc_centering(p)
            mp.magicpig_prepare_centering(p, mu, s["prepared"], s["centering"])
    if kind not in ("prefill", "chunk"):
        s["q_codes"] = mp.alloc_query_codes(p)
        s["out"] = torch.empty(B, Hq, D, device="cuda")
    if kind in ("tables", "rebuild"):
        s["indexed"] = n - c["appended"] if c["appended"] == 0 else (n - c["appended"]) // 64 * 64
        if c["live"]:
            s["indexed"] = s["indexed"] // 64 * 64
        s["tables"] = mp.alloc_tables(p)
        s["build"] = mp.make_params(n_ctx=s["indexed"], **same)
        s["build_ws"] = mp.alloc_table_build_workspace(s["build"])
        s["offsets"] = s["tables"][256:256 + B * Hkv * c["L"] * (2 ** c["K"] + 1) * 4].view(torch.int32)
        if kind == "tables":
            mp.magicpig_build_tables(s["build"], s["key_codes"], s["tables"], s["build_ws"])
            s["build_ws"] = None
    return s


# ---- the calls ---------------------------------------------------------------------------------------
def _step_codes(s):
    """The newest key of every KV head joins the codes, the queries are coded."""
    p, n = s["params"], s["n"]
    if s["projector"] == "prepared":
        mp.magicpig_hash_decode_step_prepared(p, s["q"], s["K"], s["mu"], s["centering"], s["prepared"], n - 1, 1,
                                              s["key_codes"], s["q_codes"])
    else:
        mp.magicpig_hash_decode_step(p, s["q"], s["K"], s["mu"], s["W"], n - 1, 1, s["key_codes"], s["q_codes"], s["ws"])


def run(s):
    kind, p = s["kind"], s["params"]
    if kind in ("prefill", "prompt"):
        mp.magicpig_key_mean(p, s["K"], s["mu"], s["ws"])
        mp.magicpig_hash_keys(p, s["K"], s["mu"], s["W"], 0, s["n"], s["key_codes"], s["ws"])
        if kind == "prefill":
            return {"mu": s["mu"], "key_codes": s["key_codes"]}
        mp.magicpig_hash_query(p, s["q"], s["W"], s["q_codes"], s["ws"])
        mp.magicpig_sampled_attention(p, s["q"], s["K"], s["V"], s["mu"], s["key_codes"], s["q_codes"], s["out"],
                                      workspace=s["ws"])
        return {"mu": s["mu"], "key_codes": s["key_codes"], "q_codes": s["q_codes"], "out": s["out"]}
    if kind == "chunk":
        mp.magicpig_hash_keys(p, s["K"], s["mu"], s["W"], s["first"], s["keys"], s["key_codes"], s["ws"])
        return {"key_codes": s["key_codes"]}
    if kind == "rebuild":
        mp.magicpig_build_tables(s["build"], s["key_codes"], s["tables"], s["build_ws"])
    _step_codes(s)
    if kind == "step":
        mp.magicpig_sampled_attention(p, s["q"], s["K"], s["V"], s["mu"], s["key_codes"], s["q_codes"], s["out"],
                                      workspace=s["ws"])
    else:
        mp.magicpig_sampled_attention_tables(p, s["q"], s["K"], s["V"], s["mu"], s["tables"], s["indexed"], s["key_codes"],
                                             s["q_codes"], s["out"], workspace=s["ws"])
    got = {"out": s["out"], "q_codes": s["q_codes"], "key_codes": s["key_codes"]}
    if kind == "rebuild":
        got["offsets"] = s["offsets"]       # (the order of the indices inside a bucket is unspecified; the output is made from them)
    return got


# ---- what a pass cannot do without -------------------------------------------------------------------
def _sampled_fraction(c):
    """P[Binomial(L, 2^-K) >= min_hits]: the sampled share of keys orthogonal to the query."""
    x = 2.0 ** -c["K"]
    return 1.0 - sum(math.comb(c["L"], j) * x ** j * (1 - x) ** (c["L"] - j) for j in range(c["min_hits"]))


def work(case):
    c = _full(case)
    units, heads, n = c["batch"] * c["kv_heads"], c["batch"] * c["q_heads"], c["n"]
    cols = c["K"] * c["L"]
    elem = {"bf16": 2, "fp32": 4}[c["dtype"]]
    kv = 1 if c["kv"] else elem
    code = cols / 8.0                                          # bytes of a key's code
    project = 2.0 * D * cols                                   # operations of coding one vector
    proj_bytes = D * cols * elem
    if c["kind"] in ("prefill", "chunk"):
        keys = units * (n if c["kind"] == "prefill" else c["keys"])
        return {"bytes": keys * (D * kv + code) + proj_bytes, "flops": keys * project}
    rows = heads * (SINK + LOCAL + _sampled_fraction(c) * max(0, n - SINK - LOCAL))
    step = {"bytes": rows * 2 * D * kv + proj_bytes + heads * (D * elem + D * 4 + code) + units * (D * kv + D * 4 + code),
            "flops": (heads + units) * project + rows * 4.0 * D}
    scan = units * max(0, n - SINK - LOCAL) * code
    if c["kind"] == "step":
        step["bytes"] += scan
    elif c["kind"] == "prompt":
        step["bytes"] += units * n * (D * kv + 2 * code)
        step["flops"] += units * n * project
    else:
        step["bytes"] += heads * c["L"] * (8 + 4.0 * n / 2 ** c["K"]) + units * c["appended"] * code
        if c["kind"] == "rebuild":
            step["bytes"] += units * n * (code + 4.0 * c["L"])
    return step


def tolerance(case):
    c = _full(case)
    if c["kind"] == "chunk":
        return "exact"                                        # the sign of an exact sum
    # The mean is rounded to float32 (measured 2.5e-8 from 64 bits): another order of its sums moves it
    # by an ulp here and there (5.8e-8), and with it the sign of a projection in ten million (1e-6 of the words).
    if c["kind"] == "prefill":
        return {"rel": 2.5e-7, "max": 2e-6, "differ": 5e-6}
    if c["kind"] == "prompt":
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-4}    # (one word of a small prompt is 1e-5 of them)
    # float32 sums and the float32 inclusion probability (measured 0.6e-6 to 2e-6 from 64 bits); codes are exact
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}


# ---- the same in 64 bits -----------------------------------------------------------------------------
def _codes64(x, W64, K, L):
    """[rows, 128] in 64 bits -> [rows, L] codes."""
    bits = (x @ W64 >= 0).view(-1, L, K)
    code = torch.zeros(x.shape[0], L, dtype=torch.int32, device=x.device)
    for b in range(K):
        code |= bits[:, :, b].to(torch.int32) << b
    return code


def _inclusion64(p, K, L, tau):
    x = p ** K
    head, tail = torch.zeros_like(x), torch.zeros_like(x)
    for j in range(min(L, 64) + 1):     # (the tail counts where its mean L x is below about tau: nothing is left beyond 64)
        t = float(math.comb(L, j)) * x ** j * (1 - x) ** (L - j)
        if j < tau:
            head += t
        else:
            tail += t
    return torch.where(head < 0.5, 1.0 - head, tail)


def _attention64(c, Kc, Vc, q, W, mu):
    B, Hkv, G, n, K, L, tau = c["batch"], c["kv_heads"], c["q_heads"] // c["kv_heads"], c["n"], c["K"], c["L"], c["min_hits"]
    W64 = W.double()
    out = torch.zeros(B, c["q_heads"], D, dtype=torch.float64, device="cuda")
    i = torch.arange(n, device="cuda")
    static = (i < SINK) | (i >= n - LOCAL)
    for b in range(B):
        for h in range(Hkv):
            k = Kc[b, h, :n].to(torch.float32).double()
            v = Vc[b, h, :n].to(torch.float32).double()
            m = mu[b, h].double()
            kc = k - m
            qs = q[b, h * G:(h + 1) * G].double()
            qcode = _codes64(qs, W64, K, L)
            hits = torch.empty(G, n, dtype=torch.int32, device="cuda")
            for r in range(0, n, 32768):
                kcode = _codes64(kc[r:r + 32768], W64, K, L)
                for j in range(G):
                    hits[j, r:r + 32768] = (kcode == qcode[j]).sum(1)
            norm = kc.norm(dim=1)
            for j in range(G):
                at = (static | (hits[j] >= tau)).nonzero()[:, 0]
                logit = (k[at] @ qs[j]) / math.sqrt(D)
                cos = (kc[at] @ qs[j]) / (norm[at] * qs[j].norm()).clamp_min(1e-300)
                u = _inclusion64(1.0 - torch.arccos(cos.clamp(-1.0, 1.0)) / math.pi, K, L, tau).clamp_min(1e-300)
                logit = torch.where(static[at], logit, logit - u.log())
                out[b, h * G + j] = torch.softmax(logit, 0) @ v[at]
    return out


def exact(case, seed):
    c = _full(case)
    if c["kind"] == "chunk":
        return None
    Kc, Vc, q, W, mu, _ = _inputs(c, seed)
    if c["kind"] == "prefill":
        mean = torch.stack([torch.stack([Kc[b, h, :c["n"]].to(torch.float32).double().mean(0) for h in range(c["kv_heads"])])
                            for b in range(c["batch"])])
        return {"mu": mean, "key_codes": None}
    out = _attention64(c, Kc, Vc, q, W, mu)
    if c["kind"] == "prompt":
        mean = torch.stack([torch.stack([Kc[b, h, :c["n"]].to(torch.float32).double().mean(0) for h in range(c["kv_heads"])])
                            for b in range(c["batch"])])
        return {"mu": mean, "key_codes": None, "q_codes": None, "out": out}
    return {"out": out, "q_codes": None, "key_codes": None}
