"""The calls that speed is measured on: one pass of the framework's public entry
points over the sizes that slotted decoding runs at.

Sizes are those of the repository's workloads (`workloads/`): the 0.6B, 1.7B and
4B shapes, the training layout, the Mode A denoising step, and the same shapes
for a single sequence; `draw` spreads over the ranges around them, odd and
ragged sizes included.  Distributions follow `workloads/`: Q, K, V and hidden
states are N(0, 1), the LM head N(0, 0.02^2), rounded to the storage type.

As in a serving loop, outputs and workspaces are kept by the caller and passed
in.  Calls that update the caller's state in place (prefix lengths, the mask)
first restore it with a device copy, so that a pass can be repeated.
"""

import math

import torch

import paper_2609_19868_amd as Z
from paper_2609_19868_amd import _lib

VOCAB = 151936
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


# ------------------------------------------------------------------ the cases


def _attn(name, B, heads, P, S, L, D=128, dtype="bf16", ar=False, causal=False, ragged=False):
    return dict(name=name, kind="attn", dtype=dtype, B=B, Hq=heads[0], Hkv=heads[1], D=D, P=P, S=S, L=L, ar=ar,
                causal=causal, ragged=ragged)


def _head(name, kind, M, H, V=VOCAB, dtype="bf16", targets=False, temperature=1.0):
    return dict(name=name, kind=kind, dtype=dtype, M=M, H=H, V=V, targets=targets, temperature=temperature)


def listed():
    return [
        # a whole scoring step of one interactive sequence (0.6B shape): the
        # smallest step a user runs, where launches and idle units count
        dict(_attn("score_single", 1, (16, 8), 2048, 8, 8), kind="score", H=1024, V=VOCAB),
        # one long-context sequence at the 4B shape: the cache is long, the batch is one
        _attn("attn_single_long", 1, (32, 8), 16384, 8, 16),
        # draft attention of a 0.6B serving batch
        _attn("attn_draft_0.6b", 16, (16, 8), 2048, 8, 8),
        # verification attention of a 1.7B serving batch whose rows have grown to
        # different, odd prefix lengths
        _attn("attn_verify_1.7b", 32, (16, 8), 4093, 16, 4, ar=True, ragged=True),
        # draft attention of the 4B serving batch (the headline step's attention)
        _attn("attn_draft_4b", 8, (32, 8), 16384, 8, 16),
        # training-layout attention: 4096 tokens, causal, no cache
        _attn("attn_layout", 8, (16, 8), 0, 128, 32, ar=True, causal=True),
        # draft attention in float32 (a reference-precision run of a small batch)
        _attn("attn_f32", 2, (16, 8), 1000, 8, 8, dtype="f32"),
        # LM-head confidence of the 4B serving batch with target ids (verification)
        _head("conf_verify_4b", "conf", 1024, 2560, targets=True),
        # LM-head confidence of a single sequence in float32
        _head("conf_f32", "conf", 64, 1024, dtype="f32"),
        # drafting with temperature at the 0.6B serving batch
        _head("sample_draft_0.6b", "sample", 1024, 1024, temperature=0.7),
        # a Mode A denoising step in the first-hitting sampler's order: causal
        # attention, random reveal, sampling of the revealed rows, cache append
        dict(name="mode_a_step", kind="mode_a", dtype="bf16", B=16, Hq=16, Hkv=8, D=128, P=2048, N=256, k=4, H=1024,
             V=VOCAB),
        # the bookkeeping between two model passes of a 0.6B serving batch:
        # selection, acceptance, append of the accepted tokens to the cache
        dict(name="commit_0.6b", kind="commit", dtype="bf16", B=16, Hkv=8, D=128, P=2048, S=8, L=8, topk=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_attn(rng, dtype):
    while True:
        P = 0 if rng.random() < 0.1 else _log_int(rng, 33, 16384 if dtype == "bf16" else 2048)
        causal = P == 0 or rng.random() < 0.2
        S, L = (_log_int(rng, 8, 128), _log_int(rng, 8, 32)) if P == 0 else (_log_int(rng, 1, 16), _log_int(rng, 1, 24))
        c = _attn("", _log_int(rng, 1, 32 if dtype == "bf16" else 4), rng.choice([(16, 8), (32, 8), (16, 8), (12, 4), (8, 8)]),
                  P, S, L, D=rng.choice([128, 128, 128, 64]), dtype=dtype, ar=rng.random() < 0.5, causal=causal,
                  ragged=P > 0 and rng.random() < 0.4)
        w = work(c)
        top = 2.5e11 if dtype == "bf16" else 1e9
        if w["flops"] <= top and w["bytes"] <= 6e8:
            return c


def _draw_head(rng, kind, dtype):
    while True:
        M = _log_int(rng, 1, 4096) if dtype == "bf16" else _log_int(rng, 1, 64)
        H = rng.choice([1024, 2048, 2560, 8 * rng.randint(64, 512)]) if dtype == "bf16" else rng.choice([1024, rng.randint(256, 1024)])
        V = rng.choice([VOCAB, _log_int(rng, 30000, VOCAB)])
        if 2.0 * M * H * V <= (8e11 if dtype == "bf16" else 2e10):
            return _head("", kind, M, H, V, dtype, targets=kind == "conf" and rng.random() < 0.5,
                         temperature=round(rng.uniform(0.5, 1.5), 2) if kind == "sample" else 1.0)


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "conf", "conf", "sample", "score", "mode_a", "commit", "f32"])
    if kind == "attn":
        c = _draw_attn(rng, "bf16")
    elif kind == "f32":
        c = _draw_attn(rng, "f32") if rng.random() < 0.5 else _draw_head(rng, "conf", "f32")
    elif kind in ("conf", "sample"):
        c = _draw_head(rng, kind, "bf16")
    elif kind == "score":
        c = dict(_attn("", _log_int(rng, 1, 8), (16, 8), _log_int(rng, 100, 4096), rng.randint(2, 12), rng.randint(1, 12)),
                 kind="score", H=rng.choice([1024, 2048]), V=VOCAB)
    elif kind == "mode_a":
        c = dict(name="", kind="mode_a", dtype="bf16", B=_log_int(rng, 1, 16), Hq=16, Hkv=8, D=128,
                 P=_log_int(rng, 100, 2048), N=_log_int(rng, 24, 400), k=rng.randint(1, 6), H=1024, V=VOCAB)
    else:
        c = dict(name="", kind="commit", dtype="bf16", B=_log_int(rng, 1, 32), Hkv=8, D=rng.choice([64, 128]),
                 P=_log_int(rng, 100, 4096), S=rng.randint(2, 24), L=rng.randint(1, 24), topk=rng.randint(1, 4))
    del c["name"]
    return c


# ----------------------------------------------------------------- the states


def _normal(g, shape, dtype, std=1.0):
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    step = 1 << 26
    for i in range(0, flat.numel(), step):  # in pieces: the float32 draw of a large tensor is never whole
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device="cuda") * std
    return out


def _conf_out(M, targets):
    out = {"max_prob": torch.empty(M, device="cuda"), "argmax": torch.empty(M, dtype=torch.int32, device="cuda"),
           "lse": torch.empty(M, device="cuda")}
    if targets:
        out["target_prob"] = torch.empty(M, device="cuda")
    return out


def _sample_out(M):
    return {"sample_prob": torch.empty(M, device="cuda"), "max_prob": torch.empty(M, device="cuda"),
            "lse": torch.empty(M, device="cuda"), "sample_id": torch.empty(M, dtype=torch.int32, device="cuda")}


def _head_state(c, g, M, H, V, dtype):
    return {"hidden": _normal(g, (M, H), dtype), "w": _normal(g, (V, H), dtype, 0.02)}


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device="cuda")


def _i32(*shape):
    return torch.empty(shape, dtype=torch.int32, device="cuda")


def _attn_state(c, g, T, cap):
    B, Hq, Hkv, D, dt = c["B"], c["Hq"], c["Hkv"], c["D"], DTYPES[c["dtype"]]
    s = {"q": _normal(g, (B, Hq, T, D), dt), "ks": _normal(g, (B, Hkv, T, D), dt), "vs": _normal(g, (B, Hkv, T, D), dt),
         "kc": _normal(g, (B, Hkv, cap, D), dt) if cap else None, "vc": _normal(g, (B, Hkv, cap, D), dt) if cap else None}
    s["out"], s["lse"] = torch.empty_like(s["q"]), torch.empty((B, Hq, T), device="cuda")
    return s


def _attn_options(c):
    return dict(pass_=Z.PASS_AR_INFILL if c["ar"] else Z.PASS_DIFFUSION,
                cross_slot=Z.CROSS_SLOT_CAUSAL if c["causal"] else Z.CROSS_SLOT_NONE)


def _attn_workspace(s, S, L, P, **options):
    return _bytes(_lib.slot_attn_workspace_size(Z.slot_attn_desc(s["q"], s["kc"], s["ks"], S, L, prefix_len=P, **options)))


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda").manual_seed(seed)
    kind = c["kind"]
    if kind in ("attn", "score"):
        T = c["S"] * c["L"]
        s = _attn_state(c, g, T, c["P"])
        s["lens"] = None
        if c["ragged"]:  # rows between half and all of the longest prefix
            s["lens"] = torch.randint(max(1, c["P"] // 2), c["P"] + 1, (c["B"],), generator=g, device="cuda", dtype=torch.int32)
        s["attn_ws"] = _attn_workspace(s, c["S"], c["L"], c["P"], **_attn_options(c))
        if kind == "score":
            M = c["B"] * T
            s.update(_head_state(c, g, M, c["H"], c["V"], torch.bfloat16), conf=_conf_out(M, False))
            s["conf_ws"] = _bytes(_lib.slot_confidence_workspace_size(
                _lib.ConfDesc(n_rows=M, hidden=c["H"], vocab=c["V"], dtype=Z.DTYPE_BF16)))
            s["sel"] = (torch.empty((c["B"], c["S"]), device="cuda"), _i32(c["B"], c["S"]), _i32(c["B"]))
    elif kind in ("conf", "sample"):
        dt = DTYPES[c["dtype"]]
        s = _head_state(c, g, c["M"], c["H"], c["V"], dt)
        desc = _lib.ConfDesc(n_rows=c["M"], hidden=c["H"], vocab=c["V"],
                             dtype=Z.DTYPE_BF16 if c["dtype"] == "bf16" else Z.DTYPE_F32)
        if kind == "conf":
            s["targets"] = None
            if c["targets"]:
                s["targets"] = torch.randint(0, c["V"], (c["M"],), generator=g, device="cuda", dtype=torch.int32)
            s["conf"] = _conf_out(c["M"], c["targets"])
            s["conf_ws"] = _bytes(_lib.slot_confidence_workspace_size(desc))
        else:
            s["sample"] = _sample_out(c["M"])
            s["sample_ws"] = _bytes(_lib.slot_sample_workspace_size(desc))
    elif kind == "mode_a":
        B, N, k = c["B"], c["N"], c["k"]
        s = _attn_state(c, g, N + k, c["P"] + k)  # k rows revealed by the last step, N still masked
        s["lens0"] = torch.full((B,), c["P"], dtype=torch.int32, device="cuda")
        s["lens"] = s["lens0"].clone()
        s.update(_head_state(c, g, B * N, c["H"], c["V"], torch.bfloat16))
        s["mask0"] = torch.ones((B, N), dtype=torch.uint8, device="cuda")
        s["mask"] = s["mask0"].clone()
        s["k"] = torch.full((B,), k, dtype=torch.int32, device="cuda")
        s["rev"] = (_i32(B, N), _i32(B))
        s["row_base"] = (torch.arange(B, dtype=torch.int32, device="cuda") * N).view(B, 1)
        s["rows"] = _i32(B * k)
        s["accepted"] = torch.zeros((B, N + k, 1), dtype=torch.uint8, device="cuda")
        s["accepted"][:, :k] = 1
        s["order"] = torch.arange(N + k, dtype=torch.int32, device="cuda").repeat(B, 1).contiguous()
        s["sample"] = _sample_out(B * k)
        s["attn_ws"] = _attn_workspace(s, N + k, 1, c["P"], pass_=Z.PASS_AR_INFILL, cross_slot=Z.CROSS_SLOT_CAUSAL)
        s["sample_ws"] = _bytes(_lib.slot_sample_workspace_size(
            _lib.ConfDesc(n_rows=B * k, hidden=c["H"], vocab=c["V"], dtype=Z.DTYPE_BF16)))
    else:
        B, Hkv, D, S, L = c["B"], c["Hkv"], c["D"], c["S"], c["L"]
        T, dt = S * L, DTYPES[c["dtype"]]
        s = {"kc": _normal(g, (B, Hkv, c["P"] + T, D), dt), "vc": _normal(g, (B, Hkv, c["P"] + T, D), dt),
             "ks": _normal(g, (B, Hkv, T, D), dt), "vs": _normal(g, (B, Hkv, T, D), dt)}
        s["lens0"] = torch.randint(max(1, c["P"] // 2), c["P"] + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
        s["lens"] = s["lens0"].clone()
        # draft confidences of a trained model: mostly high, with a tail
        s["conf"] = torch.rand((B, S, L), generator=g, device="cuda") ** 0.25
        s["prob"] = torch.rand((B, S, L), generator=g, device="cuda") ** 0.25
        s["sel"] = (torch.empty((B, S), device="cuda"), _i32(B, S), _i32(B))
        s["acc"] = (torch.empty((B, S, L), dtype=torch.uint8, device="cuda"), _i32(B, S), _i32(B))
    s["case"], s["seed"] = c, seed
    return s


def _run_attn(s, S, L, P, **options):
    return Z.slot_attn(s["q"], s["kc"], s["vc"], s["ks"], s["vs"], S, L, prefix_len=P, prefix_lens=s["lens"],
                       out=s["out"], lse=s["lse"], workspace=s["attn_ws"], **options)


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "attn":
        return _run_attn(s, c["S"], c["L"], c["P"], **_attn_options(c))
    if kind == "score":
        out, lse = _run_attn(s, c["S"], c["L"], c["P"], **_attn_options(c))
        conf = Z.slot_confidence(s["hidden"], s["w"], out=s["conf"], workspace=s["conf_ws"])
        sel = Z.select_slots(conf["max_prob"].view(c["B"], c["S"], c["L"]), threshold=0.9, out=s["sel"])
        return [out, lse, conf, sel]
    if kind == "conf":
        return Z.slot_confidence(s["hidden"], s["w"], target_ids=s["targets"], out=s["conf"], workspace=s["conf_ws"])
    if kind == "sample":
        return Z.slot_sample(s["hidden"], s["w"], c["temperature"], s["seed"], 1, out=s["sample"], workspace=s["sample_ws"])
    if kind == "mode_a":
        s["lens"].copy_(s["lens0"])
        s["mask"].copy_(s["mask0"])
        out, lse = _run_attn(s, c["N"] + c["k"], 1, c["P"], pass_=Z.PASS_AR_INFILL, cross_slot=Z.CROSS_SLOT_CAUSAL)
        rev = Z.mdm_reveal(s["mask"], s["k"], Z.REVEAL_RANDOM, seed=s["seed"], offset=2, out=s["rev"])
        torch.add(rev[0][:, :c["k"]], s["row_base"], out=s["rows"].view(c["B"], c["k"]))
        sample = Z.slot_sample(s["hidden"], s["w"], 1.0, s["seed"], 2, rows=s["rows"], out=s["sample"],
                               workspace=s["sample_ws"])
        cache = Z.kv_append(s["kc"], s["vc"], s["lens"], s["ks"], s["vs"], s["accepted"], s["order"])
        return [out, lse, rev, s["mask"], sample, cache]
    s["lens"].copy_(s["lens0"])
    sel = Z.select_slots(s["conf"], conf_rule=Z.SLOT_CONF_MEAN, rule=Z.SELECT_TOP_K, k=c["topk"], out=s["sel"])
    acc = Z.verify_accept(s["prob"], sel[1], 0.4, out=s["acc"])
    cache = Z.kv_append(s["kc"], s["vc"], s["lens"], s["ks"], s["vs"], acc[0], sel[1])
    return [sel, acc, cache]


# ------------------------------------------------------- the work of one pass


def _attn_work(B, Hq, Hkv, D, P, S, L, T, e, ar, causal):
    """Keys seen by a token: the prefix, its slot (AR: up to itself) and with the
    causal order every earlier slot."""
    own = (L + 1) / 2 if ar else L
    seen = P + own + (L * (S - 1) / 2 if causal else 0)
    return {"bytes": e * D * (2 * B * Hkv * (P + T) + 2 * B * Hq * T) + 4 * B * Hq * T, "flops": 4.0 * B * Hq * T * seen * D}


def _head_work(M, H, V, e, outputs=3):
    return {"bytes": e * H * (V + M) + 4 * outputs * M, "flops": 2.0 * M * H * V}


def _sum(*works):
    return {k: sum(w[k] for w in works) for k in ("bytes", "flops")}


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] in ("attn", "score"):
        T = c["S"] * c["L"]
        P = c["P"] * 0.75 if c["ragged"] else c["P"]  # the mean of the ragged rows
        a = _attn_work(c["B"], c["Hq"], c["Hkv"], c["D"], P, c["S"], c["L"], T, e, c["ar"], c["causal"])
        return _sum(a, _head_work(c["B"] * T, c["H"], c["V"], 2)) if c["kind"] == "score" else a
    if c["kind"] in ("conf", "sample"):
        return _head_work(c["M"], c["H"], c["V"], e, 4)
    if c["kind"] == "mode_a":
        a = _attn_work(c["B"], c["Hq"], c["Hkv"], c["D"], c["P"], c["N"] + c["k"], 1, c["N"] + c["k"], e, True, True)
        append = {"bytes": 4 * c["B"] * c["Hkv"] * c["k"] * c["D"] * e, "flops": 0}
        return _sum(a, _head_work(c["B"] * c["k"], c["H"], c["V"], 2, 4), append)
    # about 95% of the tokens of the selected slots are accepted: K and V read and written
    n = c["B"] * min(c["topk"], c["S"]) * c["L"]
    return {"bytes": 0.95 * n * 4 * c["Hkv"] * c["D"] * e + 9 * c["B"] * c["S"] * c["L"], "flops": 0}


def tolerance(case):
    """rel: about four times the difference between two sound implementations at
    the same precision.  bf16 attention rounds its probabilities and its output
    to bf16 (measured against `exact`: 2.3e-3); float32 attention and the LM head
    sum and report float32 (measured 5e-8 to 1.5e-6)."""
    kind = case["kind"]
    if kind == "commit":
        return "exact"
    if case["dtype"] == "f32" or kind in ("conf", "sample"):
        return {"rel": 1e-5, "max": 2e-4, "differ": 2e-3}
    return {"rel": 1e-2, "max": 0.1, "differ": 2e-3}


# ------------------------------------------------------------- 64-bit results


def _exact_attn(s, T, S, L, ar, causal, lens):
    q, B = s["q"], s["q"].shape[0]
    Hq, D, Hkv = q.shape[1], q.shape[3], s["ks"].shape[1]
    G = Hq // Hkv
    t = torch.arange(T, device="cuda")
    hi = t + 1 if ar else (t // L + 1) * L
    lo = torch.zeros_like(t) if causal else (t // L) * L
    hidden = ~((t[None] >= lo[:, None]) & (t[None] < hi[:, None]))
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(q.shape[:3], dtype=torch.float64, device="cuda")
    for b in range(B):
        n = lens[b]
        for h in range(Hkv):
            k = s["ks"][b, h].double() if not n else torch.cat([s["kc"][b, h, :n], s["ks"][b, h]]).double()
            v = s["vs"][b, h].double() if not n else torch.cat([s["vc"][b, h, :n], s["vs"][b, h]]).double()
            kt = k.t().contiguous()
            for a in range(h * G, (h + 1) * G):
                z = torch.mm(q[b, a].double(), kt) / math.sqrt(D)
                z[:, n:].masked_fill_(hidden, -math.inf)
                lse[b, a] = torch.logsumexp(z, 1)
                out[b, a] = torch.mm(torch.exp(z - lse[b, a][:, None]), v)
    return out, lse


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 words (int64 tensors holding 32 bits) of the counters."""
    m = 0xFFFFFFFF
    k0, k1 = seed & m, (seed >> 32) & m
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # low 64 bits; masked after the shift
        c0, c1, c2, c3 = ((p1 >> 32) & m) ^ c1 ^ k0, p1 & m, ((p0 >> 32) & m) ^ c3 ^ k1, p0 & m
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return torch.stack(torch.broadcast_tensors(c0, c1, c2, c3), -1)


def _uniform_words(ids, rows, offset, seed):
    """[rows, ids] 23-bit words of vocabulary ids or positions (a multiple of 4, from 0)."""
    q = (ids[::4] // 4)[None]
    zero = torch.zeros_like(q)
    w = _philox(q + 0 * rows[:, None], rows[:, None] + zero, zero + (offset & 0xFFFFFFFF), zero + (offset >> 32), seed)
    return w.reshape(rows.numel(), -1) >> 9


def _exact_head(hidden, w, targets=None, temperature=None, seed=0, offset=0):
    M, V = hidden.shape[0], w.shape[0]
    res = {k: torch.empty(M, dtype=torch.float64, device="cuda") for k in ("max_prob", "lse", "picked")}
    vocab4 = torch.arange((V + 3) // 4 * 4, device="cuda")
    for r0 in range(0, M, 128):
        h = hidden[r0:r0 + 128].double()
        z = torch.cat([torch.mm(h, w[v:v + 16384].double().t().contiguous()) for v in range(0, V, 16384)], 1)
        lse = torch.logsumexp(z, 1)
        pick = targets[r0:r0 + 128].long() if targets is not None else None
        if temperature is not None:
            u = _uniform_words(vocab4, torch.arange(r0, r0 + h.shape[0], device="cuda"), offset, seed)[:, :V]
            u = (u.double() + 0.5) * 2.0 ** -23
            pick = (z / temperature - torch.log(-torch.log(u))).argmax(1)
            del u
        res["max_prob"][r0:r0 + 128] = torch.exp(z.max(1).values - lse)
        res["lse"][r0:r0 + 128] = lse
        if pick is not None:
            res["picked"][r0:r0 + 128] = torch.exp(z.gather(1, pick[:, None])[:, 0] - lse)
    return res


def _exact_conf(e, targets):
    out = {"max_prob": e["max_prob"], "argmax": None, "lse": e["lse"]}
    if targets is not None:
        out["target_prob"] = e["picked"]
    return out


def _exact_sample(e):
    return {"sample_prob": e["picked"], "max_prob": e["max_prob"], "lse": e["lse"], "sample_id": None}


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind == "commit":  # copies, comparisons and one mean rounded to float32: nothing to compute in 64 bits
        return None
    s = prepare(c, seed)
    if kind in ("attn", "score"):
        lens = s["lens"].tolist() if s["lens"] is not None else [c["P"]] * c["B"]
        out, lse = _exact_attn(s, c["S"] * c["L"], c["S"], c["L"], c["ar"], c["causal"], lens)
        if kind == "attn":
            return out, lse
        e = _exact_head(s["hidden"], s["w"])
        first = e["max_prob"].view(c["B"], c["S"], c["L"])[:, :, 0]
        return [out, lse, _exact_conf(e, None), [first, None, None]]
    if kind == "conf":
        return _exact_conf(_exact_head(s["hidden"], s["w"], targets=s["targets"]), s["targets"])
    if kind == "sample":
        return _exact_sample(_exact_head(s["hidden"], s["w"], temperature=c["temperature"], seed=seed, offset=1))
    T = c["N"] + c["k"]
    out, lse = _exact_attn(s, T, T, 1, True, True, [c["P"]] * c["B"])
    pos = torch.arange((c["N"] + 3) // 4 * 4, device="cuda")
    words = _uniform_words(pos, torch.arange(c["B"], device="cuda"), 2, seed)[:, :c["N"]]
    order = torch.argsort(words, dim=1, stable=True)[:, :c["k"]]
    rows = (order + s["row_base"]).reshape(-1)
    e = _exact_head(s["hidden"][rows], s["w"], temperature=1.0, seed=seed, offset=2)
    return [out, lse, [None, None], None, _exact_sample(e), [None, None, None]]
