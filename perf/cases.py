"""The calls this library is timed on: one pass each through the Python entry points.

A case is a dict of plain values. The row lengths of a case follow from the case
itself ("lens" seeds them), so the work of a pass is fixed; the page order and all
values follow from the seed given to prepare(). Values are those of the repository's
workloads: bf16 N(0, 1) queries, keys and values, E4M3 codes of N(0, 1) for fp8 pools,
shuffled 16-token pages with pages between them that no row owns, hidden states N(0, 1)
and LM-head rows N(0, 1/D).

A serving loop keeps its caches, its workspace and (for decode, whose shapes are the
same from step to step) its output buffers: those are made in prepare(). It knows its
rows' lengths on the host, so the maxima are passed and no call reads them back.
"""
import math

import numpy as np
import torch

import paper_2603_18815_amd as ra

PAGE, DIM = 16, 128
SCALE = 1.0 / math.sqrt(DIM)
K_SCALE, V_SCALE = 0.02, 0.015        # fp8 pools: absmax of N(0, 1) data over 448, rounded up
DEVICE = "cuda:0"

# A drawn case does no more than this (the largest listed ones do about as much).
MOST_BYTES, MOST_FLOPS = 22e9, 6.7e12


def listed():
    return [
        # A few short trajectories at the start of a small model's rollout: launch-bound.
        dict(name="decode_b4_short", kind="decode", B=4, Hq=8, Hkv=2, lo=32, hi=256, median=0,
             fp8=False, lens=1),
        # A handful of live trajectories (the tail of a batch): too few rows to fill the chip.
        dict(name="decode_b8", kind="decode", B=8, Hq=32, Hkv=8, lo=2048, hi=16384, median=0,
             fp8=False, lens=2),
        # One decode step of a full batch, Qwen3-8B GQA shape.
        dict(name="decode_b64", kind="decode", B=64, Hq=32, Hkv=8, lo=4096, hi=32768, median=0,
             fp8=False, lens=2),
        # The same over fp8 E4M3 pools.
        dict(name="decode_b64_fp8", kind="decode", B=64, Hq=32, Hkv=8, lo=4096, hi=32768,
             median=0, fp8=True, lens=2),
        # Long-horizon decode, 32B-like heads, log-normal lengths.
        dict(name="decode_b256_long", kind="decode", B=256, Hq=64, Hkv=8, lo=512, hi=65536,
             median=16384, fp8=False, lens=4),
        # The rollouts of one task share its prompt pages: 8 tasks x 8 rollouts.
        dict(name="shared_8x8", kind="shared", groups=8, rows=8, Hq=32, Hkv=8, plo=2048,
             phi=8192, lo=2048, hi=24576, fp8=False, lens=6),
        # Two trajectories get their tool output at once: short chunks, long contexts.
        dict(name="append_b2", kind="append", B=2, Hq=32, Hkv=8, lo=2048, hi=24576, tlo=64,
             thi=512, fp8=False, lens=5),
        # The tool outputs of a whole batch (the repository's append workload).
        dict(name="append_b32", kind="append", B=32, Hq=32, Hkv=8, lo=2048, hi=24576, tlo=64,
             thi=2048, fp8=False, lens=3),
        # First prompts of eight trajectories: write with rotary embedding and prefill, no context.
        dict(name="prefill_rope_b8", kind="append_write", B=8, Hq=32, Hkv=8, lo=0, hi=0, tlo=512,
             thi=4096, fp8=False, rope=True, lens=7),
        # One rollout step: new tokens written, then decode rows and append rows in one launch.
        dict(name="step_b64", kind="step", B=64, Hq=32, Hkv=8, lo=512, hi=65536, median=12288,
             tlo=128, thi=4096, frac=0.15, fp8=False, lens=5),
        # Log-probabilities of one decode step's tokens, LM head packed once per policy.
        dict(name="logprob_n64_packed", kind="logprob", N=64, V=151936, D=4096, packed=True),
        # Scoring a stretch of trajectory under a policy that has just changed (row-major head).
        dict(name="logprob_n1000", kind="logprob", N=1000, V=151936, D=4096, packed=False),
    ]


HEADS = [(8, 2), (16, 1), (8, 8), (32, 8), (32, 8), (64, 8)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(["decode", "decode", "shared", "append", "append", "append_write", "step",
                       "logprob", "logprob"])
    if kind == "logprob":
        return dict(kind=kind, N=_log_int(rng, 1, 2048),
                    V=rng.choice([151936, 151936, 128256 + rng.randrange(64), 32000 - rng.randrange(64)]),
                    D=rng.choice([1024, 2048, 4096, 5120]), packed=rng.random() < 0.5)
    hq, hkv = rng.choice(HEADS)
    lens = rng.randrange(1 << 30)
    fp8 = rng.random() < 0.3
    hi = _log_int(rng, 64, 65536)
    lo = max(1, int(hi * rng.uniform(0.05, 0.9)))
    if kind == "decode":
        return dict(kind=kind, B=_log_int(rng, 1, 256), Hq=hq, Hkv=hkv, lo=lo, hi=hi,
                    median=0 if rng.random() < 0.7 else (lo + hi) // 3, fp8=fp8, lens=lens)
    if kind == "shared":
        phi = _log_int(rng, 256, 16384)
        hi = min(hi, 24576)
        return dict(kind=kind, groups=_log_int(rng, 1, 16), rows=_log_int(rng, 2, 16), Hq=hq,
                    Hkv=hkv, plo=max(16, phi // 4), phi=phi, lo=max(1, hi // 8), hi=hi, fp8=fp8,
                    lens=lens)
    thi = _log_int(rng, 16, 4096)
    tlo = max(1, int(thi * rng.uniform(0.05, 0.9)))
    if kind == "append":
        return dict(kind=kind, B=_log_int(rng, 1, 32), Hq=hq, Hkv=hkv, lo=min(lo, 32000),
                    hi=min(hi, 32000), tlo=tlo, thi=thi, fp8=fp8, lens=lens)
    if kind == "append_write":
        first = rng.random() < 0.5          # a first prompt has no context
        return dict(kind=kind, B=_log_int(rng, 1, 32), Hq=hq, Hkv=hkv,
                    lo=0 if first else min(lo, 16000), hi=0 if first else min(hi, 16000), tlo=tlo,
                    thi=thi, fp8=fp8, rope=rng.random() < 0.7, lens=lens)
    return dict(kind=kind, B=_log_int(rng, 8, 160), Hq=hq, Hkv=hkv, lo=lo, hi=hi,
                median=max(lo, hi // 5), tlo=tlo, thi=thi, frac=round(rng.uniform(0.05, 0.3), 2),
                fp8=fp8, lens=lens)


def draw(rng):
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["bytes"] <= MOST_BYTES and w["flops"] <= MOST_FLOPS:
            return case


# ---- lengths: a case's own ------------------------------------------------------------

def _lengths(rng, n, lo, hi, median=0):
    if median:
        x = np.rint(np.exp(rng.normal(math.log(median), 0.75, size=n)))
        return np.clip(x, lo, hi).astype(np.int64)
    return rng.integers(lo, hi + 1, size=n).astype(np.int64)


def _plan(c):
    """Per-row lengths: ctx (keys cached before the call) and t (new tokens; 0 in decode rows)."""
    rng = np.random.default_rng(c["lens"])
    if c["kind"] == "shared":
        pre = _lengths(rng, c["groups"], c["plo"], c["phi"]) // PAGE * PAGE
        suf = _lengths(rng, c["groups"] * c["rows"], c["lo"], c["hi"])
        return dict(pre=pre, suf=suf)
    if c["kind"] == "step":
        n_app = max(1, int(round(c["frac"] * c["B"])))
        app = np.zeros(c["B"], bool)
        app[rng.permutation(c["B"])[:n_app]] = True
        ctx = _lengths(rng, c["B"], c["lo"], c["hi"], c["median"])
        t = np.where(app, _lengths(rng, c["B"], c["tlo"], c["thi"]), 0)
        return dict(ctx=ctx, t=t, app=app)
    ctx = _lengths(rng, c["B"], c["lo"], c["hi"], c.get("median", 0))
    t = _lengths(rng, c["B"], c["tlo"], c["thi"]) if "tlo" in c else np.zeros(c["B"], np.int64)
    return dict(ctx=ctx, t=t, app=t > 0)


def _decode_bytes(lens, c):
    el = 1 if c["fp8"] else 2
    pages = (np.asarray(lens) + PAGE - 1) // PAGE
    return int(np.sum(lens)) * c["Hkv"] * DIM * 2 * el + len(lens) * (c["Hq"] * DIM * 6 + 4) + 4 * int(pages.sum())


def work(c):
    if c["kind"] == "logprob":
        return {"bytes": c["V"] * c["D"] * 2 + c["N"] * c["D"] * 2 + 8 * c["N"],
                "flops": 2 * c["N"] * c["V"] * c["D"]}
    p = _plan(c)
    if c["kind"] == "shared":
        el = 1 if c["fp8"] else 2
        keys = int(p["pre"].sum() + p["suf"].sum())
        all_keys = int(p["pre"].sum() * c["rows"] + p["suf"].sum())
        rows = p["suf"].shape[0]
        return {"bytes": keys * c["Hkv"] * DIM * 2 * el + rows * (c["Hq"] * DIM * 6 + 4) + 4 * (all_keys // PAGE),
                "flops": 4 * DIM * c["Hq"] * all_keys}
    if c["kind"] == "decode":
        return {"bytes": _decode_bytes(p["ctx"], c), "flops": 4 * DIM * c["Hq"] * int(p["ctx"].sum())}
    ctx, t = p["ctx"][p["app"]], p["t"][p["app"]]
    el = 1 if c["fp8"] else 2
    flops = 4 * DIM * c["Hq"] * int((t * ctx + t * (t + 1) // 2).sum())
    nbytes = int((ctx + t).sum()) * c["Hkv"] * DIM * 2 * el + int(t.sum()) * c["Hq"] * DIM * 6
    if c["kind"] in ("append_write", "step"):       # the new tokens' K and V in (the pool side is above)
        nbytes += int(t.sum()) * c["Hkv"] * DIM * 2 * (2 + el)
    if c["kind"] == "step":
        dec = p["ctx"][~p["app"]]
        nbytes += _decode_bytes(dec, c) + len(dec) * c["Hkv"] * DIM * 2 * (2 + el)
        flops += 4 * DIM * c["Hq"] * int(dec.sum())
    return {"bytes": nbytes, "flops": flops}


def tolerance(c):
    # About four times the error against exact() that the path shows.
    if c["kind"] in ("append", "append_write", "step"):
        return {"rel": 6e-3, "max": 0.1}      # weights meet V as bf16: 1.3e-3 to 1.7e-3 seen
    if c["kind"] == "logprob":
        return {"rel": 1e-6, "max": 1e-5}     # fp32 sums over D and V, in any order: 6e-8 seen
    return {"rel": 1e-5, "max": 4e-4}         # fp32 sums, weights kept to about 16 bits: 2e-6 seen


# ---- inputs -----------------------------------------------------------------------------

def _randn(shape, gen, scale=1.0):
    out = torch.empty(shape, dtype=torch.bfloat16, device=DEVICE)
    flat, step = out.view(-1), 1 << 27
    for s in range(0, flat.numel(), step):
        e = min(flat.numel(), s + step)
        x = torch.randn(e - s, generator=gen, device=DEVICE)
        flat[s:e] = x if scale == 1.0 else x * scale
    return out


def _codes(shape, gen, scale):
    out = torch.empty(shape, dtype=torch.uint8, device=DEVICE)
    flat, step = out.view(-1), 1 << 27
    for s in range(0, flat.numel(), step):
        e = min(flat.numel(), s + step)
        x = torch.randn(e - s, generator=gen, device=DEVICE) / scale
        flat[s:e] = x.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    return out


def _gpu(x):
    return torch.as_tensor(np.ascontiguousarray(x, dtype=np.int32), device=DEVICE)


def _table(rng, row_pages, shared=None):
    """Block table of rows on shuffled pages; shared: (row's group, pages each group shares)."""
    own = row_pages if shared is None else row_pages - shared[1][shared[0]]
    used = int(own.sum()) + (0 if shared is None else int(shared[1].sum()))
    spare = max(16, used // 100)
    perm = rng.permutation(used + spare).astype(np.int32)
    table = np.full((len(row_pages), max(1, int(row_pages.max()))), perm[-1], np.int32)
    at = 0
    heads = []
    if shared is not None:
        for n in shared[1]:
            heads.append(perm[at:at + int(n)])
            at += int(n)
    for b, n in enumerate(own):
        pre = heads[shared[0][b]] if shared is not None else perm[:0]
        table[b, :len(pre)] = pre
        table[b, len(pre):len(pre) + int(n)] = perm[at:at + int(n)]
        at += int(n)
    return table, used + spare


def _pools(c, pages, gen):
    ks, vs = (pages, c["Hkv"], PAGE, DIM), (pages, c["Hkv"], DIM, PAGE)
    if c["fp8"]:
        return _codes(ks, gen, K_SCALE), _codes(vs, gen, V_SCALE)
    return _randn(ks, gen), _randn(vs, gen)


def _cache(c, k, v, table):
    return ra.PagedKV(k, v, _gpu(table), K_SCALE if c["fp8"] else None, V_SCALE if c["fp8"] else None)


def _workspace(n):
    return torch.empty(max(int(n), 1), dtype=torch.uint8, device=DEVICE)


def _rope_table(rows):
    """cos | sin of the Qwen3 frequencies (theta 10^6) per position, fp32 [rows][128]."""
    inv = 1e6 ** (-torch.arange(0, DIM, 2, dtype=torch.float64, device=DEVICE) / DIM)
    ang = torch.arange(rows, dtype=torch.float64, device=DEVICE)[:, None] * inv[None, :]
    return torch.cat([ang.cos(), ang.sin()], 1).float().contiguous()


def prepare(case, seed):
    c = case
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    rng = np.random.default_rng(int(seed))
    s = {"case": c}
    if c["kind"] == "logprob":
        s["h"] = _randn((c["N"], c["D"]), gen)
        s["W"] = _randn((c["V"], c["D"]), gen, c["D"] ** -0.5)
        s["targets"] = _gpu(rng.integers(0, c["V"], c["N"]))
        if c["packed"]:
            s["Wp"] = ra.token_logprob_pack_weight(s["W"])
        s["ws"] = _workspace(ra.token_logprob_workspace_size(c["N"], c["V"], c["D"]))
        return s
    p = _plan(c)
    if c["kind"] == "shared":
        group = np.repeat(np.arange(c["groups"]), c["rows"])
        lens = p["pre"][group] + p["suf"]
        table, pages = _table(rng, p["pre"][group] // PAGE + (p["suf"] + PAGE - 1) // PAGE,
                              (group, p["pre"] // PAGE))
        s["group_start"] = _gpu(np.arange(c["groups"] + 1) * c["rows"])
        s["prefix_len"] = _gpu(p["pre"])
        s["max_prefix"] = int(p["pre"].max())
    else:
        lens = p["ctx"] + p["t"]
        table, pages = _table(rng, (lens + PAGE - 1) // PAGE)
    k, v = _pools(c, pages, gen)
    s["k_pool"], s["v_pool"] = k, v
    dec = np.nonzero(~p["app"])[0] if "app" in p else np.arange(len(lens))
    app = np.nonzero(p["app"])[0] if "app" in p else np.arange(0)
    if dec.size:
        s["kv"] = _cache(c, k, v, table[dec])
        s["q"] = _randn((dec.size, c["Hq"], DIM), gen)
        s["kv_lens"], s["max_kv"] = _gpu(lens[dec]), int(lens[dec].max())
    if app.size:
        t, ctx = p["t"][app], p["ctx"][app]
        s["kv_a"] = _cache(c, k, v, table[app])
        s["q_a"] = _randn((int(t.sum()), c["Hq"], DIM), gen)
        s["cu_q"], s["ctx"] = _gpu(np.concatenate([[0], np.cumsum(t)])), _gpu(ctx)
        s["max_t"], s["max_kv_a"] = int(t.max()), int((ctx + t).max())
    if c["kind"] in ("append_write", "step"):
        # a decode row writes the token it decodes (its last key), an append row its chunk
        n = np.concatenate([np.ones(dec.size, np.int64), p["t"][app]])
        start = np.concatenate([lens[dec] - 1, p["ctx"][app]])
        s["k_new"] = _randn((int(n.sum()), c["Hkv"], DIM), gen)
        s["v_new"] = _randn((int(n.sum()), c["Hkv"], DIM), gen)
        s["cu_new"], s["start"] = _gpu(np.concatenate([[0], np.cumsum(n)])), _gpu(start)
        s["max_new"], s["max_pos"] = int(n.max()), int((n + start).max())
        s["kv_w"] = _cache(c, k, v, np.concatenate([table[dec], table[app]]))
        s["cos_sin"] = _rope_table(int(lens.max())) if c.get("rope") else None
    B, hq, hkv = len(lens), c["Hq"], c["Hkv"]
    if c["kind"] == "decode":
        s["ws"] = _workspace(ra.decode_workspace_size(B, hq, hkv, s["max_kv"]))
    elif c["kind"] == "shared":
        s["ws"] = _workspace(ra.decode_shared_prefix_workspace_size(B, hq, hkv, s["max_kv"], s["max_prefix"]))
    elif c["kind"] == "step":
        s["ws"] = _workspace(ra.mixed_workspace_size(dec.size, app.size, hq, hkv, hkv,
                                                     s.get("max_kv", 0), s["max_t"]))
    else:
        s["ws"] = _workspace(ra.append_workspace_size(B, hq, hkv, s["max_t"]))
    if c["kind"] in ("decode", "shared"):
        s["out"] = torch.empty((B, hq, DIM), dtype=torch.float32, device=DEVICE)
        s["lse"] = torch.empty((B, hq), dtype=torch.float32, device=DEVICE)
    return s


# ---- one pass ---------------------------------------------------------------------------

def run(state):
    s, c = state, state["case"]
    if c["kind"] == "decode":
        return ra.decode(s["q"], s["kv"], s["kv_lens"], s["max_kv"], SCALE, out=s["out"],
                         lse=s["lse"], workspace=s["ws"])
    if c["kind"] == "shared":
        return ra.decode_shared_prefix(s["q"], s["kv"], s["kv_lens"], s["group_start"],
                                       s["prefix_len"], c["rows"], s["max_prefix"], s["max_kv"],
                                       SCALE, out=s["out"], lse=s["lse"], workspace=s["ws"])
    if c["kind"] == "append":
        return ra.append(s["q_a"], s["cu_q"], s["ctx"], s["kv_a"], s["max_t"], s["max_kv_a"],
                         SCALE, want_lse=True, workspace=s["ws"])
    if c["kind"] == "append_write":
        out, lse = ra.append_write(s["q_a"], s["k_new"], s["v_new"], s["cu_q"], s["ctx"],
                                   s["kv_a"], s["max_t"], s["max_kv_a"], SCALE, want_lse=True,
                                   workspace=s["ws"], cos_sin=s["cos_sin"])
        return out, lse, s["k_pool"], s["v_pool"]
    if c["kind"] == "step":
        ra.kv_page_write(s["k_new"], s["v_new"], s["cu_new"], s["start"], s["kv_w"], s["max_new"],
                         s["max_pos"])
        got = ra.mixed(s["q"], s["kv"], s["kv_lens"], s["q_a"], s["cu_q"], s["ctx"], s["kv_a"],
                       s["max_kv"], s["max_t"], s["max_kv_a"], SCALE, want_lse=True,
                       workspace=s["ws"])
        return (*got, s["k_pool"], s["v_pool"])
    if c["packed"]:
        return ra.token_logprob_packed(s["h"], s["Wp"], c["V"], s["targets"], want_lse=True,
                                       workspace=s["ws"])
    return ra.token_logprob(s["h"], s["W"], s["targets"], want_lse=True, workspace=s["ws"])


# ---- the same in 64 bits, plain torch -----------------------------------------------------

def _values(codes_or_bf16, scale):
    if codes_or_bf16.dtype == torch.uint8:
        return codes_or_bf16.view(torch.float8_e4m3fn).double() * scale
    return codes_or_bf16.double()


def _row_kv(s, table_row, length):
    """A row's keys and values in 64 bits, [Hkv][length][128]."""
    n = (length + PAGE - 1) // PAGE
    ids = table_row[:n].long()
    k = _values(s["k_pool"][ids], K_SCALE)
    v = _values(s["v_pool"][ids], V_SCALE).transpose(2, 3)
    hkv = k.shape[1]
    k = k.transpose(0, 1).reshape(hkv, n * PAGE, DIM)[:, :length]
    v = v.transpose(0, 1).reshape(hkv, n * PAGE, DIM)[:, :length]
    return k.contiguous(), v.contiguous()


def _attend(q, k, v, ctx):
    """q [T][Hq][128] at positions ctx.., k / v [Hkv][L][128]; query i sees keys 0..ctx + i."""
    T, hq, _ = q.shape
    hkv, L, _ = k.shape
    G = hq // hkv
    out = torch.empty((T, hq, DIM), dtype=torch.float64, device=DEVICE)
    lse = torch.empty((T, hq), dtype=torch.float64, device=DEVICE)
    step = max(1, (1 << 27) // max(1, G * L))
    for i in range(0, T, step):
        j = min(T, i + step)
        dead = torch.arange(L, device=DEVICE)[None, :] > (ctx + torch.arange(i, j, device=DEVICE))[:, None]
        for g in range(hkv):
            x = q[i:j, g * G:(g + 1) * G].double().reshape((j - i) * G, DIM)
            z = (x @ k[g].t()).mul_(SCALE).view(j - i, G, L)
            z.masked_fill_(dead[:, None, :], -math.inf)
            m = z.logsumexp(-1)
            w = z.sub_(m[..., None]).exp_().view((j - i) * G, L)
            out[i:j, g * G:(g + 1) * G] = (w @ v[g]).view(j - i, G, DIM)
            lse[i:j, g * G:(g + 1) * G] = m
    return out, lse


def _rope(x, pos, cos_sin):
    """Rotate-half in fp32 with separately rounded products and sums, to bf16 (what a cache holds)."""
    c, sn = cos_sin[pos, None, :DIM // 2], cos_sin[pos, None, DIM // 2:]
    lo, hi = x[..., :DIM // 2].float(), x[..., DIM // 2:].float()
    a, b, d, e = lo * c, hi * sn, hi * c, lo * sn
    return torch.cat([a - b, d + e], -1).to(torch.bfloat16)


def _encode(x, scale):
    inv = torch.tensor(scale, dtype=torch.float32).reciprocal().to(DEVICE)
    return (x.float() * inv).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)


def _write(s):
    """The new tokens into the pools, by subscripts."""
    cu, start = s["cu_new"].tolist(), s["start"].tolist()
    for b in range(len(start)):
        n = cu[b + 1] - cu[b]
        pos = start[b] + torch.arange(n, device=DEVICE)
        ids = s["kv_w"].block_table[b].long()[pos // PAGE]
        k, v = s["k_new"][cu[b]:cu[b + 1]], s["v_new"][cu[b]:cu[b + 1]]
        if s["cos_sin"] is not None:
            k = _rope(k, pos, s["cos_sin"])
        if s["case"]["fp8"]:
            k, v = _encode(k, K_SCALE), _encode(v, V_SCALE)
        s["k_pool"][ids, :, pos % PAGE, :] = k
        s["v_pool"][ids, :, :, pos % PAGE] = v


def exact(case, seed):
    s, c = prepare(case, seed), case
    if c["kind"] == "logprob":
        h, t = s["h"].double(), s["targets"].long()
        parts, target = [], torch.zeros(c["N"], dtype=torch.float64, device=DEVICE)
        for v in range(0, c["V"], 16384):
            z = h @ s["W"][v:v + 16384].double().t()
            parts.append(z.logsumexp(1))
            mine = (t >= v) & (t < v + z.shape[1])
            target[mine] = z[mine].gather(1, (t[mine] - v)[:, None])[:, 0]
        lse = torch.stack(parts).logsumexp(0)
        return target - lse, lse
    if "k_new" in s:
        _write(s)
    got_d, got_a = None, None
    if "q" in s:
        out, lse = [], []
        for b, n in enumerate(s["kv_lens"].tolist()):
            k, v = _row_kv(s, s["kv"].block_table[b], n)
            o, m = _attend(s["q"][b:b + 1], k, v, n - 1)
            out.append(o)
            lse.append(m)
        got_d = torch.cat(out), torch.cat(lse)
    if "q_a" in s:
        out, lse = [], []
        cu, ctx = s["cu_q"].tolist(), s["ctx"].tolist()
        for b in range(len(ctx)):
            T = cu[b + 1] - cu[b]
            k, v = _row_kv(s, s["kv_a"].block_table[b], ctx[b] + T)
            q = s["q_a"][cu[b]:cu[b + 1]]
            if s.get("cos_sin") is not None:
                q = _rope(q, ctx[b] + torch.arange(T, device=DEVICE), s["cos_sin"])
            o, m = _attend(q, k, v, ctx[b])
            out.append(o)
            lse.append(m)
        got_a = torch.cat(out), torch.cat(lse)
    if c["kind"] in ("decode", "shared"):
        return got_d
    if c["kind"] == "append":
        return got_a
    # the pools hold bits: nothing to compute in 64 bits
    if c["kind"] == "append_write":
        return (*got_a, None, None)
    return (got_d[0], got_a[0], got_d[1], got_a[1], None, None)
