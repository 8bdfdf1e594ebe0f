"""The work that users of this library have it do, as timed cases.

A video diffusion transformer calls the library once per attention layer and
denoising step: a mask prediction (with or without a new fit of the MOD model)
and a block-sparse attention forward over the predicted lists; the first steps
run dense attention; with the attention statistic each re-anchor step ends in
an update of that statistic.  Each case below is one of these calls (or the
whole layer step), through the public binding, on inputs resident in device
memory, with the handle, the lists' memory and the attention workspace that
such a program keeps.

Kinds of a case:
  attention  the sparse forward over lists predicted for its inputs
  dense      the forward over full lists (a warm-up step)
  predict    the mask prediction; "anchor": with a new fit (pool, block mass,
             fit, extrapolate, select), else extrapolate and select only
  step       a re-anchoring prediction and the attention over its lists
  update     the attention statistic of a dense step, its fit, and the
             prediction of the next step
"""
import math

import numpy as np
import torch

import paper_2601_11641_amd as M

HYPER_TAU_E = 0.0
DEVICE = "cuda"


def _case(kind, H, frames, hs, ws, d=128, block=128, B=1, text=0, mode="topk", amount=0.25, anchor=False, name=None):
    """amount: TOPK density, MASS mass, or PATTERN patterns as a share of the
    video blocks."""
    c = dict(kind=kind, B=B, H=H, frames=frames, hs=hs, ws=ws, d=d, block=block, text=text, mode=mode,
             amount=amount, anchor=anchor)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call in earnest: a whole layer step of a toy layer
        # (2 heads, 64-wide, 64-token blocks, 1024 tokens); latency only.
        _case("step", 2, 4, 16, 16, d=64, block=64, amount=0.3, name="tiny-step"),
        # A low-resolution preview layer (8 heads, 8192 tokens): one step's
        # prediction with a new fit, and its attention.
        _case("predict", 8, 8, 32, 32, mode="mass", amount=0.85, anchor=True, name="small-reanchor"),
        _case("attention", 8, 8, 32, 32, amount=0.25, name="small-attention"),
        # A re-anchor step's prediction at 720p, HunyuanVideo-shaped (24
        # heads, 33 latent frames of 45x80; frames straddle blocks, short
        # tail block), cumulative-mass budget.
        _case("predict", 24, 33, 45, 80, mode="mass", amount=0.75, anchor=True, name="hunyuan-reanchor"),
        # The steps between re-anchors (nine of ten at the usual interval):
        # extrapolation and selection only, Wan-shaped 720p layer.
        _case("predict", 40, 21, 45, 80, amount=0.25, name="wan-predict"),
        # The pattern-level budget (whole diagonals and columns kept).
        _case("predict", 24, 33, 45, 80, mode="pattern", amount=0.5, name="hunyuan-pattern"),
        # Sparse attention of the two 720p layers: the mass budget of the
        # benchmark, and the sparsest setting of the density sweep.
        _case("attention", 24, 33, 45, 80, mode="mass", amount=0.75, name="hunyuan-attention"),
        _case("attention", 40, 21, 45, 80, amount=0.05, name="wan-sparse"),
        # A dense warm-up step on one GPU's share of the heads (3 of 24).
        _case("dense", 3, 33, 45, 80, name="hunyuan-dense-share"),
        # 64-wide heads, two sequences at once (guided and unguided), text
        # after the video (CogVideoX-shaped: 30 heads, 32x40 per frame).
        _case("attention", 30, 23, 32, 40, d=64, B=2, text=226, amount=0.2, name="d64-text"),
        # The smaller block of the block-size comparison, on the layer of the
        # paper's operation counts (35,200 tokens with the text).
        _case("attention", 24, 21, 32, 52, block=64, text=256, amount=0.2, name="block64-text"),
        # The attention statistic at a dense step, one GPU's share of heads.
        _case("update", 3, 33, 45, 80, mode="mass", amount=0.75, name="hunyuan-update-share"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case: both head widths and block sizes, 1 to 40 heads, 512 to
    118,800 tokens, aligned and straddling frames, with and without text, all
    budgets; no dearer than the dearest listed case."""
    while True:
        kind = rng.choice(["attention", "attention", "attention", "dense", "predict", "predict", "predict", "step",
                           "update"])
        d, block = rng.choice([(128, 128), (128, 128), (64, 128), (128, 64), (64, 64)])
        B = rng.choice([1, 1, 2])
        H = round(_log(rng, 1, 40))
        frames = rng.randint(2, 33)
        hs, ws = rng.randint(8, 45), rng.randint(8, 80)
        text = rng.choice([0, 0, rng.randint(1, 512)])
        mode = rng.choice(["topk", "topk", "mass", "pattern"])
        amount = _log(rng, 0.05, 0.7) if mode == "topk" else rng.uniform(0.5, 0.95) if mode == "mass" else _log(rng, 0.1, 1.5)
        c = _case(kind, H, frames, hs, ws, d, block, B, text, mode, round(amount, 4),
                  anchor=kind == "predict" and rng.random() < 0.5)
        s = _sizes(c)
        if s["L"] < 512 or s["n"] < 4 or s["n"] > 1300 or B * H * s["n"] ** 2 > 25_000_000:
            continue
        if kind in ("dense", "update"):
            c["mode"], c["amount"] = ("mass", 0.75) if kind == "update" else ("topk", 0.25)
        if work(c)["flops"] > 8e12:
            continue
        return c


def _sizes(c):
    Lv = c["frames"] * c["hs"] * c["ws"]
    L = Lv + c["text"]
    return {"Lv": Lv, "L": L, "n": -(-L // c["block"]), "nv": -(-Lv // c["block"]),
            "tb0": Lv // c["block"] if c["text"] else -(-L // c["block"])}


# ---------------------------------------------------------------- inputs

def _axis(count, dims, omega, gen):
    w = omega * 0.7 ** torch.arange(dims // 2, device=DEVICE, dtype=torch.float64)
    ang = torch.arange(count, device=DEVICE, dtype=torch.float64)[:, None] * w
    return math.sqrt(2.0) * 3.0 * torch.cat([ang.sin(), ang.cos()], 1)


def _layer(c, gen):
    """Q, K, V of one synthetic layer, bf16 [B, H, L, d]: rotated sinusoidal
    position features plus noise; heads local in time, local in space, or
    global with sink keys, a third each; text tokens unstructured."""
    s, d = _sizes(c), c["d"]
    B, H, Lv, L = c["B"], c["H"], s["Lv"], s["L"]
    q = torch.empty((B, H, L, d), dtype=torch.bfloat16, device=DEVICE)
    k, v = torch.empty_like(q), torch.empty_like(q)

    def randn(*shape, dtype=torch.float32):
        return torch.randn(*shape, device=DEVICE, dtype=dtype, generator=gen)

    dt = d // 4
    ds = (d - dt) // 2
    kinds = torch.arange(H) % 3
    spread = torch.exp(torch.rand((B, H, 2), device=DEVICE, generator=gen) - 0.5).cpu().tolist()
    for b in range(B):
        for h in range(H):
            wt, wsp = [(1.0, 0.05), (0.05, 1.0), (0.05, 0.05)][int(kinds[h])]
            rot = torch.linalg.qr(randn(d, d, dtype=torch.float64))[0]
            at = 0.7 * _axis(c["frames"], dt, wt * spread[b][h][0], gen) @ rot[:dt]
            ay = 0.7 * _axis(c["hs"], ds, wsp * spread[b][h][1], gen) @ rot[dt:dt + ds]
            ax = 0.7 * _axis(c["ws"], ds, wsp * spread[b][h][1], gen) @ rot[dt + ds:]
            base = (at[:, None, None] + ay[:, None] + ax).reshape(Lv, d).float()
            hq = base + 0.3 * randn(Lv, d)
            hk = base + 0.3 * randn(Lv, d)
            if int(kinds[h]) == 2:
                g = randn(d)
                amp = math.sqrt(4.0 * math.sqrt(d)) * g / g.norm()
                hq += amp
                nv = s["nv"]
                sinks = torch.randperm(nv, device=DEVICE, generator=gen)[:max(1, round(0.02 * nv))]
                on = torch.zeros(nv, dtype=torch.bool, device=DEVICE)
                on[sinks] = True
                on = on.repeat_interleave(c["block"])[:Lv] & (torch.rand(Lv, device=DEVICE, generator=gen) < 0.5)
                hk += on[:, None] * amp
            q[b, h, :Lv], k[b, h, :Lv] = hq.bfloat16(), hk.bfloat16()
            if L > Lv:
                rms = float(base.square().mean() + 0.09) ** 0.5
                q[b, h, Lv:], k[b, h, Lv:] = (rms * randn(L - Lv, d)).bfloat16(), (rms * randn(L - Lv, d)).bfloat16()
            v[b, h] = randn(L, d).bfloat16()
    return q, k, v


def _drifted(x, gen):
    """The same activations some denoising steps earlier."""
    y = torch.empty_like(x)
    for b in range(x.shape[0]):
        for h in range(x.shape[1]):
            noise = torch.randn(x.shape[2:], device=DEVICE, generator=gen)
            y[b, h] = (0.97 * x[b, h].float() + 0.5 * noise).bfloat16()
    return y


def _budget(c):
    if c["mode"] == "topk":
        return M.make_budget("topk", density=c["amount"])
    if c["mode"] == "mass":
        return M.make_budget("mass", mass=c["amount"])
    nv = _sizes(c)["nv"]
    return M.make_budget("pattern", patterns=max(1, min(3 * nv - 1, round(c["amount"] * nv))))


def prepare(case, seed):
    c, kind = case, case["kind"]
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    s = _sizes(c)
    B, H, n = c["B"], c["H"], s["n"]
    shape = M.make_shape(B, H, s["L"], c["d"], c["block"], c["hs"] * c["ws"], c["text"])
    q, k, v = _layer(c, gen)
    st = {"kind": kind, "shape": shape, "q": q, "k": k, "v": v, "budget": _budget(c), "step": 0,
          # unwritten list slots (past a row's count) hold -1
          "idx": torch.full((B, H, n, n), -1, dtype=torch.int32, device=DEVICE),
          "cnt": torch.zeros((B, H, n), dtype=torch.int32, device=DEVICE),
          "o": torch.empty_like(q), "lse": torch.empty((B, H, s["L"]), dtype=torch.float32, device=DEVICE)}
    st["ws_bytes"] = M.mod_attn_workspace_bytes(shape)
    st["ws"] = torch.empty(st["ws_bytes"], dtype=torch.uint8, device=DEVICE)
    if kind in ("dense", "update"):
        st["all_idx"] = torch.arange(n, dtype=torch.int32, device=DEVICE).expand(B, H, n, n).contiguous()
        st["all_cnt"] = torch.full((B, H, n), n, dtype=torch.int32, device=DEVICE)
    if kind == "dense":
        st["idx"], st["cnt"] = st["all_idx"], st["all_cnt"]
        return st
    anchored = c["anchor"] or kind == "step"
    stats = M.Stats(shape, M.make_params(warmup_m=2, delta_t=1 if anchored else 0, tau_e=HYPER_TAU_E,
                                         statistic=1 if kind == "update" else 0))
    st["stats"] = stats
    # two warm-up anchors from earlier activations
    if kind == "update":
        for step in (1, 2):
            q0, k0 = _drifted(q, gen), _drifted(k, gen)
            _attend(st, q0, k0, st["all_idx"], st["all_cnt"])
            M.mod_update_stats(stats.handle, q0, k0, st["lse"], st["all_idx"], st["all_cnt"], step)
        _attend(st, q, k, st["all_idx"], st["all_cnt"])
        st["step"] = 3
    elif kind == "attention":
        M.mod_collect_stats(stats.handle, q, k, 1)
        M.mod_predict_block_mask(stats.handle, q, k, 2, st["budget"], st["idx"], st["cnt"])
        del st["stats"]
    else:
        # the second anchor is far from the first, so that the extrapolation
        # of the many passes that follow stays in a moderate range
        M.mod_collect_stats(stats.handle, _drifted(q, gen), _drifted(k, gen), 1)
        M.mod_collect_stats(stats.handle, q, k, 1001)
        st["step"] = 1002
    return st


def _attend(st, q, k, idx, cnt):
    M.mod_block_sparse_attn_fwd(st["shape"], q, k, st["v"], idx, cnt, 0.0, st["o"], st["lse"], st["ws"],
                                st["ws_bytes"])


def run(st):
    kind = st["kind"]
    if kind in ("attention", "dense"):
        _attend(st, st["q"], st["k"], st["idx"], st["cnt"])
        return {"o": st["o"], "lse": st["lse"]}
    if kind == "update":
        M.mod_update_stats(st["stats"].handle, st["q"], st["k"], st["lse"], st["all_idx"], st["all_cnt"], st["step"])
        st["step"] += 1
    M.mod_predict_block_mask(st["stats"].handle, st["q"], st["k"], st["step"], st["budget"], st["idx"], st["cnt"])
    st["step"] += 1
    if kind == "step":
        _attend(st, st["q"], st["k"], st["idx"], st["cnt"])
        return {"idx": st["idx"], "cnt": st["cnt"], "o": st["o"], "lse": st["lse"]}
    return {"idx": st["idx"], "cnt": st["cnt"]}


# ---------------------------------------------------------------- what a pass cannot do without

def _kept_share(c):
    """Share of the video blocks kept per row: the density of TOPK, typical
    values of the other budgets on these inputs."""
    if c["kind"] == "dense":
        return 1.0
    if c["mode"] == "topk":
        return c["amount"]
    return 0.22 if c["mode"] == "mass" else min(1.0, 0.8 * c["amount"])


def work(case):
    c, s = case, _sizes(case)
    BH, L, n, nv, d, block = c["B"] * c["H"], s["L"], s["n"], s["nv"], c["d"], c["block"]
    keep = _kept_share(c)
    # every row keeps its video selection and the text, text rows keep all
    pairs = BH * (keep * s["Lv"] ** 2 + 2 * s["Lv"] * c["text"] + c["text"] ** 2)
    lists = BH * (keep * nv * nv + 2 * nv * (n - nv) + n) * 4
    attn_bytes = 4 * BH * L * d * 2 + BH * L * 4 + lists
    qk_bytes = 2 * BH * s["Lv"] * d * 2
    fit_flops = 2 * BH * nv * nv * d
    coeffs = 2 * BH * 3 * nv * 8
    if c["kind"] in ("attention", "dense"):
        return {"bytes": attn_bytes, "flops": 4 * d * pairs}
    if c["kind"] == "step":
        return {"bytes": attn_bytes + qk_bytes + lists, "flops": 4 * d * pairs + fit_flops}
    if c["kind"] == "update":
        return {"bytes": 2 * BH * L * d * 2 + BH * (L + n * n) * 4 + lists, "flops": 2 * d * BH * s["Lv"] * L}
    return {"bytes": lists + (qk_bytes if c["anchor"] else coeffs), "flops": fit_flops if c["anchor"] else BH * nv * nv}


def tolerance(case):
    # lists: a score within rounding of the boundary may fall on either side
    if case["kind"] in ("predict", "update"):
        return {"rel": 0.0, "differ": 1e-4}
    # bf16 probabilities and outputs: rel is four times the error against 64
    # bits; the largest single difference is a few bf16 steps of the output
    return {"rel": 1e-2, "max": 0.1, "differ": 1e-4}


# ---------------------------------------------------------------- 64-bit values

def _attention64(q, k, v, lists, block):
    """Softmax attention over lists[b][h][i] (ascending block numbers), with
    the log-sum-exp of every row, one query block at a time."""
    B, H, L, d = q.shape
    o = torch.zeros((B, H, L, d), dtype=torch.float64, device=q.device)
    lse = torch.full((B, H, L), -math.inf, dtype=torch.float64, device=q.device)
    pos = torch.arange(block, device=q.device)
    n = -(-L // block)
    for b in range(B):
        for h in range(H):
            q64, k64, v64 = q[b, h].double() / math.sqrt(d), k[b, h].double(), v[b, h].double()
            for i in range(n):
                js = lists(b, h, i)
                if js.numel() == 0:
                    continue
                rows = slice(i * block, min(L, (i + 1) * block))
                if js.numel() == n:
                    kk, vv = k64, v64
                else:
                    tok = (js.long()[:, None] * block + pos).reshape(-1)
                    dead = tok >= L   # past the end of a short tail block
                    tok = tok.clamp(max=L - 1)
                    kk, vv = k64[tok], v64[tok]
                sc = q64[rows] @ kk.t()
                if js.numel() != n:
                    sc.masked_fill_(dead, -math.inf)
                top = torch.logsumexp(sc, 1)
                o[b, h, rows] = torch.exp_(sc.sub_(top[:, None])) @ vv
                lse[b, h, rows] = top
    return o, lse


def _fit64(c, q, k):
    """Per head the coefficients (diagonals, columns, frame squares) of the
    minimum-norm least-squares fit to the pooled block mass."""
    s, bs, n = _sizes(c), c["block"], _sizes(c)["nv"]
    F, T = c["frames"], c["hs"] * c["ws"]
    size = torch.full((n,), float(bs), dtype=torch.float64, device=DEVICE)
    size[-1] = s["Lv"] - (n - 1) * bs
    block_of = torch.arange(s["Lv"], device=DEVICE) // bs

    def means(x):
        z = torch.zeros(x.shape[0], x.shape[1], n, x.shape[3], dtype=torch.float64, device=DEVICE)
        return z.index_add_(2, block_of, x[:, :, :s["Lv"]].double()) / size[:, None]

    logits = means(q) @ means(k).transpose(-1, -2).contiguous() / math.sqrt(c["d"])
    G = torch.softmax(logits + size.log(), -1)
    i, j = torch.meshgrid(torch.arange(n, device=DEVICE), torch.arange(n, device=DEVICE), indexing="ij")
    D = torch.zeros(n * n, 3 * n - 1 + F, dtype=torch.float64, device=DEVICE)
    cell = torch.arange(n * n, device=DEVICE)
    D[cell, (j - i + n - 1).reshape(-1)] = 1
    D[cell, 2 * n - 1 + j.reshape(-1)] = 1
    spans = [(f * T // bs, ((f + 1) * T - 1) // bs) for f in range(F)]
    for f, (lo, hi) in enumerate(spans):
        D[((i >= lo) & (i <= hi) & (j >= lo) & (j <= hi)).reshape(-1), 3 * n - 1 + f] = 1
    X = (torch.linalg.pinv(D) @ G.reshape(-1, n * n).t().contiguous()).t()
    return X.cpu().numpy(), spans


def _lists64(c, fits, spans):
    """Per head and row the selection of a re-anchoring step (TOPK or MASS)
    from its own fit fits[-1]; the gate from the warm-up fits fits[:2]."""
    s, n, F = _sizes(c), _sizes(c)["nv"], c["frames"]
    gate = np.min([x[:, 3 * n - 1:].mean(1) for x in fits[:2]], 0) > HYPER_TAU_E
    amount = float(np.float32(c["amount"]))
    out = []
    for h, x in enumerate(fits[-1]):
        rows = []
        for i in range(s["n"]):
            if i >= s["tb0"]:
                rows.append(np.arange(s["n"]))
                continue
            jj = np.arange(n)
            key = np.float32(n * (x[jj - i + n - 1] + x[2 * n - 1 + jj]))
            forced = jj == s["tb0"]
            for lo, hi in spans:
                if gate[h] and lo <= i <= hi:
                    forced |= (jj >= lo) & (jj <= hi)
            free = [j for j in np.lexsort((jj, -key)) if not forced[j]]
            if c["mode"] == "topk":
                keep = max(0, min(n, max(1, math.ceil(amount * n - 1e-6))) - int(forced.sum()))
            else:
                pos = np.maximum(key.astype(np.float64), 0)
                have, goal, keep = pos[forced].sum(), amount * pos.sum(), 0
                if not forced.any():
                    have, keep = pos[free[0]], 1
                while have < goal and keep < len(free):
                    have, keep = have + pos[free[keep]], keep + 1
            kept = np.sort(np.concatenate([jj[forced], np.array(free[:keep], dtype=np.int64)]))
            rows.append(np.concatenate([kept, np.arange(n, s["n"])]))
        out.append(rows)
    return out


def exact(case, seed):
    """The attention in 64 bits: over the lists that prepare() holds, or for a
    whole step over lists of this file's own fit (short sequences only: the
    explicit least-squares problem).  The lists themselves are whole numbers
    and have no such value."""
    c = case
    if c["kind"] in ("attention", "dense"):
        st = prepare(c, seed)
        cnt = st["cnt"].cpu().tolist()
        o, lse = _attention64(st["q"], st["k"], st["v"], lambda b, h, i: st["idx"][b, h, i, :cnt[b][h][i]], c["block"])
        return {"o": o, "lse": lse}
    if c["kind"] != "step" or c["mode"] == "pattern" or _sizes(c)["nv"] > 80:
        return None
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    q, k, v = _layer(c, gen)
    first, spans = _fit64(c, _drifted(q, gen), _drifted(k, gen))
    now, _ = _fit64(c, q, k)
    rows = _lists64(c, [first, now], spans)
    lists = [[torch.as_tensor(r, device=DEVICE) for r in head] for head in rows]
    o, lse = _attention64(q, k, v, lambda b, h, i: lists[b * c["H"] + h][i], c["block"])
    return {"idx": None, "cnt": None, "o": o, "lse": lse}
