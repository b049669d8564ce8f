"""What this library is timed on: one pass of each of its calls as a decoding loop makes them.

A pass is one call, or the calls of one iteration in order, through the package's public
entry points on buffers that the program keeps.  The kinds:

  pass    one LogitPass.logit_pass call: confidence, draft length and verification of a
          dense draft (cmsd_logit_pass)
  fused   one LogitPass.logit_pass_fused call: the same iteration in one launch
  calls   LogitPass.run on packed target rows: cmsd_confidence, cmsd_draft_len and
          cmsd_verify, the verifier having scored k_b + 1 positions per sequence
  sample  one drafting position: cmsd_confidence and cmsd_draft_sample on its rows
  var     cmsd_confidence_var

Rows follow the recipes of the benchmark's workloads (normal rows of a log-uniform
scale, Zipf rows, and a mix of near-one-hot, Zipf and flat rows); they are made on the
GPU, so a case takes its numbers from torch's generator and not from numpy's.
"""
from __future__ import annotations

import math

import torch

from paper_2508_15371_amd import cmsd, pipeline

DEV = "cuda:0"
MODES = {"standard": cmsd.CMSD_MODE_STANDARD, "cm": cmsd.CMSD_MODE_CM, "greedy": cmsd.CMSD_MODE_GREEDY}
CHUNK = 1 << 26          # logits made at a time
MOST_BYTES = 2.3e9       # logits of a drawn case
# mean draft length over k_max of packed sequences under the default parameters: the
# rows' mean confidence (a few per cent either way per recipe and vocabulary)
PACKED_SHARE = {"normal": 0.32, "zipf": 0.5, "mixed": 0.55}


def _case(name, kind, batch, k_max, vocab, dtype="bf16", rows="normal", mode="cm", adaptive=False, masked=False, pad=0):
    return {"name": name, "kind": kind, "batch": batch, "k_max": k_max, "vocab": vocab, "dtype": dtype, "rows": rows,
            "mode": mode, "adaptive": adaptive, "masked": masked, "pad": pad}


def listed():
    return [
        # single-stream decoding: what one user waits for in every iteration
        _case("one_sequence", "pass", 1, 8, 32000),
        # the smallest call: a toy model's vocabulary in one launch, latency only
        _case("tiny_one_launch", "fused", 1, 4, 1024, "f32"),
        # a lightly loaded server
        _case("small_batch", "pass", 8, 8, 32000),
        # an iteration of the package's own decoder: fp32 logits, 16 sequences, packed
        # rows, the paper's deterministic rule
        _case("decoder_f32_greedy", "calls", 16, 8, 32000, "f32", mode="greedy"),
        # one drafting position of that decoder: confidence, then a sampled draft
        _case("decoder_f32_draft", "sample", 16, 1, 32000, "f32"),
        # an odd vocabulary: no two rows share their 16-byte phase
        _case("odd_vocab", "pass", 64, 8, 50257, rows="zipf"),
        # the largest vocabulary in use, a mid-size batch
        _case("wide_vocab", "pass", 64, 8, 152064),
        # the benchmark's default: a full server
        _case("large_batch", "pass", 256, 16, 128256, rows="mixed"),
        # the same rows from a model that hands out fp32 logits
        _case("large_batch_f32", "pass", 256, 16, 128256, "f32", rows="mixed"),
        # many sequences whose verifier scored only the k_b + 1 adaptive positions,
        # under a decoding constraint: masked tokens and a padded vocabulary
        _case("packed_masked", "calls", 512, 16, 32000, masked=True),
        # one drafting position of a full server: 512 sampled drafts
        _case("draft_512", "sample", 512, 1, 128256, rows="mixed"),
        # the logit-variance proxy over a whole draft
        _case("variance", "var", 256, 16, 128256, rows="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(("pass", "pass", "pass", "calls", "calls", "sample", "var", "fused"))
        batch, k_max = _log_int(rng, 1, 512), rng.randint(2, 16)
        vocab = _log_int(rng, 16000, 152064)
        if rng.random() < 0.6:
            vocab -= vocab % 64              # most vocabularies are padded to a round size
        if kind == "sample":
            k_max = 1
        if kind == "fused":                  # for a few hundred rows
            batch, k_max, vocab = _log_int(rng, 1, 8), rng.randint(2, 8), _log_int(rng, 1000, 32000)
        c = {"kind": kind, "batch": batch, "k_max": k_max, "vocab": vocab,
             "dtype": "f32" if rng.random() < 0.3 else "bf16", "rows": rng.choice(("normal", "zipf", "mixed")),
             "mode": "cm", "adaptive": False, "masked": rng.random() < 0.25,
             "pad": rng.choice((0, 0, 0, rng.randint(1, 128)))}
        if kind in ("pass", "calls", "fused"):
            c["mode"] = rng.choice(("cm", "cm", "cm", "standard", "greedy"))
        if kind in ("pass", "fused"):
            c["adaptive"] = rng.random() < 0.3
        if _dense_rows(c) * vocab * _size(c) <= MOST_BYTES:
            return c


def _size(c):
    return 4 if c["dtype"] == "f32" else 2


def _verifies(c):
    return c["kind"] in ("pass", "calls", "fused")


def _dense_rows(c):
    return c["batch"] * (2 * c["k_max"] + 1) if _verifies(c) else c["batch"] * c["k_max"]


# ---------------------------------------------------------------------------- inputs
def _scale(g, n, lo, hi):
    return lo + (hi - lo) * torch.rand(n, 1, generator=g, device=DEV)


def _normal(g, n, v):
    return torch.randn(n, v, generator=g, device=DEV)


def _base(c, g, n):
    """n rows of the case's recipe before their last noise, and that noise's scale."""
    v = c["vocab"]
    if c["rows"] == "normal":
        return torch.exp(_scale(g, n, math.log(0.3), math.log(10.0))) * _normal(g, n, v), 0.0
    # a * ln(rank^-1.1), the ranks uniform over the vocabulary
    z = torch.rand(n, v, generator=g, device=DEV).mul_(v - 1).add_(1).log_().mul_(_scale(g, n, -3.3, -0.55))
    if c["rows"] == "mixed":                 # a third each: near one-hot, Zipf, flat
        kind = torch.randint(0, 3, (n, 1), generator=g, device=DEV)
        top = torch.randint(0, v, (n, 1), generator=g, device=DEV)
        z.mul_((kind == 1).float())
        z.scatter_add_(1, top, 15.0 * (kind == 0).float())
        return z, 0.3
    return z, 0.2


def _logits(c, n):
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    return torch.empty((n, c["vocab"] + c["pad"]), dtype=dt, device=DEV).zero_()[:, :c["vocab"]]


def _mask(c, g, n):
    """The last 128 tokens, and 3 % of the others."""
    m = torch.rand(n, c["vocab"], generator=g, device=DEV) < 0.03
    m[:, -128:] = True
    return m


def _inputs(c, seed):
    """Drafter rows [B*K, V], dense target rows [B*(K+1), V], drafted ids (samples of the
    drafter rows) and uniforms."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    B, K, V = c["batch"], c["k_max"], c["vocab"]
    draft = _logits(c, B * K)
    target = _logits(c, B * (K + 1)) if _verifies(c) else None
    drafted = torch.empty(B * K, dtype=torch.int32, device=DEV)
    step = max(1, CHUNK // (K * V))
    for b0 in range(0, B, step):
        nb = min(step, B - b0)
        z, noise = _base(c, g, nb * K)
        d = draft[b0 * K:(b0 + nb) * K]
        d.copy_(z + noise * _normal(g, nb * K, V) if noise else z)
        mask = _mask(c, g, nb * K) if c["masked"] else None
        if mask is not None:
            d.masked_fill_(mask, -math.inf)
        drafted[b0 * K:(b0 + nb) * K] = torch.argmax(
            d.float() - torch.empty(nb * K, V, device=DEV).exponential_(generator=g).log_(), 1).int()
        if target is None:
            continue
        # the verifier agrees with the drafter up to noise; one Zipf row in five does not
        if c["rows"] == "normal":
            t = z * (1 + 0.1 * _normal(g, nb * K, V)) + 0.3 * _normal(g, nb * K, V)
        else:
            t = z + (0.5 if c["rows"] == "mixed" else noise) * _normal(g, nb * K, V)
            if c["rows"] == "zipf":
                far = torch.rand(nb * K, 1, generator=g, device=DEV) < 0.2
                t = torch.where(far, t.roll(V // 3, 1), t)
        if mask is not None:
            t.masked_fill_(mask, -math.inf)
        t3 = target[b0 * (K + 1):(b0 + nb) * (K + 1)].unflatten(0, (nb, K + 1))
        t3[:, :K] = t.view(nb, K, V).to(target.dtype)
        z, noise = _base(c, g, nb)
        z = z + noise * _normal(g, nb, V)
        if c["masked"]:
            z.masked_fill_(_mask(c, g, nb), -math.inf)
        t3[:, K] = z.to(target.dtype)
    unif = torch.randint(0, 1 << 24, (B * (K + 1) if _verifies(c) else B * K,), generator=g, device=DEV).float() * 2.0 ** -24
    return draft, target, drafted, unif


def _pack(c, k, off, rows):
    """The packed form of dense per-position rows: positions 0 .. k_b - 1, then the last."""
    K = c["k_max"]
    p = torch.arange(int(off[-1]), device=DEV)
    b = torch.searchsorted(off[1:].long().contiguous(), p, right=True)
    i = p - off.long()[b]
    src = b * (K + 1) + torch.where(i < k.long()[b], i, torch.full_like(i, K))
    if rows.dim() == 1:
        return rows[src]
    out = _logits(c, src.numel())
    out.copy_(rows[src])
    return out


def _stat_views(stats):
    """The record's fields as the types they hold."""
    i = stats.view(torch.int32)
    return {"max_logit": stats[:, 0], "sum_exp": stats[:, 1], "entropy": stats[:, 2], "margin_soft": stats[:, 3],
            "margin_logit": stats[:, 4], "conf": stats[:, 5], "top1": i[:, 6], "flags": i[:, 7]}


def _target_views(stats):
    i = stats.view(torch.int32)
    return {"max_logit": stats[:, 0], "sum_exp": stats[:, 1], "n_greater": i[:, 2], "accept": i[:, 3], "top1": i[:, 4]}


def prepare(case, seed):
    c = case
    B, K, V = c["batch"], c["k_max"], c["vocab"]
    draft, target, drafted, unif = _inputs(c, seed)
    if c["kind"] in ("sample", "var"):
        s = {"kind": c["kind"], "rows": draft, "stats": torch.zeros((B * K, 8), dtype=torch.float32, device=DEV)}
        if c["kind"] == "var":
            s["out"] = torch.zeros(B * K, dtype=torch.float32, device=DEV)
        else:
            s["out"] = torch.zeros(B * K, dtype=torch.int32, device=DEV)
            s["unif"] = unif
            s["ws"] = torch.empty((cmsd.cmsd_draft_sample_workspace_bytes(B * K, V) + 7) // 8, dtype=torch.float64, device=DEV)
        s["outputs"] = {"stats": _stat_views(s["stats"]), "out": s["out"]}
        return s
    prm = pipeline.Params(mode=MODES[c["mode"]])
    packed = c["kind"] == "calls"
    if packed:
        # the program knows the draft lengths when it has the target score the drafts
        lp = pipeline.LogitPass(B, K, V, DEV, prm, dense=False)
        lp.confidence(draft)
        lp.draft_len()
        target, unif = _pack(c, lp.k, lp.off, target), _pack(c, lp.k, lp.off, unif)
    lp = pipeline.LogitPass(B, K, V, DEV, prm, dense=not packed)
    for t in (lp.stats, lp.tstats, lp.k, lp.off, lp.n_acc, lp.next_tok):
        t.zero_()
    if c["kind"] == "fused":
        lp.logit_pass_fused(draft, target, drafted, unif, adaptive=c["adaptive"])   # its workspace, allocated once
    out = {"stats": _stat_views(lp.stats), "k": lp.k, "target": _target_views(lp.tstats), "n_acc": lp.n_acc,
           "next": lp.next_tok}
    if packed:
        out["off"] = lp.off
    return {"kind": c["kind"], "lp": lp, "draft": draft, "target": target, "drafted": drafted, "unif": unif,
            "adaptive": c["adaptive"], "outputs": out}


def run(state):
    s = state
    kind = s["kind"]
    if kind == "pass":
        s["lp"].logit_pass(s["draft"], s["target"], s["drafted"], s["unif"], adaptive=s["adaptive"])
    elif kind == "fused":
        s["lp"].logit_pass_fused(s["draft"], s["target"], s["drafted"], s["unif"], adaptive=s["adaptive"])
    elif kind == "calls":
        s["lp"].run(s["draft"], s["target"], s["drafted"], s["unif"])
    elif kind == "sample":
        cmsd.cmsd_confidence(s["rows"], s["stats"])
        cmsd.cmsd_draft_sample(s["rows"], s["stats"], s["unif"], drafted=s["out"], workspace=s["ws"])
    else:
        cmsd.cmsd_confidence_var(s["rows"], s["stats"], s["out"])
    return s["outputs"]


def work(case):
    """Every logit read once, the records written once.  Per logit: the exponent's
    multiply-add, the exponential, a sum and a comparison; one more multiply-add for the
    entropy of a drafter row."""
    c = case
    B, K = c["batch"], c["k_max"]
    d = B * K
    t = 0
    if _verifies(c):
        t = B * (K + 1) if c["kind"] != "calls" else int(B * (1 + PACKED_SHARE[c["rows"]] * K))
    return {"bytes": float((d + t) * (c["vocab"] * _size(c) + 32) + 8 * (d + t) + 12 * B),
            "flops": float(c["vocab"] * (7 * d + 5 * t))}


def tolerance(case):
    # against 64 bits, over these cases: up to 1.1e-6 in the norm (the softmax margin; the
    # others 2e-7 and less).  Whole numbers follow thresholds and cumulative sums of up to
    # 152064 terms: 1 of 512 samples fell beside the 64-bit one.
    return {"rel": 5e-6, "max": 1e-4, "differ": 0.008}


# ---------------------------------------------------------------------------- in 64 bits
def _row_stats(z):
    """The record of fp64 rows: max, sum of exponentials, entropy, margins, argmax, masks."""
    top = torch.topk(z, 2, 1).values
    m, z2 = top[:, 0], top[:, 1]
    x = z - m[:, None]
    e = torch.exp(x)
    a = e.sum(1)
    ent = torch.log1p(a - 1) - torch.where(e > 0, e * x, torch.zeros_like(e)).sum(1) / a
    one = torch.isinf(z2)
    soft = torch.where(one, 1 / a, -torch.expm1(z2 - m) / a)
    margin = torch.where(one, torch.full_like(m, math.inf), m - z2)
    v = z.shape[1]
    third = float(torch.tensor(1 / 3, dtype=torch.float32))
    conf = third * (1 - ent / math.log(v)) + third * torch.sigmoid(margin) + third * torch.clamp(soft / (1 - 1 / v), max=1.0)
    first = (z == m[:, None]).int().argmax(1).int()
    return {"max_logit": m, "sum_exp": a, "entropy": ent, "margin_soft": soft, "margin_logit": margin, "conf": conf,
            "top1": first, "flags": torch.isinf(z).any(1).int()}


def _by_chunks(rows, f):
    step = max(1, (1 << 25) // rows.shape[1])
    parts = [f(r0, rows[r0:r0 + step].double()) for r0 in range(0, rows.shape[0], step)]
    return {k: torch.cat([p[k] for p in parts]) for k in parts[0]}


def _variance(z):
    fin = torch.isfinite(z)
    n = fin.sum(1)
    mean = torch.where(fin, z, torch.zeros_like(z)).sum(1) / n
    return (torch.where(fin, z - mean[:, None], torch.zeros_like(z)) ** 2).sum(1) / n


def _pick(w, u):
    """Smallest index whose cumulative weight passes u of the row's total."""
    c = torch.cumsum(w, 1)
    y = torch.searchsorted(c, (u.double()[:, None] * c[:, -1:]), right=True)[:, 0]
    last = w.shape[1] - 1 - (w.flip(1) > 0).int().argmax(1)
    return torch.minimum(y, last).int()


def exact(case, seed):
    c = case
    B, K, V = c["batch"], c["k_max"], c["vocab"]
    draft, target, drafted, unif = _inputs(c, seed)
    if c["kind"] == "var":
        out = _by_chunks(draft, lambda r0, z: {**_row_stats(z), "var": _variance(z)})
        var = out.pop("var")
        return {"stats": out, "out": var}
    if c["kind"] == "sample":
        out = _by_chunks(draft, lambda r0, z: {**_row_stats(z), "y": _pick(torch.exp(z - z.amax(1, keepdim=True)),
                                                                          unif[r0:r0 + z.shape[0]])})
        y = out.pop("y")
        return {"stats": out, "out": y}
    st = _by_chunks(draft, lambda r0, z: _row_stats(z))
    conf32 = st["conf"].float().double().view(B, K)         # as stored
    k = torch.clamp(torch.floor(conf32.mean(1) * K), 1, K).int()
    off = torch.zeros(B + 1, dtype=torch.int32, device=DEV)
    off[1:] = torch.cumsum(k + 1, 0).int()
    packed = c["kind"] == "calls"
    kv = k.long() if packed or c["adaptive"] else torch.full((B,), K, device=DEV)
    # every position dense: row b*(K+1)+i; the packed layout keeps the last row at i = K
    row = torch.arange(B * (K + 1), device=DEV)
    b, i = row // (K + 1), row % (K + 1)
    greedy, beta = c["mode"] == "greedy", 3
    y = torch.where(i < K, drafted.long()[(b * K + i).clamp(max=B * K - 1)], torch.zeros_like(i))

    def target_rows(r0, z):
        m = z.amax(1)
        zy = z.gather(1, y[r0:r0 + z.shape[0], None])
        return {"m": m, "a": torch.exp(z - m[:, None]).sum(1), "zy": zy[:, 0], "n": (z > zy).sum(1),
                "top1": (z == m[:, None]).int().argmax(1)}

    tr = _by_chunks(target, target_rows)
    at = (b * K + i.clamp(max=K - 1))
    zd = torch.where(i < K, draft[at, y].double(), torch.zeros_like(tr["zy"]))
    lpt = tr["zy"] - tr["m"] - torch.log(tr["a"])
    lpd = zd - st["max_logit"][at] - torch.log(st["sum_exp"][at])
    stoch = (torch.log(unif.double()) < lpt - lpd) & torch.isfinite(lpt)
    count = c["mode"] != "standard"
    tau = float(torch.tensor(0.1, dtype=torch.float32)) + (1 - st["conf"].float().double()[at])
    gate = (tr["n"] < beta) & (tr["m"] - tr["zy"] <= tau) if count else torch.zeros_like(stoch)
    acc = ((y == tr["top1"]) | gate) if greedy else (stoch | gate)
    ngt = tr["n"].clamp(max=beta).int() if count else torch.zeros_like(i).int()
    rej = (~acc & (i < kv[b])).view(B, K + 1)
    n_acc = torch.where(rej.any(1), rej.int().argmax(1), kv)
    all_in = n_acc == kv
    # the packed layout keeps the row after the last draft at dense slot K
    final = torch.arange(B, device=DEV) * (K + 1) + torch.where(all_in & packed, torch.full_like(kv, K), n_acc)
    if greedy:
        nxt = tr["top1"][final].int()
    else:
        uf = unif[torch.arange(B, device=DEV) * (K + 1) + (torch.full_like(kv, K) if packed else kv)]
        parts = []
        step = max(1, (1 << 25) // V)
        for b0 in range(0, B, step):
            s = slice(b0, min(B, b0 + step))
            f = final[s]
            pt = torch.exp(target[f].double() - tr["m"][f][:, None]) / tr["a"][f][:, None]
            dr = torch.arange(B, device=DEV)[s] * K + n_acc[s].clamp(max=K - 1)
            pd = torch.exp(draft[dr].double() - st["max_logit"][dr][:, None]) / st["sum_exp"][dr][:, None]
            q = torch.where(all_in[s][:, None], pt, torch.clamp(pt - pd, min=0))
            q = torch.where(q.sum(1, keepdim=True) > 0, q, pt)
            parts.append(_pick(q, uf[s]))
        nxt = torch.cat(parts)
    last = (i == kv[b]) | (i == K)
    ts = {"max_logit": tr["m"], "sum_exp": tr["a"],
          "n_greater": torch.where(last, torch.full_like(ngt, -1), ngt),
          "accept": torch.where(last, torch.full_like(ngt, -1), acc.int()),
          "top1": tr["top1"].int() if greedy else torch.full_like(ngt, -1)}
    out = {"stats": st, "k": k, "target": ts, "n_acc": n_acc.int(), "next": nxt}
    if packed:                               # in records for every position, the rest unwritten
        out["target"] = {n: torch.cat([_pack(c, k, off, v), v.new_zeros(B * (K + 1) - int(off[-1]))]) for n, v in ts.items()}
        out["off"] = off
    return out
