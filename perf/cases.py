"""Measured cases of the denoising-step library: what a decoder built on it calls, through the
package's public entry points, over the range of sizes that it meets.

  step    eb_decode_step: one denoising iteration (attention layer, LM head with statistics, commit)
  attn    eb_block_attn, or eb_block_attn_dual where a suffix is cached as well
  lmhead  eb_lmhead_confidence, or eb_lmhead_features where the sampler needs the top-2 gap
  commit  the unmask rules on given statistics: threshold, router union (with its features), top-m
  lbs     eb_lbs_select over the generation window of every sequence

A case holds sizes only.  Ragged lengths come from the case's own "lens" number, so that the work
of a case is known without a GPU; every value comes from the seed given to prepare().
"""
from __future__ import annotations

import math
import random

import torch

import paper_2609_16450_amd as eb

# Attention heads, hidden size and vocabulary of the shapes that the workloads name, and of a
# small model with 64-wide heads.
LLADA = dict(hq=32, hkv=32, head_dim=128, hidden=4096, vocab=126464)
DREAM = dict(hq=28, hkv=4, head_dim=128, hidden=3584, vocab=152064)
TINY = dict(hq=4, hkv=4, head_dim=64, hidden=256, vocab=2048)
SMALL_HEADS = dict(hq=16, hkv=4, head_dim=64)


def _heads(m):
    return {k: m[k] for k in ("hq", "hkv", "head_dim")}


def _head(m):
    return {k: m[k] for k in ("hidden", "vocab")}


def listed():
    return [
        # The smallest call: a whole fp32 step of a toy model, as in unit tests and debugging;
        # latency and launches are everything.
        dict(name="step_tiny_f32_b1", kind="step", dtype="f32", batch=1, block_lo=32, block_hi=32,
             prefix_lo=96, prefix_hi=96, lens=1, tau=0.9, **TINY),
        # One user decoding with an 8B model and the base block of 32: a pass over the LM head.
        dict(name="step_llada8b_b1", kind="step", dtype="bf16", batch=1, block_lo=32, block_hi=32,
             prefix_lo=512, prefix_hi=512, lens=2, tau=0.9, **LLADA),
        # A served batch of equal blocks.
        dict(name="step_llada8b_b16", kind="step", dtype="bf16", batch=16, block_lo=64,
             block_hi=64, prefix_lo=1024, prefix_hi=1024, lens=3, tau=0.9, **LLADA),
        # The largest call: a full batch of blocks of very different lengths, grouped heads.
        dict(name="step_dream7b_b64", kind="step", dtype="bf16", batch=64, block_lo=16,
             block_hi=256, prefix_lo=4096, prefix_hi=4096, lens=5, tau=0.9, **DREAM),
        # One attention layer of a small model with 64-wide heads, a few sequences.
        dict(name="attn_d64_b8", kind="attn", dtype="bf16", batch=8, block_lo=32, block_hi=64,
             prefix_lo=700, prefix_hi=1500, suffix_lo=0, suffix_hi=0, lens=6, **SMALL_HEADS),
        # One attention layer of the 8B model over ragged blocks: one K/V head per query head, so
        # the cached keys and values are read for a handful of queries each.
        dict(name="attn_llada_ragged_b32", kind="attn", dtype="bf16", batch=32, block_lo=8,
             block_hi=128, prefix_lo=2048, prefix_hi=2048, suffix_lo=0, suffix_hi=0, lens=7,
             **_heads(LLADA)),
        # The dual cache: odd prefixes and a cached suffix, grouped heads, a full batch.
        dict(name="attn_dual_dream_b64", kind="attn", dtype="bf16", batch=64, block_lo=16,
             block_hi=256, prefix_lo=1001, prefix_hi=4096, suffix_lo=1, suffix_hi=511, lens=8,
             **_heads(DREAM)),
        # LM head with the sampler's features for one or two odd blocks.
        dict(name="lmhead_dream_gap_48", kind="lmhead", dtype="bf16", rows=48, gap=True,
             **_head(DREAM)),
        # LM head of four sequences with the base block of 32.
        dict(name="lmhead_llada_128", kind="lmhead", dtype="bf16", rows=128, gap=False,
             **_head(LLADA)),
        # LM head with features of a handful of ragged blocks: an odd number of rows.
        dict(name="lmhead_llada_gap_301", kind="lmhead", dtype="bf16", rows=301, gap=True,
             **_head(LLADA)),
        # The budgeted commit of a full batch.
        dict(name="commit_topm_b64", kind="commit", rule="topm", m=2, batch=64, block_lo=16,
             block_hi=256, lens=9, tau=0.9),
        # Choosing the next active blocks of a full batch over windows of generation length 512.
        dict(name="lbs_b64", kind="lbs", n_seq=64, window=512, l_min=8, l_b=32, g_max=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _span(rng, lo, hi):
    a = _log_int(rng, lo, hi)
    return (a, a) if rng.random() < 0.4 else (max(lo, a // rng.choice((2, 4, 8))), a)


def draw(rng):
    kind = rng.choice(("step", "step", "attn", "attn", "attn", "lmhead", "lmhead", "lmhead",
                       "commit", "lbs"))
    lens = rng.randrange(1 << 20)
    if kind in ("step", "attn"):
        f32 = rng.random() < 0.15
        batch = _log_int(rng, 1, 4 if f32 else 64)
        lo, hi = _span(rng, 4, 64 if f32 else 256)
        if batch * (lo + hi) > 2 * 8192:  # no more rows than the largest listed case
            lo, hi = min(lo, 64), 128
        plo, phi = _span(rng, 16, 256 if f32 else 4096)
        c = dict(kind=kind, dtype="f32" if f32 else "bf16", batch=batch, block_lo=lo, block_hi=hi,
                 prefix_lo=plo, prefix_hi=phi, lens=lens)
        if kind == "attn":
            slo, shi = _span(rng, 1, 512) if rng.random() < 0.35 else (0, 0)
            heads = TINY if f32 else rng.choice((LLADA, DREAM, LLADA, DREAM, SMALL_HEADS))
            return dict(c, suffix_lo=slo, suffix_hi=shi, **_heads(heads))
        if f32:
            return dict(c, tau=0.9, **dict(TINY, hidden=rng.randrange(96, 513),
                                           vocab=_log_int(rng, 500, 8192)))
        return dict(c, tau=rng.choice((0.7, 0.8, 0.9)), **rng.choice((LLADA, DREAM)))
    if kind == "lmhead":
        if rng.random() < 0.15:
            return dict(kind=kind, dtype="f32", rows=_log_int(rng, 1, 256),
                        hidden=rng.randrange(96, 513), vocab=_log_int(rng, 500, 8192),
                        gap=rng.random() < 0.5)
        head = dict(rng.choice((_head(LLADA), _head(DREAM))))
        if rng.random() < 0.3:  # another backbone
            head = dict(hidden=64 * rng.randrange(16, 65), vocab=rng.randrange(32000, 152064))
        return dict(kind=kind, dtype="bf16", rows=_log_int(rng, 1, 4096), gap=rng.random() < 0.5,
                    **head)
    if kind == "commit":
        lo, hi = _span(rng, 8, 512)
        return dict(kind=kind, rule=rng.choice(("threshold", "union", "topm")),
                    m=rng.randrange(1, 9), batch=_log_int(rng, 1, 128), block_lo=lo, block_hi=hi,
                    lens=lens, tau=rng.choice((0.7, 0.9)))
    return dict(kind=kind, n_seq=_log_int(rng, 1, 128), window=_log_int(rng, 64, 2048),
                l_min=rng.randrange(4, 17), l_b=rng.choice((16, 32, 64)),
                g_max=rng.randrange(1, 9))


# --------------------------------------------------------------------------------------------
# sizes and inputs (plain torch; shared by prepare() and exact())
# --------------------------------------------------------------------------------------------
def _lens(case):
    """Block, prefix and suffix lengths of every sequence (fixed by the case)."""
    rng = random.Random(case["lens"])

    def some(what):
        lo, hi = case.get(what + "_lo", 0), case.get(what + "_hi", 0)
        return [rng.randint(lo, hi) for _ in range(case["batch"])]

    return some("block"), some("prefix"), some("suffix")


def _cu(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return cu


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _attn_inputs(case, g):
    """Queries, keys and values N(0, 1)."""
    bl, pl, sl = _lens(case)
    dt, hkv, d = _dtype(case), case["hkv"], case["head_dim"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=dt)

    x = dict(q=normal(sum(bl), case["hq"], d))
    for seg, n in (("blk", sum(bl)), ("pre", sum(pl)), ("suf", sum(sl))):
        x["k_" + seg], x["v_" + seg] = normal(n, hkv, d), normal(n, hkv, d)
    return x


def _lm_inputs(case, rows, g):
    """W ~ N(0, 1/d).  Half of the rows are hard (h is noise); the others point at a token whose
    logit is spread from 4 to about 6 above ln(vocab), so that their confidences cover the whole
    range up to 0.997."""
    dt, d, vocab = _dtype(case), case["hidden"], case["vocab"]
    w = torch.randn(vocab, d, generator=g, device="cuda", dtype=dt).mul_(d ** -0.5)
    t = torch.randint(0, vocab, (rows,), generator=g, device="cuda")
    u = w[t].float()
    u = u / u.norm(dim=1, keepdim=True)
    r = torch.rand(2, rows, 1, generator=g, device="cuda")
    lift = torch.where(r[0] < 0.5, 4.0 + (math.log(vocab) + 2.2) * r[1], torch.zeros_like(r[1]))
    h = torch.randn(rows, d, generator=g, device="cuda") + lift * u
    return dict(w=w, h=h.to(dt))


def _mask_inputs(case, rows, vocab, g):
    """Half of the positions are still masked; the others hold a token already."""
    masked = (torch.rand(rows, generator=g, device="cuda") < 0.5).to(torch.uint8)
    tokens = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
    return masked, torch.where(masked.bool(), torch.full_like(tokens, -1), tokens)


def _out(n, dtype):
    return torch.zeros(n, dtype=dtype, device="cuda")


# --------------------------------------------------------------------------------------------
# prepare / run
# --------------------------------------------------------------------------------------------
def prepare(case, seed):
    g = _gen(seed)
    return {"step": _prepare_step, "attn": _prepare_attn, "lmhead": _prepare_lmhead,
            "commit": _prepare_commit, "lbs": _prepare_lbs}[case["kind"]](case, g)


def run(state):
    return state["run"](state)


def _prepare_step(case, g):
    bl, pl, _ = _lens(case)
    rows, batch = sum(bl), case["batch"]
    a, m = _attn_inputs(case, g), _lm_inputs(case, rows, g)
    masked, tokens = _mask_inputs(case, rows, case["vocab"], g)
    tau = torch.full((batch,), case["tau"], dtype=torch.float32, device="cuda")
    out = dict(attn=torch.zeros_like(a["q"]), conf=_out(rows, torch.float32),
               entropy=_out(rows, torch.float32), max_logit=_out(rows, torch.float32),
               argmax=_out(rows, torch.int32), masked=masked, tokens=tokens,
               unmask=_out(rows, torch.uint8), n_commit=_out(batch, torch.int32),
               resolved=_out(batch, torch.uint8))
    buffers = eb.StepBuffers(
        eb.Ragged.from_lengths(bl, pl), a["q"], a["k_blk"], a["v_blk"], a["k_pre"], a["v_pre"],
        out["attn"], m["h"], m["w"], out["conf"], out["entropy"], out["argmax"], tau, masked,
        tokens, out["unmask"], out["n_commit"], out["resolved"], max_logit=out["max_logit"])
    return dict(run=_run_step, buffers=buffers, out=out)


def _run_step(s):
    # a decoder steps a block again and again; masked and tokens carry on from pass to pass
    eb.eb_decode_step(s["buffers"])
    return s["out"]


def _prepare_attn(case, g):
    bl, pl, sl = _lens(case)
    x = _attn_inputs(case, g)
    s = dict(run=_run_attn, x=x, r=eb.Ragged.from_lengths(bl, pl), out=torch.zeros_like(x["q"]),
             ws=None, max_suffix=max(sl))
    if max(sl):
        s["cu_suffix"] = torch.tensor(_cu(sl), dtype=torch.int32, device="cuda")
    else:
        need = eb.eb_block_attn_workspace(eb.EB_F32 if case["dtype"] == "f32" else eb.EB_BF16,
                                          s["r"], case["hq"], case["hkv"], case["head_dim"])
        s["ws"] = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    return s


def _run_attn(s):
    x = s["x"]
    if s["max_suffix"]:
        eb.eb_block_attn_dual(s["r"], s["cu_suffix"], s["max_suffix"], x["q"], x["k_blk"],
                              x["v_blk"], x["k_pre"], x["v_pre"], x["k_suf"], x["v_suf"],
                              s["out"])
    else:
        eb.eb_block_attn(s["r"], x["q"], x["k_blk"], x["v_blk"], x["k_pre"], x["v_pre"],
                         s["out"], ws=s["ws"])
    return s["out"]


def _prepare_lmhead(case, g):
    rows = case["rows"]
    m = _lm_inputs(case, rows, g)
    out = dict(conf=_out(rows, torch.float32), entropy=_out(rows, torch.float32),
               max_logit=_out(rows, torch.float32), argmax=_out(rows, torch.int32))
    if case["gap"]:
        out["gap"] = _out(rows, torch.float32)
    need = (eb.eb_lmhead_features_workspace if case["gap"] else eb.eb_lmhead_workspace)(
        eb.EB_F32 if case["dtype"] == "f32" else eb.EB_BF16, rows, case["hidden"], case["vocab"])
    ws = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    return dict(run=_run_lmhead, out=out, ws=ws, **m)


def _run_lmhead(s):
    o = s["out"]
    if "gap" in o:
        eb.eb_lmhead_features(s["h"], s["w"], o["conf"], o["entropy"], o["argmax"], o["gap"],
                              max_logit=o["max_logit"], ws=s["ws"])
    else:
        eb.eb_lmhead_confidence(s["h"], s["w"], o["conf"], o["entropy"], o["argmax"],
                                max_logit=o["max_logit"], ws=s["ws"])
    return o


COMMIT_VOCAB = 126464


def _commit_inputs(case, g):
    """Statistics as an LM head leaves them: half the rows near their least confidence, the rest
    spread up to one, with entropy and gap to match; router scores uniform."""
    rows = sum(_lens(case)[0])
    r = torch.rand(4, rows, generator=g, device="cuda")
    conf = torch.where(r[0] < 0.5, 1e-4 + 1e-3 * r[1], torch.sigmoid(20.0 * r[1] - 8.0))
    masked, tokens = _mask_inputs(case, rows, COMMIT_VOCAB, g)
    return dict(conf=conf, entropy=(1.0 - conf) * 11.0, gap=conf * (0.5 + 0.5 * r[2]),
                p_psi=r[3].contiguous(), masked=masked, tokens=tokens,
                argmax=torch.randint(0, COMMIT_VOCAB, (rows,), generator=g, device="cuda",
                                     dtype=torch.int32))


def _prepare_commit(case, g):
    bl = _lens(case)[0]
    rows, batch = sum(bl), case["batch"]
    x = _commit_inputs(case, g)
    # mask flags and tokens, which a step updates, lie in one buffer: a program that starts on a
    # new block fills both with one copy
    fresh = torch.cat([x["tokens"].view(torch.uint8), x["masked"]])
    work = fresh.clone()
    out = dict(tokens=work[:4 * rows].view(torch.int32), masked=work[4 * rows:],
               unmask=_out(rows, torch.uint8), n_commit=_out(batch, torch.int32),
               resolved=_out(batch, torch.uint8))
    if case["rule"] == "union":
        out.update(feat=torch.zeros(rows, 4, device="cuda"), pos=_out(rows, torch.float32),
                   ratio=_out(batch, torch.float32))
    tau = torch.full((batch,), case["tau"], dtype=torch.float32, device="cuda")
    return dict(run=_run_commit, rule=case["rule"], m=case["m"], x=x, fresh=fresh, work=work,
                tau=tau, out=out, r=eb.Ragged.from_lengths(bl, [0] * batch))


def _run_commit(s):
    x, o, r = s["x"], s["out"], s["r"]
    s["work"].copy_(s["fresh"])
    args = (o["masked"], o["tokens"], o["unmask"], o["n_commit"], o["resolved"])
    if s["rule"] == "union":
        eb.eb_lps_features(r, COMMIT_VOCAB, x["conf"], x["entropy"], x["gap"], o["masked"],
                           o["feat"], o["pos"], mask_ratio=o["ratio"])
        eb.eb_unmask_select_lps(r, x["conf"], x["argmax"], s["tau"], x["p_psi"], 0.8, *args)
    elif s["rule"] == "topm":
        eb.eb_unmask_select_topm(r, x["conf"], x["argmax"], s["tau"], s["m"], *args)
    else:
        eb.eb_unmask_select(r, x["conf"], x["argmax"], s["tau"], *args)
    return o


LBS_EOS = 2


def _prepare_lbs(case, g):
    """Windows at different progress: few positions masked behind the front, most beyond it; the
    predictions end in a tail of EOS; router scores uniform."""
    n, length = case["n_seq"], case["window"]
    r = torch.rand(2, n, length, generator=g, device="cuda")
    at = torch.rand(2, n, 1, generator=g, device="cuda")
    pos = torch.arange(length, device="cuda") / length
    masked = (r[0] < torch.where(pos < at[0], 0.05, 0.9)).to(torch.uint8)
    x_hat = torch.randint(3, 126464, (n, length), generator=g, device="cuda", dtype=torch.int32)
    x_hat[pos >= 0.6 + 0.4 * at[1]] = LBS_EOS
    out = dict(block=torch.zeros(n, length, dtype=torch.uint8, device="cuda"),
               size=_out(n, torch.int32), first=_out(n, torch.int32))
    return dict(run=_run_lbs, masked=masked, p_phi=r[1].contiguous(), x_hat=x_hat, out=out,
                limits=(case["l_min"], case["l_b"], case["g_max"]))


def _run_lbs(s):
    o = s["out"]
    eb.eb_lbs_select(s["masked"], s["p_phi"], s["x_hat"], LBS_EOS, *s["limits"], o["block"],
                     o["size"], o["first"])
    return o


# --------------------------------------------------------------------------------------------
# work, tolerance
# --------------------------------------------------------------------------------------------
def _work_attn(case):
    bl, pl, sl = _lens(case)
    e, d = (4 if case["dtype"] == "f32" else 2), case["head_dim"]
    rows, keys = sum(bl), sum(bl) + sum(pl) + sum(sl)
    return {"bytes": e * d * (2 * case["hq"] * rows + 2 * case["hkv"] * keys),
            "flops": 4 * case["hq"] * d * sum(b * (b + p + s) for b, p, s in zip(bl, pl, sl))}


def _work_lm(case, rows, outs):
    e = 4 if case["dtype"] == "f32" else 2
    return {"bytes": e * case["hidden"] * (case["vocab"] + rows) + 4 * outs * rows,
            "flops": 2 * rows * case["hidden"] * case["vocab"]}


def work(case):
    kind = case["kind"]
    if kind == "attn":
        return _work_attn(case)
    if kind == "lmhead":
        return _work_lm(case, case["rows"], 5 if case["gap"] else 4)
    if kind == "lbs":  # flag, score and predicted token of a position, and its answer
        return {"bytes": case["n_seq"] * (10 * case["window"] + 8), "flops": 0}
    rows, batch = sum(_lens(case)[0]), case["batch"]
    # conf, argmax, mask flag and token in; unmask, mask flag and token out
    commit = 8 * rows + 5 * rows + 6 * rows + 9 * batch
    if kind == "commit":  # the flags and tokens also come from the program's copy
        commit += 10 * rows
        if case["rule"] == "union":  # conf, entropy, gap, flag in; features out; the score in
            commit += 13 * rows + 20 * rows + 4 * rows + 4 * batch
        return {"bytes": commit, "flops": 0}
    a, m = _work_attn(case), _work_lm(case, rows, 4)
    return {"bytes": a["bytes"] + m["bytes"] + commit, "flops": a["flops"] + m["flops"]}


def tolerance(case):
    if case["kind"] == "lbs" or (case["kind"] == "commit" and case["rule"] != "union"):
        return "exact"
    if case["kind"] == "commit":  # one rounding of a quotient or product per feature
        return {"rel": 1e-6, "max": 1e-5}
    # LM head: sums in 32 bits, 2e-7 to 6e-7 off 64 bits over many rows; the entropy of a single
    # confident row is a small difference of sums near one and up to ten times that
    if case["kind"] == "lmhead" and case["gap"]:  # a few rows whose two top logits nearly tie:
        return {"rel": 5e-5, "max": 1e-3, "differ": 2e-3}  # 1.2e-5 seen
    if case["kind"] == "lmhead" or case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4, "differ": 2e-3}
    # attention: probabilities and outputs rounded to bf16, 2.1e-3 to 2.3e-3 off 64 bits
    return {"rel": 1e-2, "max": 0.1, "differ": 2e-3}


# --------------------------------------------------------------------------------------------
# the same outputs in 64 bits
# --------------------------------------------------------------------------------------------
def _exact_attn(case, x):
    bl, pl, sl = _lens(case)
    cb, cp, cs = _cu(bl), _cu(pl), _cu(sl)
    hq, hkv, d = case["hq"], case["hkv"], case["head_dim"]
    out = torch.zeros(x["q"].shape, dtype=torch.float64, device="cuda")
    for b in range(case["batch"]):
        at = {"pre": slice(cp[b], cp[b + 1]), "blk": slice(cb[b], cb[b + 1]),
              "suf": slice(cs[b], cs[b + 1])}
        k, v = (torch.cat([x[n + s][i] for s, i in at.items()]).double().transpose(0, 1)
                .contiguous() for n in ("k_", "v_"))                     # [hkv, keys, d]
        q = x["q"][at["blk"]].double().reshape(-1, hkv, hq // hkv, d)
        q = q.permute(1, 0, 2, 3).reshape(hkv, -1, d)                    # [hkv, rows, d]
        p = torch.softmax(torch.bmm(q, k.transpose(1, 2).contiguous()) * d ** -0.5, dim=-1)
        o = torch.bmm(p, v).reshape(hkv, bl[b], hq // hkv, d)
        out[at["blk"]] = o.permute(1, 0, 2, 3).reshape(bl[b], hq, d)
    return out


def _exact_lm(x, gap):
    w, h = x["w"].double().t(), x["h"]
    got = []
    for i in range(0, h.shape[0], 1024):
        z = h[i:i + 1024].double() @ w
        top, lse = z.topk(2, dim=1).values, torch.logsumexp(z, dim=1)
        logp = z - lse[:, None]
        p = (top - lse[:, None]).exp()
        got.append((p[:, 0], -(logp.exp() * logp).sum(dim=1), top[:, 0], p[:, 0] - p[:, 1]))
    conf, entropy, max_logit, delta = (torch.cat(c) for c in zip(*got))
    out = dict(conf=conf, entropy=entropy, max_logit=max_logit, argmax=None)
    return dict(out, gap=delta) if gap else out


def exact(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind == "attn":
        return _exact_attn(case, _attn_inputs(case, g))
    if kind == "lmhead":
        return _exact_lm(_lm_inputs(case, case["rows"], g), case["gap"])
    if kind == "step":
        a = _attn_inputs(case, g)
        out = dict(_exact_lm(_lm_inputs(case, a["q"].shape[0], g), False),
                   attn=_exact_attn(case, a))
        return dict(out, **dict.fromkeys(("masked", "tokens", "unmask", "n_commit", "resolved")))
    if kind == "commit" and case["rule"] == "union":
        x, bl = _commit_inputs(case, g), _lens(case)[0]
        masked = x["masked"].double()
        ratio = torch.stack([m.mean() for m in masked.split(bl)])
        pos = torch.cat([torch.arange(n, dtype=torch.float64, device="cuda") / n for n in bl])
        feat = torch.stack([x["conf"].double(), x["entropy"].double() / math.log(COMMIT_VOCAB),
                            x["gap"].double(),
                            ratio.repeat_interleave(torch.tensor(bl, device="cuda"))], dim=1)
        none = dict.fromkeys(("tokens", "masked", "unmask", "n_commit", "resolved"))
        return dict(none, feat=feat, pos=pos, ratio=ratio)
    return None
