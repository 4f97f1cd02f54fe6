"""The work a program has this library do, as measurable cases.

A case is a dict of plain values.  Its "kind" names the call:

  step    one whole decode step, PreparedStep.step(): verify + select + draft
  paged   verify attention over a paged cache, verify_attn_paged()
  seed    the prefill-seeded first scores: verify_attn() over the last 16
          prompt positions
  draft   one draft-round step after `drafted` drafted tokens,
          PreparedRound.step(), through the index list or materialized rows
  entropy token entropy and argmax of logit rows, logit_stats()
  greedy  greedy acceptance of one verify pass, greedy_accept()
  sample  speculative-sampling acceptance, spec_accept()

Inputs.  Real attention is skewed and consecutive queries of a head resemble
each other, so the queries of a (sequence, head) share a direction and its
logits over random keys have a standard deviation of about 3; keys and values
are N(0, 1).  Logit rows are N(0, 2^2) with a handful of likely tokens raised,
the same ones in the drafter's and the target's rows.
"""
import math
import random

import torch

from paper_2607_27735_amd import binding as B

HEAD_DIM = 128
WINDOW, K_SINK, K_RECENT = 16, 4, 32
SM_SCALE = 1.0 / math.sqrt(HEAD_DIM)
DEVICE = "cuda"


def attention(name, kind, batch, hq, hkv, ctx_lo, ctx_hi, q_lo, q_hi, budget, **more):
    case = dict(kind=kind, batch=batch, hq=hq, hkv=hkv, ctx_lo=ctx_lo, ctx_hi=ctx_hi, q_lo=q_lo,
                q_hi=q_hi, budget=budget, fp32=False, per_head=False, lens=1)
    case.update(more)
    if name:
        case["name"] = name
    return case


def vocabulary(name, kind, batch, max_k, vocab, dtype, lens=1):
    case = dict(kind=kind, batch=batch, max_k=max_k, vocab=vocab, dtype=dtype, lens=lens)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest step: few heads, a short context (the smoke test's shape)
        attention("step_small_4k", "step", 1, 8, 2, 4096, 4096, 5, 5, 256),
        # one user of an 8B-shaped model at 32K: the benchmark's headline step
        attention("step_8b_32k", "step", 1, 32, 8, 32768, 32768, 7, 7, 2048),
        # one user, a book-length context, long speculation
        attention("step_8b_131k", "step", 1, 32, 8, 131072, 131072, 9, 9, 4096),
        # a serving batch of long ragged contexts
        attention("step_8b_b8_ragged", "step", 8, 32, 8, 16384, 65536, 3, 11, 4096),
        # a 70B-shaped layer, four users at 64K: the most bytes per call
        attention("step_70b_b4_64k", "step", 4, 64, 8, 65536, 65536, 6, 6, 4096),
        # a chat batch: many short odd contexts
        attention("step_8b_b16_chat", "step", 16, 32, 8, 1000, 8191, 2, 8, 1024),
        # an index set per query head, fp32 outputs, an odd length
        attention("step_per_head_24k", "step", 1, 32, 8, 24577, 24577, 5, 5, 1024, fp32=True,
                  per_head=True),
        # verify as a serving engine calls it: paged cache, ragged batch
        attention("verify_paged_b12", "paged", 12, 32, 8, 3000, 30000, 2, 7, 2048, page=64),
        # first scores of a prompt: 16 positions, 128 rows per KV head
        attention("seed_70b_20k", "seed", 1, 64, 8, 20011, 20011, 16, 16, 2048),
        # one drafted token, the call a step makes k times
        attention("draft_8b_32k", "draft", 1, 32, 8, 32762, 32762, 1, 1, 2048, drafted=3,
                  copied=False),
        # the acceptance of one step's tokens, greedy and sampling
        vocabulary("greedy_b4_128k", "greedy", 4, 6, 128256, "bf16"),
        vocabulary("sample_b4_128k", "sample", 4, 6, 128256, "bf16"),
    ]


def log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(["step", "paged", "seed", "draft", "entropy", "greedy", "sample"],
                       [10, 3, 2, 3, 1, 2, 2])[0]
    lens = rng.randrange(1 << 20)
    if kind in ("entropy", "greedy", "sample"):
        return vocabulary(None, kind, log_int(rng, 1, 16), rng.randint(2, 10),
                          log_int(rng, 32000, 160000), rng.choice(["bf16", "bf16", "f32"]), lens)
    while True:
        hq, hkv = rng.choice([(8, 2), (32, 8), (32, 8), (64, 8), (16, 2), (16, 16)])
        hi = log_int(rng, 1000, 131072)
        batch = log_int(rng, 1, 16)
        # K and V no more than the largest listed case's (first scores read them several times)
        if batch * hi * hkv * 4 * HEAD_DIM <= (300_000_000 if kind == "seed" else 1_070_000_000):
            break
    lo = hi if rng.random() < 0.4 else max(600, int(hi * rng.uniform(0.2, 0.9)))
    lo = min(lo, hi)
    budget = min(log_int(rng, 256, 4096), hi)
    if kind == "seed":
        return attention(None, kind, batch, hq, hkv, lo, hi, 16, 16, budget, lens=lens)
    if kind == "draft":
        return attention(None, kind, batch, hq, hkv, lo, hi, 1, 1, budget, lens=lens,
                         drafted=rng.randint(0, 12), copied=rng.random() < 0.4)
    q_hi = rng.randint(2, 12) if hq // hkv <= 4 else rng.randint(2, 8)
    q_lo = q_hi if rng.random() < 0.5 else rng.randint(2, q_hi)
    if kind == "paged":
        return attention(None, kind, batch, hq, hkv, lo, hi, q_lo, q_hi, budget, lens=lens,
                         page=rng.choice([32, 64, 128]))
    return attention(None, kind, batch, hq, hkv, lo, hi, q_lo, q_hi, budget, lens=lens,
                     fp32=rng.random() < 0.25, per_head=rng.random() < 0.15)


# ---- lengths, seeds, tensors -------------------------------------------------------

def lengths(case):
    """(ctx_len, q_len) of every sequence: from the case alone."""
    r = random.Random(case["lens"])
    ctx = [r.randint(case["ctx_lo"], case["ctx_hi"]) for _ in range(case["batch"])]
    ql = [r.randint(case["q_lo"], case["q_hi"]) for _ in range(case["batch"])]
    return ctx, ql


def drafts(case):
    """Drafted tokens of every sequence of a vocabulary case."""
    r = random.Random(case["lens"])
    k = [r.randint(max(1, case["max_k"] - 3), case["max_k"]) for _ in range(case["batch"])]
    k[0] = case["max_k"]
    return k


def generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def normal(g, *shape, dtype=torch.bfloat16):
    return torch.randn(*shape, generator=g, device=DEVICE, dtype=torch.float32).to(dtype)


def cache(g, batch, hkv, rows):
    """[batch][hkv][rows][128] bf16, drawn a sequence at a time."""
    t = torch.empty(batch, hkv, rows, HEAD_DIM, device=DEVICE, dtype=torch.bfloat16)
    for b in range(batch):
        t[b] = normal(g, hkv, rows, HEAD_DIM)
    return t


def queries(g, batch, positions, hq, hkv):
    """Rows of a (sequence, KV head) share a direction: |q| = 3 sqrt(128), of
    which the shared part holds 0.8 in variance."""
    shared = normal(g, batch, 1, hkv, 1, HEAD_DIM, dtype=torch.float32)
    own = normal(g, batch, positions, hkv, hq // hkv, HEAD_DIM, dtype=torch.float32)
    q = 3.0 * (math.sqrt(0.8) * shared + math.sqrt(0.2) * own)
    return q.reshape(batch, positions, hq, HEAD_DIM).to(torch.bfloat16)


def params_of(case):
    return B.make_params(SM_SCALE, window=WINDOW, k_sink=K_SINK, k_recent=K_RECENT,
                         budget=case["budget"], out_fp32=case["fp32"], per_head=case["per_head"])


def out_type(case):
    return torch.float32 if case["fp32"] else torch.bfloat16


def attention_inputs(case, seed):
    g = generator(seed)
    ctx, ql = lengths(case)
    batch, hq, hkv = case["batch"], case["hq"], case["hkv"]
    s = dict(case=case, ctx=ctx, ql=ql, params=params_of(case))
    max_q = max(ql)
    s["q"] = queries(g, batch, max_q + 1, hq, hkv)
    s["q_draft"] = s["q"][:, max_q].contiguous()
    s["q"] = s["q"][:, :max_q].contiguous()
    s["max_ctx"] = (max(ctx) + 63 + case.get("drafted", 0)) // 64 * 64
    s["k"] = cache(g, batch, hkv, s["max_ctx"])
    s["v"] = cache(g, batch, hkv, s["max_ctx"])
    units = hq if case["per_head"] else hkv
    s["out"] = torch.zeros(s["q"].shape, dtype=out_type(case), device=DEVICE)
    s["scores"] = torch.zeros(batch, units, s["max_ctx"], dtype=torch.float32, device=DEVICE)
    return g, s


def to_pages(g, s, page):
    """The dense caches as page pools with a shuffled block table."""
    batch, hkv = s["case"]["batch"], s["case"]["hkv"]
    blocks = -(-s["max_ctx"] // page)
    perm = torch.randperm(batch * blocks, generator=g, device=DEVICE)
    s["table"] = perm.to(torch.int32).reshape(batch, blocks)
    for name in ("k", "v"):
        dense = s.pop(name)
        pool = torch.zeros(batch * blocks, hkv, page, HEAD_DIM, dtype=torch.bfloat16, device=DEVICE)
        for b in range(batch):
            rows = torch.zeros(hkv, blocks * page, HEAD_DIM, dtype=torch.bfloat16, device=DEVICE)
            rows[:, :s["max_ctx"]] = dense[b]
            pool[s["table"][b].long()] = rows.reshape(hkv, blocks, page, HEAD_DIM).transpose(0, 1)
        s[name] = pool


def from_pages(s, name, b):
    pool = s[name][s["table"][b].long()]                    # [blocks][hkv][page][128]
    return pool.transpose(0, 1).reshape(pool.shape[1], -1, HEAD_DIM)


def index_sets(g, case, ctx, budget):
    """An ascending index list per unit, as select leaves it at lengths ctx:
    sink, random middle positions, recent."""
    units = case["hkv"]
    idx = torch.zeros(case["batch"], units, budget, dtype=torch.int32, device=DEVICE)
    for b, T in enumerate(ctx):
        s_end = min(K_SINK, T)
        r0 = max(T - K_RECENT, s_end)
        mid = min(budget - K_SINK - K_RECENT, r0 - s_end)
        order = torch.rand(units, r0 - s_end, generator=g, device=DEVICE).argsort(dim=1)[:, :mid]
        parts = [torch.arange(s_end, device=DEVICE).expand(units, -1), order.sort(dim=1).values + s_end,
                 torch.arange(r0, T, device=DEVICE).expand(units, -1)]
        row = torch.cat(parts, dim=1).to(torch.int32)
        idx[b, :, :row.shape[1]] = row
    return idx


def logits_of(g, batch, rows, vocab, raised, dtype):
    """[batch][rows][stride] logit rows (the stride vocab padded to a multiple
    of 8): N(0, 2^2), the tokens raised[b][row] (the same for drafter and
    target) 9 to 15 higher."""
    x = 2.0 * torch.randn(batch, rows, (vocab + 7) // 8 * 8, generator=g, device=DEVICE)
    up = 9.0 + 6.0 * torch.rand(raised[:, :rows].shape, generator=g, device=DEVICE)
    x.scatter_add_(2, raised[:, :rows], up)
    return x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)


def vocabulary_inputs(case, seed):
    g = generator(seed)
    batch, max_k, vocab = case["batch"], case["max_k"], case["vocab"]
    s = dict(case=case, k_len=drafts(case))
    raised = torch.randint(0, vocab, (batch, max_k + 1, 8), generator=g, device=DEVICE)
    s["target"] = logits_of(g, batch, max_k + 1, vocab, raised, case["dtype"])
    s["draft"] = logits_of(g, batch, max_k, vocab, raised, case["dtype"])
    # drafted tokens: mostly the target's own choice, now and then another likely one
    best = s["target"][:, :max_k, :vocab].argmax(dim=2)
    other = torch.rand(batch, max_k, generator=g, device=DEVICE) < 0.15
    s["tokens"] = torch.where(other, raised[:, :max_k, 0], best).to(torch.int32)
    s["u_accept"] = torch.rand(batch, max_k, generator=g, device=DEVICE)
    s["u_sample"] = torch.rand(batch, generator=g, device=DEVICE)
    return s


# ---- what a program has in hand, and one pass -----------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("entropy", "greedy", "sample"):
        s = vocabulary_inputs(case, seed)
        if kind == "entropy":
            s["rows"] = s["draft"].reshape(-1, s["draft"].shape[2])
        return s
    g, s = attention_inputs(case, seed)
    batch, hkv, hq = case["batch"], case["hkv"], case["hq"]
    if kind == "step":
        units = hq if case["per_head"] else hkv
        s["idx"] = torch.zeros(batch, units, case["budget"], dtype=torch.int32, device=DEVICE)
        s["n_idx"] = torch.zeros(batch, dtype=torch.int32, device=DEVICE)
        s["draft_out"] = torch.zeros(s["q_draft"].shape, dtype=out_type(case), device=DEVICE)
        s["call"] = B.PreparedStep(s["q"], s["k"], s["v"], s["q_draft"], s["ctx"], s["ql"],
                                   s["params"], s["out"], s["scores"], s["idx"], s["n_idx"],
                                   s["draft_out"], shared_workspace=True)
    elif kind == "draft":
        s["idx"] = index_sets(g, case, s["ctx"], case["budget"])
        s["draft_out"] = torch.zeros(s["q_draft"].shape, dtype=out_type(case), device=DEVICE)
        sel = None, None
        if case["copied"]:
            sel = B.draft_materialize(s["k"], s["v"], s["idx"], s["ctx"], s["params"])
        s["call"] = B.PreparedRound(s["q_draft"], s["k"], s["v"], s["idx"], s["ctx"],
                                    case["drafted"], s["params"], s["draft_out"], *sel)
    else:
        shape = B.Shape(batch, hq, hkv, HEAD_DIM, s["max_ctx"], s["q"].shape[1])
        if kind == "paged":
            to_pages(g, s, case["page"])
        s["workspace"] = torch.empty(B.verify_workspace_bytes(shape, s["params"], s["ctx"], s["ql"]),
                                     dtype=torch.uint8, device=DEVICE)
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "step":
        s["call"].step()
        return {"out": s["out"], "scores": s["scores"], "idx": s["idx"], "n_idx": s["n_idx"],
                "draft_out": s["draft_out"]}
    if kind == "paged":
        out, scores = B.verify_attn_paged(s["q"], s["k"], s["v"], s["table"], s["max_ctx"], s["ctx"],
                                          s["ql"], s["params"], out=s["out"], scores=s["scores"],
                                          workspace=s["workspace"])
        return {"out": out, "scores": scores}
    if kind == "seed":
        out, scores = B.verify_attn(s["q"], s["k"], s["v"], s["ctx"], s["ql"], s["params"],
                                    out=s["out"], scores=s["scores"], workspace=s["workspace"])
        return {"out": out, "scores": scores}
    if kind == "draft":
        s["call"].step(s["case"]["drafted"])
        return {"draft_out": s["draft_out"]}
    if kind == "entropy":
        entropy, best = B.logit_stats(s["rows"], vocab=s["case"]["vocab"])
        return {"entropy": entropy, "best": best}
    if kind == "greedy":
        accepted, token = B.greedy_accept(s["target"], s["tokens"], s["k_len"],
                                          vocab=s["case"]["vocab"])
    else:
        accepted, token = B.spec_accept(s["target"], s["draft"], s["tokens"], s["k_len"], 0.8,
                                        s["u_accept"], s["u_sample"], vocab=s["case"]["vocab"])
    return {"accepted": accepted, "token": token}


def index_count(case, T):
    s_end = min(K_SINK, T)
    r0 = max(T - K_RECENT, s_end)
    return s_end + min(case["budget"] - K_SINK - K_RECENT, r0 - s_end) + T - r0


def work(case):
    kind = case["kind"]
    if kind in ("entropy", "greedy", "sample"):
        size = 2 if case["dtype"] == "bf16" else 4
        k, vocab = drafts(case), case["vocab"]
        rows = case["batch"] * case["max_k"] if kind == "entropy" else sum(k) + case["batch"]
        if kind == "sample":
            rows += sum(k)
        return {"bytes": rows * vocab * size + 16 * case["batch"] * case["max_k"],
                "flops": 4.0 * rows * vocab}
    ctx, ql = lengths(case)
    hq, hkv, g = case["hq"], case["hkv"], case["hq"] // case["hkv"]
    osize = 4 if case["fp32"] else 2
    units = hq if case["per_head"] else hkv
    n_bytes = flops = 0
    for T, n in zip(ctx, ql):
        picked = index_count(case, T)
        if kind != "draft":
            n_bytes += hkv * T * 4 * HEAD_DIM + n * hq * HEAD_DIM * (2 + osize) + 4 * units * T
            flops += 4 * HEAD_DIM * n * hq * T
        else:
            n_bytes += hkv * picked * 4 * HEAD_DIM + (0 if case["copied"] else 4 * hkv * picked)
        if kind in ("step", "draft"):
            n_bytes += hq * HEAD_DIM * (2 + osize) + (4 * units * picked if kind == "step" else 0)
            flops += 4 * HEAD_DIM * hq * picked
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    # whole numbers: the acceptance rules have one answer for given logits
    if case["kind"] in ("greedy", "sample"):
        return "exact"
    # fp32 sums over the vocabulary, merged in another order; the argmax has one answer
    if case["kind"] == "entropy":
        return {"rel": 1e-5, "max": 1e-4}
    # bf16 probabilities in the value product (relative 2^-9) and bf16 outputs; a key whose score
    # ties with the last one taken to fp32 rounding may be exchanged for it, which shifts the
    # entries between the two in one ascending list
    tol = {"rel": 1e-2, "max": 1e-1}
    if case["kind"] == "step":
        tol["differ"] = 1e-2
    return tol


# ---- the same in 64 bits ------------------------------------------------------------------

def exact_attention(s, b, c, k, v):
    """(out [rows][group][128], per-head probabilities summed over the window
    [group][T]) of KV head c of sequence b."""
    case = s["case"]
    g, n, T = case["hq"] // case["hkv"], s["ql"][b], s["ctx"][b]
    q = s["q"][b, :n, c * g:(c + 1) * g].double().reshape(n * g, HEAD_DIM)
    y = (q @ k[:T].double().T) * SM_SCALE
    last = torch.arange(T - n, T, device=DEVICE).repeat_interleave(g)
    y.masked_fill_(torch.arange(T, device=DEVICE)[None, :] > last[:, None], -math.inf)
    p = torch.softmax(y, dim=1)
    out = (p @ v[:T].double()).reshape(n, g, HEAD_DIM)
    return out, p.reshape(n, g, T)[max(0, n - WINDOW):].sum(dim=0)


def exact_draft(q, k, v, rows):
    """Softmax attention of q [heads][128] over the given cache rows."""
    y = (q.double() @ k[rows].double().T) * SM_SCALE
    return torch.softmax(y, dim=1) @ v[rows].double()


def exact_rows(case, score, T):
    """The rows of Eq. 4's set for one unit's scores."""
    s_end = min(K_SINK, T)
    r0 = max(T - K_RECENT, s_end)
    take = min(case["budget"] - K_SINK - K_RECENT, r0 - s_end)
    order = torch.sort(score[s_end:r0], descending=True, stable=True).indices[:take] + s_end
    return torch.cat([torch.arange(s_end, device=DEVICE), order, torch.arange(r0, T, device=DEVICE)])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("greedy", "sample"):
        return None
    s = prepare(case, seed)
    if kind == "entropy":
        lp = torch.log_softmax(s["rows"][:, :case["vocab"]].double(), dim=1)
        return {"entropy": -(lp.exp() * lp).sum(dim=1), "best": None}
    hq, hkv, g = case["hq"], case["hkv"], case["hq"] // case["hkv"]
    if kind == "draft":
        out = torch.zeros(s["q_draft"].shape, dtype=torch.float64, device=DEVICE)
        for b, T in enumerate(s["ctx"]):
            cur = T + case["drafted"]
            r0 = max(T - K_RECENT, min(K_SINK, T))
            n_fixed = index_count(case, T) - (T - r0)
            window = torch.arange(max(r0, cur - K_RECENT), cur, device=DEVICE)
            for c in range(hkv):
                rows = torch.cat([s["idx"][b, c, :n_fixed].long(), window])
                out[b, c * g:(c + 1) * g] = exact_draft(s["q_draft"][b, c * g:(c + 1) * g],
                                                        s["k"][b, c], s["v"][b, c], rows)
        return {"draft_out": out}
    out = torch.zeros(s["q"].shape, dtype=torch.float64, device=DEVICE)
    scores = torch.zeros(s["scores"].shape, dtype=torch.float64, device=DEVICE)
    draft_out = torch.zeros(s["q_draft"].shape, dtype=torch.float64, device=DEVICE)
    for b, T in enumerate(s["ctx"]):
        kb = from_pages(s, "k", b) if kind == "paged" else s["k"][b]
        vb = from_pages(s, "v", b) if kind == "paged" else s["v"][b]
        for c in range(hkv):
            o, per_head = exact_attention(s, b, c, kb[c], vb[c])
            heads = slice(c * g, (c + 1) * g)
            out[b, :s["ql"][b], heads] = o
            score = per_head if case["per_head"] else per_head.sum(dim=0, keepdim=True)
            scores[b, heads if case["per_head"] else slice(c, c + 1), :T] = score
            if kind == "step":
                for h in range(g):
                    rows = exact_rows(case, score[h if case["per_head"] else 0], T)
                    draft_out[b, c * g + h] = exact_draft(s["q_draft"][b, c * g + h][None], kb[c],
                                                          vb[c], rows)[0]
    r = {"out": out, "scores": scores}
    if kind == "step":
        r.update(idx=None, n_idx=None, draft_out=draft_out)
    return r
