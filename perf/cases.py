"""The calls whose time matters to a user of this library, as cases that can be
timed and compared: prefix prefill, head grouping, decode attention and whole
generations, through the public entry points (Session and the C ABI's step
loop), over the sizes of the repository's workloads and around them.

listed() and draw() give cases (dicts of plain values), prepare() the inputs
and the handle a decoder holds before the call, run() one pass, work() what a
pass cannot do without, tolerance() how far two correct implementations may
differ, exact() the same results in plain 64-bit torch.
"""
from __future__ import annotations

import math

import torch

from paper_2605_20600_amd import binding as B
from paper_2605_20600_amd import synth
from paper_2605_20600_amd.session import Session, make_config
from paper_2605_20600_amd.workloads import (BUDGET_OVERRIDE, BUDGET_PAPER, BUDGET_TOTAL,
                                            Workload)

BUDGETS = {"paper": (BUDGET_PAPER, None), "total": (BUDGET_TOTAL, None),
           "rows_1_16": (BUDGET_OVERRIDE, "rows_1_16"),
           "loguniform_64_1024": (BUDGET_OVERRIDE, "loguniform_64_1024")}
SCORES = {"mean_logit": B.HEADKV_SCORE_MEAN_LOGIT, "attn_sum": B.HEADKV_SCORE_ATTN_SUM}

# Shapes of the repository's workloads.
LUMINA768 = dict(batch=8, heads=32, head_dim=128, prefix=128, rows=48, cols=48, row_end=True,
                 period=49, threshold=300, rho_den=8, budgets="paper", amp="lumina",
                 score="mean_logit", cfg_pairs=False)
LUMINA1024 = dict(LUMINA768, batch=4, rows=64, cols=64, period=65, threshold=500,
                  budgets="rows_1_16")
JANUS7B = dict(LUMINA768, batch=16, prefix=64, rows=24, cols=24, row_end=False, period=24,
               threshold=100, rho_den=4, budgets="total", amp="janus")
STRESS = dict(LUMINA768, batch=64, period=1, budgets="loguniform_64_1024")
LLAMAGEN = dict(LUMINA768, batch=256, heads=20, head_dim=64, prefix=1, rows=24, cols=24,
                row_end=False, period=24, threshold=100, rho_den=4, cfg_pairs=True)
TINY = dict(LUMINA768, batch=1, heads=4, head_dim=64, prefix=32, rows=16, cols=16,
            row_end=False, period=16, threshold=64, rho_den=2, amp="tiny")


def listed():
    return [
        # prefix prefill, Step 1: a text prompt of the 768 px workload, batch 8
        dict(LUMINA768, name="prefill_c128", kind="prefill", layers=8, steps=0),
        # short text prompts at a larger batch
        dict(JANUS7B, name="prefill_c64", kind="prefill", layers=8, steps=0),
        # a prompt whose length is no multiple of any tile, heads of 64
        dict(LLAMAGEN, name="prefill_c300_d64", kind="prefill", batch=16, prefix=300, layers=4,
             steps=0, cfg_pairs=False),
        # the longest prefix: an image or a document as the condition
        dict(LUMINA768, name="prefill_c2048", kind="prefill", batch=2, prefix=2048, layers=2,
             steps=0),
        # head grouping and the sizing call of the budgets, at the grouping step
        dict(LUMINA768, name="group_768", kind="group", layers=8, steps=300),
        # one image at a time: 32 heads, every layer's attention of one step
        dict(LUMINA768, name="decode_768_b1", kind="decode", batch=1, layers=32, steps=325),
        # the headline shape's attention over the compressed cache
        dict(LUMINA768, name="decode_768_b8", kind="decode", layers=16, steps=325),
        # heads of 64, guidance pairs, thousands of heads a layer
        dict(LLAMAGEN, name="decode_llamagen_b256", kind="decode", layers=4, steps=112),
        # a whole small generation: one layer of four heads, launches and latency
        dict(TINY, name="generate_tiny", kind="generate", layers=1, steps=256),
        # the headline shape, a whole image
        dict(LUMINA768, name="generate_768_b8", kind="generate", layers=8, steps=2352),
        # 1024 px, heads of 1 to 16 rows, attention-sum eviction scores
        dict(LUMINA1024, name="generate_1024_attn_sum", kind="generate", layers=4, steps=890,
             score="attn_sum"),
        # eviction on every step, batch 64
        dict(STRESS, name="generate_stress_p1", kind="generate", layers=1, steps=1100),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("prefill", "prefill", "group", "decode", "decode", "generate", "generate"))
    d = rng.choice((64, 128, 128))
    heads = rng.choice((4, 8, 16, 20, 24, 32, 32))
    case = dict(LUMINA768, kind=kind, head_dim=d, heads=heads, batch=_log(rng, 1, 32))
    if kind == "prefill":
        case["prefix"] = _log(rng, 1, 2048)
        # bounded products and inputs: at most the longest listed prefix's
        most = 128 * 2048 * 2048
        case["batch"] = max(1, min(case["batch"], most // (heads * case["prefix"] ** 2)))
        case["layers"] = rng.randint(1, 4)
        return dict(case, steps=0)
    rows, cols = rng.randint(16, 40), rng.randint(12, 40)
    row_end = rng.random() < 0.5
    row = cols + row_end
    N = rows * row
    case.update(rows=rows, cols=cols, row_end=row_end, prefix=_log(rng, 1, 400),
                rho_den=rng.choice((2, 4, 6, 8)), amp=rng.choice(("lumina", "janus")),
                budgets=rng.choice(("paper", "paper", "total", "rows_1_16")),
                period=rng.choice((1, row, row, rng.randint(2, 2 * row))),
                threshold=rng.randint(2 * row, min(N - 1, 500)))
    if kind != "generate":
        case["layers"] = rng.randint(1, 8)
        case["steps"] = case["threshold"]
        if kind == "decode":
            case["steps"] = min(N, case["threshold"] + rng.randint(1, 80))
        return case
    case["batch"] = max(1, min(case["batch"], 512 // heads))
    case.update(layers=rng.randint(1, 2), steps=min(N, case["threshold"] + rng.randint(50, 400)),
                score=rng.choice(("mean_logit", "mean_logit", "attn_sum")))
    if case["batch"] % 2 == 0:
        case["cfg_pairs"] = rng.random() < 0.3
    return case


def _workload(case):
    mode, override = BUDGETS[case["budgets"]]
    return Workload(name="case", batch=case["batch"], layers=case["layers"], heads=case["heads"],
                    head_dim=case["head_dim"], prefix_len=case["prefix"], grid_rows=case["rows"],
                    grid_cols=case["cols"], row_end=case["row_end"], period=case["period"],
                    group_threshold=case["threshold"], rho=(1, case["rho_den"]), budget_mode=mode,
                    amp_mode=case["amp"], override=override, cfg_pairs=case["cfg_pairs"],
                    score_mode=SCORES[case["score"]])


# ------------------------------------------------------------------- inputs
def _visual(wl, layer, steps, seed):
    """q, k, v of the first `steps` visual steps of a layer: bf16 [steps][B][H][d]."""
    shape = (steps, wl.batch, wl.heads, wl.head_dim)
    out = [torch.empty(shape, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    chunk = max(1, (1 << 24) // (wl.batch * wl.heads * wl.head_dim))
    for t0 in range(0, steps, chunk):
        t1 = min(steps, t0 + chunk)
        for o, x in zip(out, synth.visual_qkv(wl, layer, t0, t1, "cuda", seed)):
            o[t0:t1] = x
    return out


def _override(wl):
    ov = synth.budget_override(wl)
    if ov is None:
        return [None] * wl.layers
    return [torch.from_numpy(ov[l].reshape(-1).copy()).cuda() for l in range(wl.layers)]


class State:
    """The handle with its buffers, and the inputs of every layer."""

    def __init__(self, case, seed):
        self.case = case
        self.wl = wl = _workload(case)
        self.sess = Session(make_config(wl))
        L = range(wl.layers)
        self.qc = [synth.prefix_q(wl, l, "cuda", seed) for l in L]
        kv = [synth.prefix_kv(wl, l, "cuda", seed) for l in L]
        self.kc, self.vc = [x[0] for x in kv], [x[1] for x in kv]
        head = (wl.layers, wl.batch, wl.heads)
        # prefix attention is a case of its own, whose weights enter in bf16;
        # a generation stores the prefix (headkv_prefill)
        self.prefix_out = torch.empty((*head, wl.prefix_len, wl.head_dim), device="cuda")
        self.out = torch.empty((*head, wl.head_dim), device="cuda")
        self.q, self.k, self.v = [], [], []
        if case["steps"]:
            for l in L:
                q, k, v = _visual(wl, l, case["steps"], seed)
                self.q.append(q)
                self.k.append(k)
                self.v.append(v)
            self.override = _override(wl)

    def prefill_attn(self):
        for l in range(self.wl.layers):
            self.sess.prefill_attn(l, self.qc[l], self.kc[l], self.vc[l], self.prefix_out[l])

    def prefill(self):
        for l in range(self.wl.layers):
            self.sess.prefill(l, self.kc[l], self.vc[l])

    def steps(self, t0, t1):
        """Decode steps [t0, t1), none of them the grouping step."""
        ptr = lambda xs: [x.data_ptr() for x in xs]
        wl = self.wl
        B.headkv_run_steps(self.sess.h, t0, t1, ptr(self.q), ptr(self.k), ptr(self.v),
                           wl.batch * wl.heads * wl.head_dim, ptr(self.out), 0,
                           self.sess.stream())

    def append(self, t):
        for l in range(self.wl.layers):
            self.sess.append_and_evict(l, t, self.q[l][t], self.k[l][t], self.v[l][t])

    def group(self, t):
        for l in range(self.wl.layers):
            self.sess.score_heads(l, self.q[l][t])
            self.sess.assign_budgets(l, override=self.override[l])
            self.sess.decode_attn(l, self.q[l][t], self.out[l])

    def generate(self):
        """Prefix store and every step, the grouping step through its own calls."""
        t_g, steps = self.wl.group_threshold - 1, self.case["steps"]
        self.prefill()
        self.steps(0, min(t_g, steps))
        if steps > t_g:
            self.append(t_g)
            self.group(t_g)
            self.steps(t_g + 1, steps)


def prepare(case, seed):
    s = State(case, seed)
    if case["kind"] == "group":  # up to the grouping step's append
        s.prefill()
        s.steps(0, case["steps"] - 1)
        s.append(case["steps"] - 1)
    elif case["kind"] == "decode":  # a generation in progress
        s.generate()
        s.last_q = [q[-1].clone() for q in s.q]
        s.q, s.k, s.v = [], [], []
    return s


# --------------------------------------------------------------------- pass
def run(state):
    kind = state.case["kind"]
    sess, L = state.sess, range(state.wl.layers)
    if kind == "prefill":
        state.prefill_attn()
        return state.prefix_out
    if kind == "decode":
        for l in L:
            sess.decode_attn(l, state.last_q[l], state.out[l])
        return state.out
    if kind == "group":
        need = []
        for l in L:
            sess.score_heads(l, state.q[l][-1])
            ov = state.override[l]
            need.append(B.headkv_assign_budgets(
                sess.h, l, sess.is_local[l].data_ptr(), None if ov is None else ov.data_ptr(),
                sess.budgets[l].data_ptr(), None, 0, sess.stream())[1])
        return {"n_star": sess.n_star, "is_local": sess.is_local, "budgets": sess.budgets,
                "bytes": sum(need)}
    state.generate()
    return {"out": state.out, "n_star": sess.n_star, "is_local": sess.is_local,
            "budgets": sess.budgets, "retained": [sess.export_retained(l)[0] for l in L]}


# --------------------------------------------------------------------- work
def _budget_list(case):
    """Expected budgets of all heads of all layers (the planted share local)."""
    wl = _workload(case)
    ov = synth.budget_override(wl)
    if ov is not None:
        return [int(b) for b in ov.reshape(-1)]
    heads = wl.layers * wl.batch * wl.heads
    local = int(heads * {"lumina": 13 / 32, "janus": 0.54, "tiny": 0.5}[case["amp"]])
    rhoN, w = wl.num_visual // case["rho_den"], min(wl.recent_len, wl.num_visual)
    g = max(1, rhoN)
    if case["budgets"] == "total":
        g = max(w, (rhoN * heads - local * w) // (heads - local) // wl.row_len * wl.row_len)
    return [w] * local + [g] * (heads - local)


def work(case):
    wl = _workload(case)
    d, C, S, t_g, P = (wl.head_dim, wl.prefix_len, case["steps"], wl.group_threshold - 1,
                       wl.period)
    heads = wl.layers * wl.batch * wl.heads
    row = 2 * d  # bytes of a bf16 row
    token = 2 * row  # K and V
    if case["kind"] == "prefill":
        return {"bytes": heads * C * (3 * row + 2 * row + 4 * d),
                "flops": heads * 4 * d * C * (C + 1) // 2}
    if case["kind"] == "group":
        return {"bytes": heads * ((C + S) * row + row + 9), "flops": heads * 2 * d * (C + S)}
    budgets = _budget_list(case)

    def tokens(t):  # attended at step t, all heads
        if t < t_g:
            return heads * (C + t + 1)
        return sum(C + min(t + 1, b + (t - t_g) % P) for b in budgets)

    step_io = heads * (row + 4 * d)
    if case["kind"] == "decode":
        n = tokens(S - 1)
        return {"bytes": n * token + step_io, "flops": n * 4 * d}
    total, moved = 0, 0
    period = {}
    for t in range(S):
        # after every budget is reached the lengths repeat with the period
        key = (t - t_g) % P if t > max(budgets) + P else -1 - t
        if key not in period:
            period[key] = tokens(t)
        total += period[key]
        moved += heads * 3 * row
        if t >= t_g and (t - t_g) % P == 0:  # keys of the histories that lose tokens
            full = [b for b in budgets if t + 1 > b > wl.recent_len]
            moved += sum((b + P - wl.recent_len) * row for b in full)
    return {"bytes": heads * C * 4 * row + total * token + S * step_io + moved,
            "flops": total * 4 * d}


def tolerance(case):
    if case["kind"] == "group":
        return "exact"
    if case["kind"] == "prefill":  # attention weights rounded to bf16
        return {"rel": 5e-3, "max": 0.16}
    return {"rel": 4e-6, "max": 8e-5}  # fp32 sums; labels and retained sets exact


# -------------------------------------------------------------------- exact
def _f64(x):
    """[steps][B][H][d] -> fp64 [B*H][steps][d]"""
    return x.double().permute(1, 2, 0, 3).reshape(-1, x.shape[0], x.shape[-1])


def _prefix_attention(qc, kc, vc):
    Bn, H, C, d = qc.shape
    out = torch.empty(qc.shape, dtype=torch.float64, device="cuda")
    mask = torch.ones((C, C), dtype=torch.bool, device="cuda").tril()
    for b in range(Bn):
        s = torch.bmm(qc[b].double(), kc[b].double().transpose(1, 2).contiguous()) / math.sqrt(d)
        w = torch.softmax(s.masked_fill(~mask, -math.inf), -1)
        out[b] = torch.bmm(w, vc[b].double())
    return out


def _evict(keep, scores, lo, hi, m):
    """Drops, per head, the m lowest-scored of the positions with ranks [lo, hi)."""
    rank = keep.cumsum(1) - 1
    part = keep & (rank >= lo[:, None]) & (rank < hi[:, None])
    order = scores.masked_fill(~part, math.inf).sort(dim=1, stable=True).indices
    gone = torch.zeros_like(keep).scatter_(
        1, order, torch.arange(keep.shape[1], device="cuda")[None] < m[:, None])
    return part & gone


def _simulate(wl, layer, steps, seed, ov):
    """n*, labels and budgets, and after `steps` steps the retained set and the
    last step's attention, of every head of a layer."""
    d, C, t_g, N = wl.head_dim, wl.prefix_len, wl.group_threshold - 1, wl.num_visual
    q, k, v = (_f64(x) for x in _visual(wl, layer, steps, seed))
    kc, vc = (x.double().reshape(-1, C, d) for x in synth.prefix_kv(wl, layer, "cuda", seed))
    BH, sd = q.shape[0], math.sqrt(d)
    logits = lambda qq, kk: (kk * qq[:, None]).sum(-1) / sd
    keep = torch.zeros((BH, N), dtype=torch.bool, device="cuda")
    n_star = is_local = budget = None
    for t in range(t_g, steps, wl.period):
        if t == t_g:
            w = torch.softmax(torch.cat((logits(q[:, t], kc), logits(q[:, t], k[:, :t + 1])), 1), 1)
            reached = w.flip(1).cumsum(1) >= wl.tau
            n_star = torch.where(reached.any(1), reached.int().argmax(1) + 1, C + t + 1)
            is_local = n_star < wl.local_window
            loc = is_local.view(wl.batch, wl.heads)
            if wl.cfg_pairs:
                loc = loc[0::2].repeat_interleave(2, 0)
            rhoN, bl = N * wl.rho[0] // wl.rho[1], min(wl.recent_len, N)
            if ov is not None:
                budget = ov.long()
            else:
                g = torch.full((wl.batch, 1), max(1, rhoN), device="cuda")
                if wl.budget_mode == BUDGET_TOTAL:
                    nl = loc.sum(1, keepdim=True)
                    rest = (rhoN * wl.heads - nl * bl).clamp(min=0)
                    g = (rest // (wl.heads - nl).clamp(min=1) // wl.row_len * wl.row_len)
                    g = g.clamp(bl, N)
                budget = torch.where(loc, bl, g).reshape(-1)
            loc = loc.reshape(-1)
        keep[:, max(0, t - wl.period + 1) if t > t_g else 0:t + 1] = True
        n = keep.sum(1)
        w_eff = budget.clamp(max=wl.recent_len)
        T = (n - w_eff).clamp(min=0)
        M = (T - (budget - w_eff)).clamp(min=0)
        if not bool(M.any()):
            continue
        u, p0 = (t - t_g) // wl.period, max(0, t - wl.period + 1)
        now = keep[:, :t + 1]
        if wl.score_mode == B.HEADKV_SCORE_ATTN_SUM:
            kt = torch.cat((kc, k[:, :t + 1]), 1).transpose(1, 2).contiguous()
            pos = torch.arange(t + 1, device="cuda")
            steps_w = torch.arange(p0, t + 1, device="cuda")
            seen = now[:, None] & (pos[None] <= steps_w[:, None])[None]
            seen = torch.cat((seen.new_ones(BH, t + 1 - p0, C), seen), 2)
            w = torch.softmax((torch.bmm(q[:, p0:t + 1].contiguous(), kt) / sd)
                              .masked_fill(~seen, -math.inf), -1)
            score = w.sum(1)[:, C:]
        else:
            score = logits(q[:, p0:t + 1].sum(1), k[:, :t + 1])
        n_long = T * wl.r_s[0] // wl.r_s[1]
        n_near = T - n_long
        m_long = (M + (u & 1)) // 2
        m_near = M - m_long
        over = (m_long - n_long).clamp(min=0)
        m_long, m_near = m_long - over, m_near + over
        over = (m_near - n_near).clamp(min=0)
        m_long, m_near = m_long + over, m_near - over
        zero = torch.zeros_like(T)
        gone = _evict(now, score, zero, n_long, m_long) | _evict(now, score, n_long, T, m_near)
        old = now & (now.cumsum(1) - 1 < M[:, None])
        keep[:, :t + 1] = now & ~torch.where(loc[:, None], old, gone)
    last = steps - 1
    since = last if last < t_g else (last - t_g) % wl.period
    keep[:, last - since + (last >= t_g):last + 1] = True
    s = torch.cat((logits(q[:, last], kc),
                   logits(q[:, last], k).masked_fill(~keep[:, :steps], -math.inf)), 1)
    out = (torch.softmax(s, 1)[..., None] * torch.cat((vc, v), 1)).sum(1)
    return {"out": out.view(wl.batch, wl.heads, d), "n_star": n_star.int(),
            "is_local": is_local.to(torch.uint8), "budgets": budget.int(),
            "retained": keep.to(torch.uint8)}


def exact(case, seed):
    wl = _workload(case)
    if case["kind"] == "prefill":
        return torch.stack([_prefix_attention(synth.prefix_q(wl, l, "cuda", seed),
                                              *synth.prefix_kv(wl, l, "cuda", seed))
                            for l in range(wl.layers)])
    # a period of one step is a loop over every step, too slow in this form
    if case["kind"] == "generate" and wl.period < 4:
        return None
    ov = _override(wl)
    sim = [_simulate(wl, l, case["steps"], seed, ov[l]) for l in range(wl.layers)]
    every = lambda key: [s[key] for s in sim]
    if case["kind"] == "decode":
        return torch.stack(every("out"))
    res = {key: every(key) for key in ("n_star", "is_local", "budgets")}
    if case["kind"] == "group":
        return dict(res, bytes=None)
    return dict(res, out=torch.stack(every("out")), retained=every("retained"))
