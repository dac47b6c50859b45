"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is a batch of prompts (shared header, stacked documents, answer branches) and one call
sequence of the C ABI on it, through paper_2604_26209_amd.binding:

  decode_pass    every decode step of one attention layer, one hpd_decode_step each
  decode_step    one hpd_decode_step of one attention layer, the earlier tokens being in the cache
  serve          the first tokens of a serving loop with several layers: hpd_dynamic_begin, then per
                 token one hpd_dynamic_step per layer and one hpd_dynamic_prune on the flags
  prefill        hpd_prefix_fill and hpd_prefill_attention of one attention layer
  finetune_mask  hpd_finetune_mask: position IDs and mask of one training sequence

Values are N(0,1), as in paper_2604_26209_amd.workloads: attention cost depends on shapes only, and
queries and keys of a trained layer are normalised to that size.
"""
import math

import numpy as np
import torch

from paper_2604_26209_amd import binding as B
from paper_2604_26209_amd import workloads as W

ROPE = {"f32": 10000.0, "bf16": 500000.0}


def _case(name, kind, **kw):
    base = dict(name=name, kind=kind, dtype="bf16", hq=32, hkv=8, d=128, max_new=16, step=0, prompts=1, header=64, docs=1,
                doc_len=512, branches=16, ragged=False, mask="block", page=0, layers=1, tokens=1, struct=5)
    base.update(kw)
    if name is None:
        del base["name"]
    return base


def listed():
    return [
        # the smallest call that the benchmark has: a tiny fp32 layer, where launches and latency count
        _case("tiny_f32_pass", "decode_pass", dtype="f32", hq=4, hkv=4, d=64, max_new=8, header=16, doc_len=48, branches=4),
        # fp32 inference with 64 channels on an ordinary batch: what a validation run of a model does
        _case("f32_step", "decode_step", dtype="f32", hq=16, hkv=4, d=64, max_new=16, step=9, prompts=8, header=64, doc_len=384, branches=12),
        # Llama-3-8B-like GQA 32/8 x 128, one document per prompt: the ordinary decode step
        _case("step_llama3_8b", "decode_step", max_new=16, step=8, prompts=32, header=64, doc_len=512, branches=16),
        # four stacked documents, 96 branches per prompt
        _case("step_stacked", "decode_step", max_new=12, step=9, prompts=64, header=64, docs=4, doc_len=384, branches=24),
        # 70B-like GQA 64/8 x 128, long documents, many branches: the most arithmetic per byte
        _case("step_long_70b", "decode_step", hq=64, max_new=32, step=17, prompts=16, header=128, docs=2, doc_len=2048, branches=48),
        # the largest batch: ragged documents and branch counts, branches that end early
        _case("step_ragged", "decode_step", max_new=32, step=10, prompts=128, header=64, docs=8, doc_len=2048, branches=24, ragged=True),
        # a serving loop that learns from its sampled tokens which branches have ended; paged tails
        _case("serve_ragged_paged", "serve", max_new=32, prompts=48, header=64, docs=8, doc_len=2048, branches=24, ragged=True,
              page=8, layers=2, tokens=4),
        # the mask of the paper taken literally: a branch sees every document of its prompt
        _case("literal_step_stacked", "decode_step", mask="literal", max_new=12, step=7, prompts=64, header=64, docs=4, doc_len=384, branches=24),
        # the first inference step of the ordinary and of the long batch
        _case("prefill_llama3_8b", "prefill", max_new=16, prompts=32, header=64, doc_len=512, branches=16),
        _case("prefill_long_70b", "prefill", hq=64, max_new=32, prompts=16, header=128, docs=2, doc_len=2048, branches=48),
        # the same for ragged prompts under the literal mask
        _case("literal_prefill_ragged", "prefill", mask="literal", max_new=32, prompts=16, header=64, docs=8, doc_len=2048, branches=24, ragged=True),
        # data preparation for fine-tuning: one training sequence of about 4000 tokens
        _case("finetune_mask", "finetune_mask", max_new=16, header=2560, branches=128),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    while True:
        kind = rng.choice(["decode_pass", "decode_step", "decode_step", "decode_step", "decode_step", "serve", "prefill", "prefill",
                           "prefill", "finetune_mask"])
        kw = dict(struct=rng.randrange(1, 1 << 20), ragged=rng.random() < 0.5)
        if kind == "finetune_mask":
            kw.update(ragged=False, header=_log_int(rng, 100, 2600), branches=_log_int(rng, 4, 128), max_new=rng.randint(4, 32))
        else:
            f32 = kind == "decode_pass" or (kind == "decode_step" and rng.random() < 0.25)
            hq, hkv = rng.choice([(4, 4), (4, 2), (8, 2), (16, 4)] if f32 else [(32, 8), (32, 8), (64, 8), (40, 8), (16, 8), (16, 16)])
            top = rng.choice([4, 8, 12, 16, 24, 32])
            kw.update(dtype="f32" if f32 else "bf16", hq=hq, hkv=hkv, d=64 if f32 else 128, max_new=top,
                      step=rng.randrange(top) if kind == "decode_step" else 0,
                      prompts=_log_int(rng, 1, 4 if kind == "decode_pass" else 128), header=rng.randint(1, 200), docs=rng.randint(1, 8),
                      doc_len=_log_int(rng, 40, 512 if f32 else 3000), branches=_log_int(rng, 1, 48))
            if kind == "decode_pass":
                kw.update(max_new=rng.randint(2, 8), docs=rng.randint(1, 2), doc_len=_log_int(rng, 16, 160), branches=rng.randint(1, 8))
            if not f32 and kind in ("decode_step", "prefill") and rng.random() < 0.3:
                kw.update(mask="literal")
            if kind == "serve":
                kw.update(page=rng.choice([0, 8, 16]), layers=rng.randint(1, 4), tokens=rng.randint(2, 4))
            elif kind == "decode_step" and not f32 and kw.get("mask") != "literal" and rng.random() < 0.2:
                kw.update(page=rng.choice([8, 16, 32]))
        c = _case(None, kind, **kw)
        if kind == "finetune_mask":
            return c
        w = work(c)
        # no drawn case costs more than the largest listed one of its path; the literal mask keeps to
        # the prompts that its kernel takes (256 branches, 512 blocks of 32 keys)
        if c["mask"] == "literal" and (c["docs"] * c["branches"] > 256 or c["docs"] * (c["doc_len"] + 32) + 5 * c["docs"] * c["branches"] > 16000):
            continue
        most = {"decode_pass": (4e6, 1e9), "decode_step": (2.5e9, 1.1e11), "serve": (9e9, 4e11), "prefill": (8e9, 2.4e12)}[kind]
        if c["dtype"] == "f32":
            most = (4e7, 6e8)
        if kind == "decode_step" and c["mask"] == "literal":
            most = (2.5e9, 2e11)
        if w["bytes"] <= most[0] and w["flops"] <= most[1]:
            return c


# ---------------------------------------------------------------------------------------
# Structure of a batch
# ---------------------------------------------------------------------------------------
class _Batch:
    def __init__(self, c):
        self.c = c
        P, J, L, N, T = c["prompts"], c["docs"], c["doc_len"], c["branches"], c["max_new"]
        if c["ragged"]:
            r = np.random.default_rng(c["struct"])
            per = r.integers(1, J + 1, P)
            n = int(per.sum())
            doc_len = r.integers(max(1, L // 32), L + 1, n)
            nbr = r.integers(max(1, N // 6), N + 1, n)
            blen = r.integers(1, T + 1, int(nbr.sum()))
        else:
            per, doc_len, nbr, blen = np.full(P, J), np.full(P * J, L), np.full(P * J, N), np.full(P * J * N, T)
        self.literal = c["mask"] == "literal"
        if c["kind"] == "serve":
            blen = np.full(len(blen), T)  # how long a branch runs is not known beforehand
        self.wl = W.make_workload("case", c["dtype"], c["hq"], c["hkv"], c["d"], ROPE[c["dtype"]], T, [c["header"]] * P, per, doc_len, nbr, blen)
        wl = self.wl
        self.attr = np.random.default_rng(c["struct"] + 1).integers(1, 5, wl.n_branches).astype(np.int32) if self.literal else None
        self.branch_doc = np.repeat(np.arange(wl.n_docs), np.diff(wl.branch_ptr))
        self.doc_prompt = np.repeat(np.arange(P), np.diff(wl.doc_ptr))
        self.prompt_branch = wl.branch_ptr[wl.doc_ptr]
        self.n_names = int(self.attr.sum()) if self.literal else 0
        self.n_tok = wl.n_prefix_tokens + self.n_names

    def live(self, t):
        return np.nonzero(self.wl.branch_len > t)[0]

    def prompts(self):
        """Per prompt: (raw offset, header tokens, [(document, tokens)], (first, last + 1) branch, name lengths)."""
        raw, wl = 0, self.wl
        for p in range(wl.n_prompts):
            docs = [(d, int(wl.doc_len[d])) for d in range(wl.doc_ptr[p], wl.doc_ptr[p + 1])]
            b0, b1 = int(self.prompt_branch[p]), int(self.prompt_branch[p + 1])
            names = self.attr[b0:b1] if self.literal else np.zeros(b1 - b0, np.int32)
            yield raw, int(wl.header_len[p]), docs, (b0, b1), names
            raw += int(wl.header_len[p]) + sum(n for _, n in docs) + int(names.sum())

    def positions(self):
        """(position IDs of the prefix tokens in input order, base position of every branch)."""
        pos, base, T = [], np.zeros(self.wl.n_branches, np.int64), self.c["max_new"]
        for _, H, docs, (b0, b1), names in self.prompts():
            pos.append(np.arange(H))
            run = H
            for d, n in docs:
                pos.append(np.arange(n) + (run if self.literal else H))
                run += n
                if not self.literal:
                    base[self.wl.branch_ptr[d]:self.wl.branch_ptr[d + 1]] = H + n - 1
            if self.literal:
                owner = np.repeat(np.arange(b1 - b0), names)
                pos.append(run + np.arange(len(owner)) + owner * T)
                base[b0:b1] = run + np.cumsum(names) - 1 + np.arange(b1 - b0) * T
        return np.concatenate(pos), base


def _draws(c, b, seed):
    """Every random tensor of a case, on the GPU, from the seed alone."""
    if c["kind"] == "finetune_mask":
        # the lengths belong to the case, their order to the seed: one size of sequence per case
        r, order = np.random.default_rng(c["struct"]), np.random.default_rng(int(seed) % (1 << 32))
        return {"attr": order.permutation(r.integers(1, 5, c["branches"])),
                "value": order.permutation(r.integers(0, c["max_new"] + 1, c["branches"]))}
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dt)

    hq, hkv, d, n_br = c["hq"], c["hkv"], c["d"], b.wl.n_branches
    x = {"layers": []}
    for _ in range(c["layers"]):
        y = {"k_raw": normal(b.n_tok, hkv, d), "v_raw": normal(b.n_tok, hkv, d)}
        if c["kind"] == "prefill":
            y["q"] = normal(b.n_tok, hq, d)
        elif c["kind"] == "serve":
            steps = range(c["tokens"])
            y["q"] = [normal(n_br, hq, d) for _ in steps]
            y["k"], y["v"] = [normal(n_br, hkv, d) for _ in steps], [normal(n_br, hkv, d) for _ in steps]
        else:
            steps = range(c["max_new"] if c["kind"] == "decode_pass" else c["step"] + 1)
            new = range(c["max_new"]) if c["kind"] == "decode_pass" else [c["step"]]
            n = [len(b.live(t)) for t in steps]
            y["k"], y["v"] = [normal(n[t], hkv, d) for t in steps], [normal(n[t], hkv, d) for t in steps]
            y["q"] = {t: normal(n[t], hq, d) for t in new}
        x["layers"].append(y)
    if c["kind"] == "serve":  # about one branch in eight ends with every token
        x["finished"] = [(torch.rand(n_br, generator=g, device="cuda") < 0.125).to(torch.uint8) for _ in range(c["tokens"] - 1)]
    if c["page"]:
        per = -(-c["max_new"] // c["page"])
        x["table"] = torch.randperm(n_br * per, generator=g, device="cuda").to(torch.int32).view(n_br, per).contiguous()
    return x


def _pool(x):
    """A pool with the element type that its bits have."""
    return x.view(torch.float16) if x.dtype == torch.bfloat16 else x


def prepare(case, seed):
    if case["kind"] == "finetune_mask":
        x = _draws(case, None, seed)
        S = case["header"] + int(x["attr"].sum() + x["value"].sum())
        return {"case": case, "x": x, "pos": torch.empty(S, dtype=torch.int32, device="cuda"),
                "mask": torch.empty(S, S, dtype=torch.uint8, device="cuda")}
    b = _Batch(case)
    x = _draws(case, b, seed)
    literal = b.literal
    layout = B.layout_from_workload(b.wl, pos_mode=B.HPD_POS_PAPER_GAP if literal else B.HPD_POS_CONTIG, attr_len=b.attr,
                                    mask_mode=B.HPD_MASK_PAPER if literal else B.HPD_MASK_BLOCK)
    if case["page"]:
        B.hpd_set_tail_pages(layout, case["page"], x["table"].numel(), x["table"])
    s = {"case": case, "layout": layout, "x": x, "layers": []}
    hq, d = case["hq"], case["d"]
    for y in x["layers"]:
        pools = B.alloc_pools(layout)
        for p in pools:
            p.zero_()
        kp, vp, kt, vt = pools
        z = {"pools": pools}
        if case["kind"] == "prefill":
            z["out"] = torch.zeros(b.n_tok, hq, d, dtype=y["q"].dtype, device="cuda")
        else:
            B.hpd_prefix_fill(layout, y["k_raw"], y["v_raw"], kp, vp)
            if case["kind"] == "decode_step":  # the tokens before this step
                for t in range(case["step"]):
                    B.hpd_kv_append(layout, t, y["k"][t], y["v"][t], kt, vt)
            qs = y["q"].items() if isinstance(y["q"], dict) else enumerate(y["q"])
            z["out"] = {t: torch.zeros_like(q) for t, q in qs}
            del y["k_raw"], y["v_raw"]  # a decoding program has them in the cache only
        s["layers"].append(z)
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "finetune_mask":
        x = s["x"]
        B.hpd_finetune_mask(c["header"], x["attr"], x["value"], c["max_new"], s["pos"], s["mask"])
        return {"pos": s["pos"], "mask": s["mask"]}
    lay, kind, got = s["layout"], c["kind"], []
    if kind == "serve":
        B.hpd_dynamic_begin(lay)
        for t in range(c["tokens"]):
            for y, z in zip(s["x"]["layers"], s["layers"]):
                B.hpd_dynamic_step(lay, t, y["q"][t], y["k"][t], y["v"][t], *z["pools"], z["out"][t])
            if t + 1 < c["tokens"]:
                B.hpd_dynamic_prune(lay, s["x"]["finished"][t])
    for y, z in zip(s["x"]["layers"], s["layers"]):
        kp, vp, kt, vt = z["pools"]
        if kind == "prefill":
            B.hpd_prefix_fill(lay, y["k_raw"], y["v_raw"], kp, vp)
            B.hpd_prefill_attention(lay, y["q"], kp, vp, z["out"])
            got.append({"out": z["out"], "k_prefix": _pool(kp), "v_prefix": _pool(vp)})
            continue
        if kind != "serve":
            for t in z["out"]:
                B.hpd_decode_step(lay, t, y["q"][t], y["k"][t], y["v"][t], kp, vp, kt, vt, z["out"][t])
        got.append({"out": list(z["out"].values()), "k_tail": _pool(kt), "v_tail": _pool(vt)})
    return got


# ---------------------------------------------------------------------------------------
# The work that a pass cannot do without
# ---------------------------------------------------------------------------------------
def _step_work(c, b, t, live):
    """Bytes and operations of one decode step: every prefix token and every tail token that a live
    row sees once, queries, new keys and values in, new keys, values and outputs out."""
    wl = b.wl
    eb = 4 if c["dtype"] == "f32" else 2
    tok = 2 * c["hkv"] * c["d"] * eb
    if len(live) == 0:
        return 0, 0
    docs = np.unique(b.branch_doc[live])
    prompts = np.unique(b.doc_prompt[docs])
    if not b.literal:
        seen = int(wl.header_len[prompts].sum() + wl.doc_len[docs].sum()) + len(live) * t
        doc = b.branch_doc[live]
        keys = int((wl.header_len[b.doc_prompt[doc]] + wl.doc_len[doc] + t + 1).sum())
    else:
        csum = np.concatenate([[0], np.cumsum(np.minimum(wl.branch_len, t + 1) + b.attr)])
        dsum = np.concatenate([[0], np.cumsum(wl.doc_len.astype(np.int64))])
        plen = wl.header_len + dsum[wl.doc_ptr[1:]] - dsum[wl.doc_ptr[:-1]]
        p_of = b.doc_prompt[b.branch_doc[live]]
        own = csum[live + 1] - csum[b.prompt_branch[p_of]]
        keys = int((plen[p_of] + own).sum())
        last = np.zeros(wl.n_prompts, np.int64)
        np.maximum.at(last, p_of, own)
        seen = int(plen[prompts].sum() + last[prompts].sum()) - len(live)
    rows = len(live) * (2 * c["hq"] * c["d"] * eb + 2 * tok)
    return seen * tok + rows, 4 * c["d"] * c["hq"] * keys


def work(case):
    c = case
    if c["kind"] == "finetune_mask":
        x = _draws(c, None, 0)
        S = c["header"] + int(x["attr"].sum() + x["value"].sum())
        return {"bytes": S * S + 4 * S, "flops": 0}
    b = _Batch(c)
    if c["kind"] == "prefill":
        row = 2 * c["d"]
        total = b.n_tok * row * (2 * c["hq"] + 4 * c["hkv"])
        pairs = 0
        for _, H, docs, _, names in b.prompts():
            if b.literal:
                S = H + sum(n for _, n in docs) + int(names.sum())
                pairs += S * (S + 1) // 2
            else:
                pairs += H * (H + 1) // 2 + sum(n * H + n * (n + 1) // 2 for _, n in docs)
        return {"bytes": total, "flops": 4 * c["d"] * c["hq"] * pairs}
    if c["kind"] == "serve":
        got = [_step_work(c, b, t, np.arange(int(b.wl.n_branches * 0.875 ** t))) for t in range(c["tokens"])]
    else:
        got = [_step_work(c, b, t, b.live(t)) for t in (range(c["max_new"]) if c["kind"] == "decode_pass" else [c["step"]])]
    return {"bytes": c["layers"] * sum(g[0] for g in got), "flops": c["layers"] * sum(g[1] for g in got)}


def tolerance(case):
    if case["kind"] == "finetune_mask":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 4e-5}
    # bf16 outputs (an error of 2^-9 at most from their rounding alone, 1.7e-3 on the average), keys
    # rounded to bf16 on their way into the cache
    return {"rel": 8e-3, "max": 8e-2}


# ---------------------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------------------
class _Exact:
    def __init__(self, c, b):
        self.c, self.b = c, b
        pos, self.base = b.positions()
        self.pos = torch.from_numpy(pos).cuda()
        i = torch.arange(c["d"] // 2, device="cuda", dtype=torch.float64)
        self.theta = ROPE[c["dtype"]] ** (-2.0 * i / c["d"])

    def rotate(self, x, pos):
        """x [n, heads, d] at position IDs [n]."""
        a = pos.double()[:, None, None] * self.theta
        lo, hi = x.double().chunk(2, -1)
        return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)

    def cached(self, k):
        """The rotated key as the cache holds it: in the precision of the inputs."""
        return k if self.c["dtype"] == "f32" else k.to(torch.bfloat16).double()

    def heads(self, x):
        """[n, hkv, d] -> [hkv, n, d]"""
        return x.transpose(0, 1).contiguous()

    def attend(self, q, parts):
        """q [hkv, rows, d]; parts: (k [hkv, n, d], v, visible [rows, n] or None).  Softmax over all parts."""
        s = [(q @ k.transpose(1, 2).contiguous()) / math.sqrt(self.c["d"]) for k, _, _ in parts]
        for x, (_, _, ok) in zip(s, parts):
            if ok is not None:
                x.masked_fill_(~ok, -math.inf)
        m = torch.stack([x.amax(-1) for x in s]).amax(0)[..., None]
        s = [(x - m).exp_() for x in s]
        total = sum(x.sum(-1, keepdim=True) for x in s)
        return sum(x @ v for x, (_, v, _) in zip(s, parts)) / total

    def grouped(self, q):
        """[n, hq, d] -> [hkv, n * G, d]"""
        n, hkv = q.shape[0], self.c["hkv"]
        return q.view(n, hkv, -1, self.c["d"]).transpose(0, 1).reshape(hkv, -1, self.c["d"]).contiguous()

    def ungrouped(self, o, n):
        return o.view(self.c["hkv"], n, -1, self.c["d"]).transpose(0, 1).reshape(n, self.c["hq"], self.c["d"])

    def decode(self, t, live, q, prefix, tail_k, tail_v, length):
        """prefix: (cached keys, values) [hkv, tokens, d] of all prompts; tail_k / tail_v [B, hkv, T, d]; `length`:
        tokens in memory of every branch."""
        c, b, G = self.c, self.b, self.c["hq"] // self.c["hkv"]
        qr = self.rotate(q, torch.from_numpy(self.base[live] + 1 + t).cuda())
        out = torch.zeros(len(live), c["hq"], c["d"], dtype=torch.float64, device="cuda")
        for raw, H, docs, (b0, b1), names in b.prompts():
            n_pre = H + sum(n for _, n in docs)
            at = raw + H
            for d, n in ([(None, n_pre - H)] if b.literal else docs):
                lo, hi = (b0, b1) if d is None else (int(b.wl.branch_ptr[d]), int(b.wl.branch_ptr[d + 1]))
                r0, r1 = np.searchsorted(live, [lo, hi])
                if r1 > r0:
                    rows = torch.from_numpy(live[r0:r1]).cuda()
                    row_b = rows.repeat_interleave(G)
                    parts = [tuple(x[:, i:j] for x in prefix) + (None,) for i, j in ((raw, raw + H), (at, at + n)) if j > i]
                    if b.literal:
                        owner = torch.from_numpy(np.repeat(np.arange(b0, b1), names)).cuda()
                        j = at + n
                        parts.append(tuple(x[:, j:j + len(owner)] for x in prefix) + (owner[None] <= row_b[:, None],))
                    # tails: of the document's (literal: the prompt's) branches
                    tk, tv = (x[lo:hi, :, :t + 1].double().transpose(0, 1).reshape(c["hkv"], -1, c["d"]) for x in (tail_k, tail_v))
                    kb = torch.arange(lo, hi, device="cuda").repeat_interleave(t + 1)
                    kt = torch.arange(t + 1, device="cuda").repeat(hi - lo)
                    ok = (kb[None] <= row_b[:, None]) if b.literal else (kb[None] == row_b[:, None])
                    parts.append((tk, tv, ok & (kt < length[kb])[None]))
                    out[r0:r1] = self.ungrouped(self.attend(self.grouped(qr[r0:r1]), parts), r1 - r0)
                at += n
        return out

    def prefill(self, q, k, v):
        """k: cached keys [hkv, tokens, d]."""
        c, b, G = self.c, self.b, self.c["hq"] // self.c["hkv"]
        qr = self.rotate(q, self.pos)
        out = torch.zeros(b.n_tok, c["hq"], c["d"], dtype=torch.float64, device="cuda")
        for raw, H, docs, _, names in b.prompts():
            spans = [(raw, H)]
            at = raw + H
            for _, n in docs:
                spans.append((at, n))
                at += n
            if b.literal:
                spans = [(raw, at - raw + int(names.sum()))]
            for first, n in spans:
                if n == 0:
                    continue
                tri = torch.ones(n, n, dtype=torch.bool, device="cuda").tril_().repeat_interleave(G, 0)
                qg = self.grouped(qr[first:first + n])
                for h in range(c["hkv"]):  # a head at a time: the scores of a prompt are large
                    parts = [(k[h:h + 1, first:first + n], v[h:h + 1, first:first + n], tri)]
                    if first != raw:
                        parts.append((k[h:h + 1, raw:raw + H], v[h:h + 1, raw:raw + H], None))
                    o = self.attend(qg[h:h + 1], parts)
                    out[first:first + n, h * G:(h + 1) * G] = o.view(n, G, c["d"])
        return out

    def prefix_pools(self, k, v):
        """The prefix pools, laid out as the header file says: [hkv][slots][d] and [hkv][slots / 8][d][8]."""
        slots, first, where = 0, 0, []
        for _, H, docs, _, names in self.b.prompts():
            for n in [H] + [n for _, n in docs] + ([int(names.sum())] if self.b.literal else []):
                where.append(np.arange(n) + slots)
                slots += -(-n // 32) * 32
                first += n
        slots += 128
        at = torch.from_numpy(np.concatenate(where)).cuda()
        hkv, d = self.c["hkv"], self.c["d"]
        kp = torch.zeros(hkv, slots, d, dtype=torch.float64, device="cuda")
        vp = torch.zeros(hkv, slots, d, dtype=torch.float64, device="cuda")
        kp[:, at], vp[:, at] = k, v
        return kp.reshape(-1), vp.view(hkv, slots // 8, 8, d).transpose(2, 3).reshape(-1)

    def tail_pool(self, x, table):
        """[B, hkv, T, d] as the pool holds it."""
        if table is None:
            return x.reshape(-1)
        n_br, hkv, T, d = x.shape
        page, per = self.c["page"], table.shape[1]
        y = torch.zeros(n_br, hkv, per * page, d, dtype=x.dtype, device="cuda")
        y[:, :, :T] = x
        out = torch.zeros(table.numel(), hkv, page, d, dtype=x.dtype, device="cuda")
        out[table.long().reshape(-1)] = y.view(n_br, hkv, per, page, d).transpose(1, 2).reshape(-1, hkv, page, d)
        return out.reshape(-1)


def exact(case, seed):
    c = case
    if c["kind"] == "finetune_mask":
        x = _draws(c, None, seed)
        owner, k, end, pos, nxt = [np.full(c["header"], -1)], [np.zeros(c["header"], int)], 0, [np.arange(c["header"])], c["header"]
        for n, (a, v) in enumerate(zip(x["attr"], x["value"])):
            pos += [nxt + n * c["max_new"] + np.arange(a), nxt + n * c["max_new"] + a - 1 + np.arange(1, v + 1)]
            nxt += a
            owner += [np.full(a + v, n)]
            k += [np.zeros(a, int), np.arange(1, v + 1)]
        owner, k, pos = (torch.from_numpy(np.concatenate(y)).cuda() for y in (owner, k, pos))
        i = torch.arange(len(k), device="cuda")
        value, name = k > 0, (k == 0) & (owner >= 0)
        ok = i[None] <= i[:, None]
        ok &= ~(value[None] & name[:, None])
        ok &= ~(value[None] & value[:, None] & (owner[None] < owner[:, None]) & (k[None] > k[:, None]))
        return {"pos": pos.to(torch.int32), "mask": ok.to(torch.uint8)}
    b = _Batch(c)
    x, e = _draws(c, b, seed), _Exact(c, b)
    got = []
    T, hkv, d, n_br = c["max_new"], c["hkv"], c["d"], b.wl.n_branches
    for y in x["layers"]:
        k64 = e.heads(e.rotate(y["k_raw"], e.pos))
        v64 = e.heads(y["v_raw"].double())
        if c["kind"] == "prefill":
            kp, vp = e.prefix_pools(k64, v64)
            got.append({"out": e.prefill(y["q"], e.cached(k64), v64), "k_prefix": kp, "v_prefix": vp})
            continue
        prefix = (e.cached(k64), v64)
        tk, tc, tv = (torch.zeros(n_br, hkv, T, d, dtype=torch.float64, device="cuda") for _ in range(3))
        length = torch.zeros(n_br, dtype=torch.int64, device="cuda")
        outs, live = [], np.arange(n_br)
        for t in range(len(y["k"])):
            if c["kind"] != "serve":
                live = b.live(t)
            rows = torch.from_numpy(live).cuda()
            k = e.rotate(y["k"][t][:len(live)], torch.from_numpy(e.base[live] + 1 + t).cuda())
            tk[rows, :, t], tc[rows, :, t], tv[rows, :, t] = k, e.cached(k), y["v"][t][:len(live)].double()
            length[rows] = t + 1
            if c["kind"] == "serve" or t in y["q"]:
                o = torch.zeros(y["q"][t].shape, dtype=torch.float64, device="cuda")
                o[:len(live)] = e.decode(t, live, y["q"][t][:len(live)], prefix, tc, tv, length)
                outs.append(o)
            if c["kind"] == "serve" and t + 1 < c["tokens"]:
                live = live[x["finished"][t][:len(live)].cpu().numpy() == 0]
        table = x.get("table")
        got.append({"out": outs, "k_tail": e.tail_pool(tk, table), "v_tail": e.tail_pool(tv, table)})
    return got
