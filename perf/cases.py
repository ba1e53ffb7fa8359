"""The work that users of this library have it do, as measured cases.

Each case is one pass through the public entry points of ``NgpuLM``: the
batched query, the fused greedy step launched once per frame, the whole greedy
decode, and the beam expansion.  The language models are generated here (closed
and close to normalised, Zipf-distributed tokens, random continuation weights);
a program loads its model once and keeps it, so a model is built once per
process and shared by the states of all cases that use it.  Query states are
uniform over the model's states, decodes start at the start state, and ASR
scores are log-softmax rows of N(0, 3) logits with a boosted blank.
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2505_22857_amd as ng

DEV = "cuda"
MODES = {"plain": ng.NGPU_FUSION_PLAIN, "ctc": ng.NGPU_FUSION_CTC,
         "transducer": ng.NGPU_FUSION_TRANSDUCER, "aed": ng.NGPU_FUSION_AED}
# The 6-gram over 1024 BPE tokens with 20 million n-grams is the largest model
# that the benchmark and the tests use (1.3 GB on the GPU).
BIG = {"vocab": 1024, "order": 6, "ngrams": 20_000_000, "markers": False}


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # a handful of hypotheses on a tiny command model: the smallest call
        {"name": "query_4_trigram128", "kind": "query", "vocab": 128, "order": 3, "ngrams": 5_000,
         "markers": False, "batch": 4},
        # one call of a batched decoder over the large model: latency-bound
        {"name": "query_512_sixgram", "kind": "query", **BIG, "batch": 512},
        # rescoring in bulk: 128 such batches in one call, bound by the output
        {"name": "query_65536_sixgram", "kind": "query", **BIG, "batch": 65536},
        # a 10-gram over an odd vocabulary at a ragged batch: deep backoff chains
        {"name": "query_3001_tengram999", "kind": "query", "vocab": 999, "order": 10, "ngrams": 2_000_000,
         "markers": False, "batch": 3001},
        # streaming CTC recognition of 256 utterances, one launch per frame
        {"name": "step_ctc_256_sixgram", "kind": "step", **BIG, "mode": "ctc", "batch": 256, "frames": 32,
         "blank": 4.0},
        # an attention decoder's greedy search: the row of each step comes from
        # the network, and <eos> is scored with the final weight
        {"name": "step_aed_40_fivegram500", "kind": "step", "vocab": 500, "order": 5, "ngrams": 300_000,
         "markers": True, "mode": "aed", "batch": 40, "frames": 24, "blank": 0.0},
        # offline CTC decoding of a batch of utterances in one call
        {"name": "decode_ctc_256x1000_sixgram", "kind": "decode", **BIG, "mode": "ctc", "batch": 256,
         "frames": 1000, "blank": 4.0, "ragged": False},
        # offline CTC decoding of a whole corpus shard in one call
        {"name": "decode_ctc_4096x200_sixgram", "kind": "decode", **BIG, "mode": "ctc", "batch": 4096,
         "frames": 200, "blank": 4.0, "ragged": False},
        # a transducer's label loop over utterances of different lengths with
        # a large word-piece vocabulary, most frames blank
        {"name": "decode_rnnt_700x150_trigram4096", "kind": "decode", "vocab": 4096, "order": 3,
         "ngrams": 1_000_000, "markers": False, "mode": "transducer", "batch": 700, "frames": 150,
         "blank": 11.0, "ragged": True},
        # plain fusion of a small batch over a small model, all steps in one call
        {"name": "decode_plain_32x200_fourgram", "kind": "decode", "vocab": 1024, "order": 4, "ngrams": 200_000,
         "markers": False, "mode": "plain", "batch": 32, "frames": 200, "blank": 0.0, "ragged": False},
        # beam search over 256 utterances with a beam of 4
        {"name": "topk_1024x16_sixgram", "kind": "topk", **BIG, "batch": 1024, "k": 16},
        # the same for a large word-piece vocabulary
        {"name": "topk_320x32_fourgram5000", "kind": "topk", "vocab": 5000, "order": 4, "ngrams": 1_000_000,
         "markers": False, "batch": 320, "k": 32},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("query", "step", "decode", "topk"))
    mode = rng.choice(("plain", "ctc", "transducer", "aed"))
    if mode != "aed" and rng.random() < 0.4:
        c = dict(BIG)
    else:
        vocab = _log_int(rng, 100, 6000)
        if rng.random() < 0.4:
            vocab = (vocab + 127) // 128 * 128
        c = {"vocab": vocab, "order": rng.randint(2, 10 if vocab <= 4000 else 8),
             "ngrams": _log_int(rng, 8_000, 2_000_000), "markers": mode == "aed"}
    V = c["vocab"]
    if kind == "query":
        return {"kind": kind, **c, "batch": _log_int(rng, 1, min(65536, (1 << 26) // V))}
    if kind == "topk":
        return {"kind": kind, **c, "batch": _log_int(rng, 4, 4096), "k": min(V, _log_int(rng, 1, 200))}
    blank = 0.0 if mode in ("plain", "aed") else rng.choice((4.0, 11.0))
    if kind == "step":
        return {"kind": kind, **c, "mode": mode, "batch": _log_int(rng, 1, 4096), "frames": rng.randint(8, 32),
                "blank": blank}
    batch = _log_int(rng, 4, 4096)
    frames = max(8, min(_log_int(rng, 40, 1000), 800_000 * 1024 // (batch * V)))
    return {"kind": kind, **c, "mode": mode, "batch": batch, "frames": frames, "blank": blank,
            "ragged": rng.random() < 0.5}


# ---------------------------------------------------------------- the models

class _Level:
    """The n-grams of one order, sorted by (prefix, token): row of the prefix
    and of the suffix one order down, last token, weight, backoff weight."""

    def __init__(self, pid, tok, sid, w, cum):
        self.pid, self.tok, self.sid, self.w, self.cum = pid, tok, sid, w, cum
        self.b = torch.zeros_like(w)
        self.begin = self.end = None     # per row: its continuations in the next level
        self.state = None                # per row: its state id (-1: </s> ends the n-gram)


def _segment_sums(x, begin, end):
    """Sums of x[begin:end] per segment, in fixed point so that they do not
    depend on the order of the additions."""
    q = torch.cumsum((x * 2.0 ** 36).long(), 0)
    q = torch.cat([torch.zeros(1, dtype=torch.int64, device=x.device), q])
    return (q[end] - q[begin]).double() * 2.0 ** -36


def _counts(vocab, order, ngrams):
    """N-grams per order: growing to order 4, then falling, bigrams at most
    three quarters of all pairs."""
    if order == 1:
        return [vocab]
    left = max(order - 1, ngrams - vocab)
    share = [1.6 ** (min(k, 4) - 2) * 0.6 ** max(0, k - 4) for k in range(2, order + 1)]
    bigrams = min(int(left * share[0] / sum(share)), vocab * vocab * 3 // 4)
    rest = left - bigrams
    return [vocab, max(1, bigrams)] + [max(1, int(rest * s / sum(share[1:]))) for s in share[1:]]


def _pick_pairs(lv, need, ctx_ok, tok_ok, g):
    """Bigrams drawn without replacement, in proportion to P(c) P(v)."""
    n = lv.tok.numel()
    clock = torch.empty((n, n), dtype=torch.float64, device=DEV).exponential_(generator=g).log_()
    clock -= lv.cum[:, None]
    clock -= lv.w.double()[None, :]
    clock[~ctx_ok] = math.inf
    clock[:, ~tok_ok] = math.inf
    clock = clock.reshape(-1)
    need = min(need, int(ctx_ok.sum()) * int(tok_ok.sum()))
    return torch.sort(torch.sort(clock, stable=True).indices[:need]).values


def _pick_longer(lv, low, need, ctx_ok, g):
    """N-grams (c, v) with c and c[1:] + v listed, drawn in proportion to
    P(c) P(v | c[1:]) until there are ``need`` distinct ones (or nearly)."""
    n = lv.tok.numel()
    lo, hi = low.begin[lv.sid], low.end[lv.sid]
    grain = (lv.w.double().exp() * 2.0 ** 38).long() + 1
    cum = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), torch.cumsum(grain, 0)])
    mass = (cum[hi] - cum[lo]).double()
    weight = (lv.cum - lv.cum.max()).exp() * mass
    weight = (weight / weight.max() * 2.0 ** 38).long() + 1
    weight = torch.where(ctx_ok & (hi > lo), weight, torch.zeros_like(weight))
    cdf = torch.cumsum(weight, 0)
    total = int(cdf[-1])
    seen = torch.zeros(0, dtype=torch.int64, device=DEV)
    if total == 0:
        return seen
    batch = int(1.5 * need) + 1024
    for _ in range(24):
        c = torch.searchsorted(cdf, torch.randint(0, total, (batch,), generator=g, device=DEV), right=True)
        a, z = cum[lo[c]], cum[hi[c]]
        u = a + (torch.rand(batch, generator=g, device=DEV, dtype=torch.float64) * (z - a).double()).long()
        y = torch.searchsorted(cum, u.clamp_(max=int(cum[-1]) - 1), right=True) - 1
        y = torch.minimum(torch.maximum(y, lo[c]), hi[c] - 1)
        seen = torch.unique(torch.cat([seen, c * n + y]))
        if seen.numel() >= need:
            keep = torch.randperm(seen.numel(), generator=g, device=DEV)[:need]
            return torch.sort(seen[keep]).values
        batch = min(max(int(4.0 * (need - seen.numel())), 1 << 18), 1 << 25)
    return seen


class Model:
    """A generated model and its handle, uploaded once."""

    def __init__(self, vocab, order, ngrams, markers):
        V = self.V = vocab
        self.N, self.markers = order, markers
        counts = _counts(vocab, order, ngrams)
        g = torch.Generator(device=DEV)
        g.manual_seed(V * 1_000_003 + order * 10_007 + ngrams)
        perm = torch.randperm(V, generator=g, device=DEV)
        rank = torch.arange(1, V + 1, dtype=torch.float64, device=DEV)
        p = torch.empty(V, dtype=torch.float64, device=DEV)
        p[perm] = 1.0 / rank / math.fsum(1.0 / r for r in range(1, V + 1))
        tok = torch.arange(V + 2 if markers else V, dtype=torch.int32, device=DEV)
        if markers:   # token V is <s> (opens contexts only), V + 1 is </s> (predicted only)
            ends = torch.tensor([1e-99, 0.04], dtype=torch.float64, device=DEV)
            p = torch.cat([p * 0.96, ends])
        w = p.log().float()
        cum = w.double().clone()
        if markers:
            cum[V] = math.log(0.05)
        zero = torch.zeros(tok.numel(), dtype=torch.int64, device=DEV)
        root = _Level(torch.zeros(1, dtype=torch.int64, device=DEV), tok[:1], zero[:1], w[:1], cum[:1])
        root.begin = torch.zeros(1, dtype=torch.int64, device=DEV)
        root.end = torch.full((1,), tok.numel(), dtype=torch.int64, device=DEV)
        self.levels = [root, _Level(zero, tok, zero, w, cum)]
        for k in range(2, order + 1):
            lv, low = self.levels[k - 1], self.levels[k - 2]
            n = lv.tok.numel()
            ctx_ok = lv.tok != V + 1
            if k == 2:
                keys = _pick_pairs(lv, counts[1], ctx_ok, lv.tok != V, g)
            else:
                keys = _pick_longer(lv, low, counts[k - 1], ctx_ok, g)
            pid, sid = keys // n, keys % n
            rows = torch.arange(n, dtype=torch.int64, device=DEV)
            lv.begin = torch.searchsorted(pid, rows)
            lv.end = torch.searchsorted(pid, rows, right=True)
            p_low = lv.w[sid].double().exp()
            raw = p_low * torch.randn(pid.numel(), generator=g, device=DEV, dtype=torch.float64).exp() + 1e-9
            m = 0.5 + 0.45 * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
            w = (m[pid] * raw / _segment_sums(raw, lv.begin, lv.end)[pid]).clamp_(max=0.999).log().float()
            left = (1.0 - _segment_sums(p_low, lv.begin, lv.end)).clamp_(min=1e-3)
            lv.b = torch.where(lv.end > lv.begin, (1.0 - m).log() - left.log(), torch.zeros_like(m)).float()
            self.levels.append(_Level(pid, lv.tok[sid], sid, w, lv.cum[pid] + w.double()))
        last = self.levels[order]
        last.begin = last.end = torch.zeros(last.tok.numel(), dtype=torch.int64, device=DEV)
        # state ids: the empty context, then the contexts in (order, tuple) order
        self.first, self.S = [0], 1
        for lv in self.levels[1:order]:
            self.first.append(self.S)
            ok = lv.tok != V + 1
            lv.state = torch.where(ok, torch.cumsum(ok.long(), 0) - 1 + self.S, torch.full_like(lv.pid, -1))
            lv.row_of = torch.nonzero(ok).flatten()
            self.S += int(lv.row_of.numel())
        self.lm = self._load()
        assert self.lm.num_states == self.S
        self.start = self.lm.start_state

    def _load(self):
        order, tokens, w, b, cols = [], [], [], [], None
        for k, lv in enumerate(self.levels[1:], 1):
            cols = lv.tok[:, None] if k == 1 else torch.cat([cols[lv.pid], lv.tok[:, None]], 1)
            order.append(torch.full((lv.tok.numel(),), k, dtype=torch.int32))
            t = torch.full((lv.tok.numel(), self.N), -1, dtype=torch.int32, device=DEV)
            t[:, :k] = cols
            tokens.append(t.cpu())
            w.append(lv.w.cpu())
            b.append(lv.b.cpu())
        arrays = [torch.cat(x).numpy() for x in (order, tokens, w, b)]
        return ng.NgpuLM(self.V, self.N, *arrays, bos_eos=self.markers).upload(DEV)

    def mean_chain(self):
        """Mean number of levels and of arcs (orders above 2) on a state's chain."""
        states = torch.randint(0, self.S, (4096,), generator=torch.Generator().manual_seed(1)).to(DEV)
        levels = arcs = 0.0
        for j, ok, rows in self.chain(states):
            if j >= 2:
                lv = self.levels[j]
                levels += float(ok.double().mean())
                arcs += float(((lv.end - lv.begin)[rows] * ok).double().mean())
        return levels, arcs

    def chain(self, states):
        """(order, which states have a context of it, its rows), shortest context first."""
        order = torch.zeros_like(states)
        for k in range(1, self.N):
            order = torch.where(states >= self.first[k], torch.full_like(order, k), order)
        out, rows = [], torch.zeros_like(states)
        for k in range(self.N - 1, 0, -1):
            lv = self.levels[k]
            here = lv.row_of[(states - self.first[k]).clamp(0, lv.row_of.numel() - 1)]
            above = self.levels[k + 1].sid[rows] if k + 1 < self.N else here
            rows = torch.where(order == k, here, above)
            ok = order >= k
            rows = torch.where(ok, rows, torch.zeros_like(rows))
            out.append((k, ok, rows))
        return out[::-1]

    def query64(self, states):
        """The backoff query in 64 bits: scores and next states [B, V], and the </s> scores [B]."""
        V, states = self.V, states.long()
        B = states.numel()
        width = V + 2 if self.markers else V
        uni = self.levels[1]
        score = uni.w.double()[None, :].repeat(B, 1)
        one = uni.state if self.N > 1 else torch.zeros(width, dtype=torch.int64, device=DEV)
        to = one[None, :].repeat(B, 1)
        for j, ok, rows in self.chain(states):
            lv, up = self.levels[j], self.levels[j + 1]
            score += torch.where(ok, lv.b[rows].double(), 0.0)[:, None]
            n = (lv.end - lv.begin)[rows] * ok
            b = torch.repeat_interleave(torch.arange(B, device=DEV), n)
            at = torch.arange(b.numel(), device=DEV) - (torch.cumsum(n, 0) - n)[b] + lv.begin[rows][b]
            tok = up.tok[at].long()
            score[b, tok] = up.w[at].double()
            to[b, tok] = up.state[at] if j + 1 < self.N else lv.state[up.sid[at]]
        return score[:, :V], to[:, :V], score[:, V + 1] if self.markers else None


@functools.lru_cache(maxsize=12)
def _model(vocab, order, ngrams, markers):
    return Model(vocab, order, ngrams, markers)


def model_of(case):
    return _model(case["vocab"], case["order"], case["ngrams"], case["markers"])


# ---------------------------------------------------------------- measuring

def _asr(shape, blank, g):
    x = torch.randn(shape, generator=g, device=DEV)
    x *= 3.0
    if blank:
        x[..., -1] += blank
    return torch.log_softmax(x, -1)


def _classes(case):
    return case["vocab"] + (0 if case["mode"] == "plain" else 1)


LAM = 0.5


def prepare(case, seed):
    m = model_of(case)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    B, V = case["batch"], case["vocab"]
    s = {"lm": m.lm, "case": case, "mode": MODES[case.get("mode", "plain")]}
    if case["kind"] in ("query", "topk"):
        s["states"] = torch.randint(0, m.S, (B,), generator=g, device=DEV).int()
        if case["kind"] == "query":
            s["scores"] = torch.empty((B, V), dtype=torch.float32, device=DEV)
            s["next"] = torch.empty((B, V), dtype=torch.int32, device=DEV)
        else:
            s["asr"] = _asr((B, V), 0.0, g)
        return s
    T, C = case["frames"], _classes(case)
    s["start"] = torch.full((B,), m.start, dtype=torch.int32, device=DEV)
    s["blank"] = torch.full((B,), V, dtype=torch.int32, device=DEV)
    if case["kind"] == "step":
        s["asr"] = _asr((T, B, C), case["blank"], g)
        s["rows"] = list(s["asr"].unbind(0))
        s["labels"] = torch.empty((T, B), dtype=torch.int32, device=DEV)
        s["label_rows"] = list(s["labels"].unbind(0))
    else:
        s["asr"] = _asr((B, T, C), case["blank"], g)
        s["lengths"] = None
        if case["ragged"]:
            s["lengths"] = torch.randint(T // 4, T + 1, (B,), generator=g, device=DEV).int()
        s["label_states"] = torch.empty((B, T), dtype=torch.int32, device=DEV)
    return s


def run(s):
    lm, kind = s["lm"], s["case"]["kind"]
    if kind == "query":
        return lm.advance(s["states"], s["scores"], s["next"])
    if kind == "topk":
        return lm.fused_topk(s["asr"], LAM, s["case"]["k"], s["states"])
    states, mode = s["start"].clone(), s["mode"]
    prev = s["blank"].clone() if mode == ng.NGPU_FUSION_CTC else None
    if kind == "step":
        for row, labels in zip(s["rows"], s["label_rows"]):
            lm.fused_greedy_step(row, LAM, states, prev, mode=mode, tokens=labels)
        return s["labels"], states
    labels = lm.fused_greedy_decode(s["asr"], LAM, states, prev, lengths=s["lengths"], mode=mode,
                                    label_states=s["label_states"])
    return labels, s["label_states"], states


def _lm_share(case):
    """Share of frames that consult the model: those whose best class is not
    blank, for a boosted blank among N(0, 3) logits."""
    if case["mode"] in ("plain", "aed"):
        return 1.0
    z = np.linspace(-6.0, 6.0, 4001)
    logit = case["blank"] + 3.0 * z
    below = np.array([0.5 * (1.0 + math.erf(x / 3.0 / math.sqrt(2.0))) for x in logit])
    return float(1.0 - np.sum(np.exp(-z * z / 2) * below ** case["vocab"]) / np.sum(np.exp(-z * z / 2)))


def work(case):
    m, B, V = model_of(case), case["batch"], case["vocab"]
    levels, arcs = m.mean_chain()
    arc_total = 8.0 * sum(lv.tok.numel() for lv in m.levels[3:])

    def model_bytes(queries):   # chain records, arcs and dense rows, each read at most once
        chain = min(queries * 16.0 * (1 + levels), 16.0 * m.S * m.N)
        return chain + min(8.0 * arcs * queries, arc_total) + 8.0 * V * min(queries, V + 1)

    if case["kind"] == "query":
        return {"bytes": B * (4.0 + 8.0 * V) + model_bytes(B), "flops": float(B) * V}
    if case["kind"] == "topk":
        return {"bytes": B * (4.0 + 4.0 * V + 12.0 * case["k"]) + model_bytes(B), "flops": 3.0 * B * V}
    frames = B * case["frames"] * (0.625 if case.get("ragged") else 1.0)
    queries = frames * _lm_share(case)
    return {"bytes": frames * (4.0 * _classes(case) + (4.0 if case["kind"] == "step" else 8.0)) + 8.0 * B
            + model_bytes(queries), "flops": 3.0 * queries * V}


def tolerance(case):
    # Measured against 64-bit results of the same inputs: scores, sums of at
    # most ``order`` 32-bit weights, are off by up to 3.5e-8 (2-norm) and by up
    # to 1.5e-7 of their root mean square; labels and states differ at 2.4e-6
    # of the places of the largest decode (two fused scores alike to the last
    # bits), next states nowhere.  Allowed is four times that.
    if case["kind"] == "query":
        return {"rel": 1.4e-7, "max": 6e-7}
    return {"rel": 1.4e-7, "max": 6e-7, "differ": 1e-5}


def exact(case, seed):
    m, s, V = model_of(case), prepare(case, seed), case["vocab"]
    if case["kind"] == "query":
        score, to, _ = m.query64(s["states"])
        return score, to.int()
    if case["kind"] == "topk":
        score, to, _ = m.query64(s["states"])
        value, tok = torch.sort(s["asr"].double() + LAM * score, dim=1, descending=True, stable=True)
        tok = tok[:, :case["k"]]
        return tok.int(), value[:, :case["k"]].contiguous(), torch.gather(to, 1, tok).int()
    mode, B, T = case["mode"], case["batch"], case["frames"]
    states, prev = s["start"].long(), s["blank"].long()
    labels = torch.full((T, B), -1, dtype=torch.int64, device=DEV)
    after = torch.zeros((T, B), dtype=torch.int64, device=DEV)
    lengths = s.get("lengths")
    every = torch.arange(B, device=DEV)
    for t in range(T):
        row = (s["asr"][t] if case["kind"] == "step" else s["asr"][:, t]).double()
        live = lengths > t if lengths is not None else torch.ones(B, dtype=torch.bool, device=DEV)
        score, to, final = m.query64(states)
        fused = row[:, :V] + LAM * score
        raw = row.argmax(1)
        if mode == "ctc":
            known = prev < V
            fused[every[known], prev[known]] = -math.inf
        best = fused.argmax(1)
        stay = torch.zeros_like(live)
        if mode == "aed":
            stay = row[:, V] + LAM * final > fused[every, best]
            raw = torch.full_like(raw, V)
        elif mode != "plain":
            stay = (raw == V) | ((raw == prev) if mode == "ctc" else torch.zeros_like(live))
        label = torch.where(stay, raw, best)
        states = torch.where(live & ~stay, to[every, best], states)
        prev = torch.where(live, label, prev)
        labels[t] = torch.where(live, label, labels[t])
        after[t] = states
    if case["kind"] == "step":
        return labels.int(), states.int()
    return labels.T.contiguous().int(), after.T.contiguous().int(), states.int()
