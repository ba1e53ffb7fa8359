"""NaN among the ASR scores: a NaN loses as -inf does, whatever its sign and
payload, so labels stay classes of the vocabulary and states stay valid.

Each vocabulary and batch reaches another kernel: one, several and sixteen
wavefronts per hypothesis, vocabularies that leave lanes or wavefronts without a
token, and the whole decode of large batches with 4-byte and with 8-byte dense
rows.  The oracle is given -inf in place of every NaN.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_2505_22857_amd as ng  # noqa: E402
from oracle import MODE_AED, MODE_CTC, MODE_PLAIN, MODE_TRANSDUCER, Oracle  # noqa: E402
from synth import asr_logprobs, generate_model, uniform_states  # noqa: E402

# quiet NaNs: the usual one, the sign bit set (what x86 makes), all bits set, another payload
NANS = np.array([0x7fc00000, 0xffc00000, 0xffffffff, 0x7fffffff], np.uint32).view(np.float32)


def spoil(asr, V, seed):
    """Rows [B, T, C] with NaN: whole rows, all but a few classes, the first
    classes, class V, every token beside a finite class V, and -inf among them."""
    rng = np.random.default_rng(seed)
    B, T, C = asr.shape
    for b in range(B):
        for t in range(0, T, 2):
            row, nan = asr[b, t], NANS[(b + t // 2) % len(NANS)]
            kind = (b // len(NANS) + t // 2) % 8
            keep = rng.permutation(V)[:3]
            kept = row[keep].copy()
            if kind == 0:
                row[:] = nan
            elif kind == 1:
                row[:V] = nan
            elif kind == 2:
                row[:] = nan
                row[keep] = kept
            elif kind == 3:
                row[:V // 2 + 1] = nan
            elif kind == 4:
                row[C - 1] = nan
            elif kind == 5:
                row[:] = nan
                row[keep] = -np.inf
            elif kind == 6:
                row[:V] = -np.inf
                row[keep] = nan
                row[0] = nan
            else:
                row[rng.permutation(C)[:C // 3]] = nan
    return asr


def without_nan(asr):
    return np.where(np.isnan(asr), np.float32(-np.inf), asr)


@pytest.mark.parametrize("V,B,mode,dense4", [
    (1, 64, MODE_CTC, True), (63, 64, MODE_CTC, True), (300, 64, MODE_PLAIN, True), (300, 64, MODE_AED, True),
    (700, 64, MODE_CTC, True), (700, 1100, MODE_PLAIN, True), (700, 1100, MODE_CTC, True), (700, 1100, MODE_AED, True),
    (700, 1100, MODE_PLAIN, False), (700, 1100, MODE_TRANSDUCER, False), (1024, 1100, MODE_CTC, True),
    (1024, 1100, MODE_PLAIN, True), (1024, 64, MODE_TRANSDUCER, True), (1500, 64, MODE_CTC, True),
    (1500, 800, MODE_PLAIN, True), (1100, 2049, MODE_PLAIN, True), (1100, 2049, MODE_CTC, True),
    (1900, 1281, MODE_AED, True), (4096, 33, MODE_AED, True), (4097, 33, MODE_PLAIN, True),
    (4097, 33, MODE_CTC, True)])
def test_greedy(V, B, mode, dense4):
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    m = generate_model(V, [V, 3 * V, 2 * V], 1.0, seed=V, bos_eos=mode == MODE_AED)
    order, tokens, W, Bo = m.to_list()
    if not dense4:   # a bigram weight whose sign bit is clear: no 4-byte dense rows
        W = W.copy()
        W[np.nonzero(order == 2)[0][5]] = 0.0
    args = (V, m.max_order, order, tokens, W, Bo, m.unk_logprob)
    lm, o = ng.NgpuLM(*args, bos_eos=mode == MODE_AED).upload("cuda:0"), Oracle(*args, bos_eos=mode == MODE_AED)
    T = 16
    asr = spoil(asr_logprobs((B, T, V + (mode != MODE_PLAIN)), seed=B, blank_boost=2.0 if mode != MODE_PLAIN else 0.0),
                V, V)
    starts = uniform_states(m, B, seed=V)
    prev0 = np.random.default_rng(B).choice([0, 1, V - 1, V], B).astype(np.int32)
    want, after = o.decode(without_nan(asr), mode, 0.5, starts, prev=prev0, nthreads=8)
    rows = torch.from_numpy(asr).cuda()
    st, pv = torch.from_numpy(starts.copy()).cuda(), torch.from_numpy(prev0.copy()).cuda()
    out = torch.empty((B, T), dtype=torch.int32, device="cuda")
    print(f"[case] decode V={V} B={B} mode={mode} dense4={dense4}", flush=True)
    labels = lm.fused_greedy_decode(rows, 0.5, st, pv, mode=mode, label_states=out)
    assert np.array_equal(labels.cpu().numpy(), want)
    assert np.array_equal(out.cpu().numpy(), after)
    st, pv = torch.from_numpy(starts.copy()).cuda(), torch.from_numpy(prev0.copy()).cuda()
    print(f"[case] step V={V} B={B} mode={mode}", flush=True)
    for t in range(T):
        got = lm.fused_greedy_step(rows[:, t], 0.5, st, pv, mode=mode)
        assert np.array_equal(got.cpu().numpy(), want[:, t]), t
        assert np.array_equal(st.cpu().numpy(), after[:, t]), t
    assert lm.check_states() == 0


@pytest.mark.parametrize("V,B,k", [(63, 64, 63), (200, 64, 100), (400, 64, 200), (700, 64, 16), (1024, 64, 256),
                                   (1500, 64, 1), (2048, 64, 40), (3000, 64, 256), (4096, 200, 16), (5000, 64, 32),
                                   (8192, 64, 256)])
def test_topk(V, B, k):
    """Also more NaNs of one bit pattern than the selection's list holds, and none
    of the k places left unwritten."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    m = generate_model(V, [V, 3 * V, 2 * V], 1.0, seed=V)
    lm, o = ng.NgpuLM.from_model(m).upload("cuda:0"), Oracle.from_model(m)
    asr = spoil(asr_logprobs((B, 1, V), seed=V, blank_boost=0.0), V, V + 1)[:, 0].copy()
    states = uniform_states(m, B, seed=B)
    for lam in (0.0, 0.5):
        tok = torch.full((B, k), -7, dtype=torch.int32, device="cuda")
        print(f"[case] top-k V={V} B={B} k={k} lambda={lam}", flush=True)
        _, sc, nx = lm.fused_topk(torch.from_numpy(asr).cuda(), lam, k, torch.from_numpy(states).cuda(), tok)
        assert lm.check_states() == 0
        wt, ws, wn = o.fused_topk(without_nan(asr), lam, k, states)
        assert np.array_equal(tok.cpu().numpy(), wt)
        assert np.array_equal(nx.cpu().numpy(), wn)
        nan = np.isnan(np.take_along_axis(asr, wt, 1))   # their scores come out as they are
        assert np.array_equal(sc.cpu().numpy(), np.where(nan, np.float32(np.nan), ws), equal_nan=True)
