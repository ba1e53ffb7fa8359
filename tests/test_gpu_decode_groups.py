"""The whole decode at the edges of its dispatch against the CPU oracle.

Each vocabulary and batch sits at a change of the wavefronts per utterance or
of the tokens per lane (256, 512, 1024, 2048 and 4096 tokens; 1024 and 768
utterances), where a token range can be read past its end, a tie can cross two
wavefronts or a stripe can be left out.  Labels and states must be equal.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_2505_22857_amd as ng  # noqa: E402
from oracle import MODE_AED, MODE_CTC, MODE_PLAIN, MODE_TRANSDUCER, Oracle  # noqa: E402
from synth import asr_logprobs, generate_model, tiny_model, uniform_states  # noqa: E402


def check(m, asr, mode, starts, prev=None, lengths=None, lam=0.5):
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    lm, o = ng.NgpuLM.from_model(m).upload("cuda:0"), Oracle.from_model(m)
    B = len(starts)
    prev = np.full(B, m.vocab_size, np.int32) if prev is None else prev
    st, pv = torch.from_numpy(starts.copy()).cuda(), torch.from_numpy(prev.copy()).cuda()
    out = torch.empty(asr.shape[:2], dtype=torch.int32, device="cuda")
    ln = torch.from_numpy(lengths).cuda() if lengths is not None else None
    print(f"[case] decode V={m.vocab_size} N={m.max_order} B={B} T={asr.shape[1]} mode={mode}", flush=True)
    labels = lm.fused_greedy_decode(torch.from_numpy(asr).cuda(), lam, st, pv, lengths=ln, mode=mode, label_states=out)
    assert lm.check_states() == 0
    want, states = o.decode(asr, mode, lam, starts, prev=prev, nthreads=8, lengths=lengths)
    assert np.array_equal(labels.cpu().numpy(), want)
    assert np.array_equal(out.cpu().numpy(), states)
    return labels


@pytest.mark.parametrize("V,B,mode", [
    (255, 9, MODE_CTC), (256, 3, MODE_AED), (257, 9, MODE_TRANSDUCER), (512, 70, MODE_CTC), (513, 1024, MODE_PLAIN),
    (768, 17, MODE_AED), (900, 1025, MODE_TRANSDUCER), (1024, 1024, MODE_CTC), (1024, 1025, MODE_AED),
    (1025, 768, MODE_CTC), (2047, 769, MODE_TRANSDUCER), (2049, 33, MODE_AED), (4096, 5, MODE_CTC),
    (4097, 6, MODE_PLAIN), (8192, 3, MODE_CTC), (1025, 769, MODE_CTC), (1280, 2048, MODE_AED),
    (1025, 2049, MODE_TRANSDUCER), (1100, 2049, MODE_CTC), (1280, 2049, MODE_PLAIN), (1281, 769, MODE_CTC),
    (1281, 1153, MODE_TRANSDUCER), (1536, 1536, MODE_PLAIN), (1536, 1537, MODE_CTC), (1281, 1537, MODE_AED),
    (1537, 1280, MODE_CTC), (1537, 1281, MODE_CTC), (2047, 1400, MODE_AED), (2048, 1536, MODE_TRANSDUCER),
    (2049, 513, MODE_CTC), (2560, 513, MODE_AED), (2561, 513, MODE_PLAIN)])
def test_decode_dispatch_edges(V, B, mode):
    m = generate_model(V, [V, 4 * V, 3 * V, V], 1.0, seed=V, bos_eos=mode == MODE_AED)
    T = 130 if B < 100 else 9   # past the 64 frames whose labels are stored at once, and not a multiple of it
    asr = asr_logprobs((B, T, V + (mode != MODE_PLAIN)), seed=B, blank_boost=6.0 if mode != MODE_PLAIN else 0.0)
    lengths = np.random.default_rng(V).integers(0, T + 1, B).astype(np.int32)
    lengths[:3] = [T, 0, 1]
    check(m, asr, mode, uniform_states(m, B, seed=V + B), lengths=lengths)


@pytest.mark.parametrize("V,B", [(300, 8), (700, 8), (700, 1100), (1100, 800), (1100, 2050), (1500, 8), (1500, 1200),
                                 (1500, 1540), (1600, 1300), (2100, 520)])
def test_decode_ties_and_empty_candidate_sets(V, B):
    """Rows of few distinct scores (ties within a lane, across lanes and across
    wavefronts go to the lowest token), rows all at -inf, and previous labels at
    both ends of the vocabulary."""
    m = generate_model(V, [V, 3 * V, 2 * V], 1.0, seed=V + 1)
    rng = np.random.default_rng(V)
    asr = rng.integers(-3, 1, (B, 40, V + 1)).astype(np.float32) * 4.0
    asr[:, 3] = -np.inf
    asr[:, 7, :V] = -np.inf
    asr[:, 9, 1:] = -np.inf
    asr[:, 10, 1:] = -np.inf
    prev = rng.choice([0, 1, V - 1, V], B).astype(np.int32)
    for lam in (0.0, 0.5):   # 0: the fused scores tie as the ASR scores do
        check(m, asr, MODE_CTC, uniform_states(m, B, seed=3), prev=prev, lam=lam)


@pytest.mark.parametrize("V,N,n1", [(9, 3, 6), (300, 3, 200), (600, 2, 590), (1100, 1, 1100), (77, 1, 70)])
def test_decode_without_every_unigram(V, N, n1):
    """Models whose tokens have no unigram of their own (the state's dense row
    then follows from the empty context's row), and unigram models."""
    m = tiny_model(V, N, seed=5, fill=0.02 if V > 50 else 0.5, n_unigrams=n1)
    asr = asr_logprobs((12, 70, V + 1), seed=V, blank_boost=2.0)
    check(m, asr, MODE_CTC, uniform_states(m, 12, seed=6))


_NOISE = []


@pytest.mark.parametrize("V,B,mode", [
    (900, 1000, MODE_TRANSDUCER), (1100, 700, MODE_CTC), (2048, 700, MODE_TRANSDUCER), (1100, 1000, MODE_CTC),
    (1280, 1000, MODE_TRANSDUCER), (1400, 1300, MODE_CTC), (1536, 1300, MODE_CTC), (1400, 1000, MODE_TRANSDUCER),
    (1536, 1000, MODE_CTC), (2000, 800, MODE_CTC), (2048, 800, MODE_CTC), (2300, 600, MODE_TRANSDUCER),
    (2560, 600, MODE_CTC), (3000, 500, MODE_CTC), (4096, 500, MODE_TRANSDUCER), (5000, 300, MODE_CTC),
    (8192, 200, MODE_TRANSDUCER)])
def test_decode_streamed_rows(V, B, mode):
    """ASR tensors just above 256 MiB, whose rows are loaded non-temporally by every
    kernel of several wavefronts per utterance: each width the launcher has for
    them, with lanes past V and without (V = 1024 with four wavefronts is decoded
    that way by the 20M 6-gram's test).  About two frames in three are blank."""
    m = generate_model(V, [V, 4 * V, 3 * V], 1.0, seed=V)
    T = (1 << 26) // (B * (V + 1)) + 1
    n = B * T * (V + 1)
    if not _NOISE:
        _NOISE.append(np.random.default_rng(0).standard_normal((1 << 26) + (1 << 22), dtype=np.float32) * 3.0)
    asr = _NOISE[0][:n].reshape(B, T, V + 1).copy()
    asr[:, :, V] += 3.0 * np.sqrt(2.0 * np.log(V))   # near the largest of V such scores
    assert asr.nbytes > 256 << 20
    labels = check(m, asr, mode, uniform_states(m, B, seed=9))
    spoken = (labels.cpu().numpy() != V).mean()
    assert 0.1 < spoken < 0.9
