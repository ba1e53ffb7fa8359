"""Top-k and the fused step at the edges of their dispatch against the CPU oracle.

The vocabularies, batches and k sit at changes of the wavefronts per hypothesis
and of the tokens per lane, with wavefronts that hold few tokens or none, with
more ties than the selection's list holds, and with every token taken.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_2505_22857_amd as ng  # noqa: E402
from oracle import MODE_AED, MODE_CTC, MODE_PLAIN, MODE_TRANSDUCER, Oracle  # noqa: E402
from synth import asr_logprobs, generate_model, uniform_states  # noqa: E402

_MODELS = {}


def model(V, bos_eos=False):
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    if (V, bos_eos) not in _MODELS:
        m = generate_model(V, [V, 3 * V, 2 * V], 1.0, seed=V, bos_eos=bos_eos)
        _MODELS[V, bos_eos] = (m, ng.NgpuLM.from_model(m).upload("cuda:0"), Oracle.from_model(m))
    return _MODELS[V, bos_eos]


def check_topk(V, B, k, asr, lam=0.5):
    m, lm, o = model(V)
    states = uniform_states(m, B, seed=B)
    print(f"[case] top-k V={V} B={B} k={k}", flush=True)
    tok, sc, nx = lm.fused_topk(torch.from_numpy(asr).cuda(), lam, k, torch.from_numpy(states).cuda())
    assert lm.check_states() == 0
    wt, ws, wn = o.fused_topk(asr, lam, k, states)
    assert np.array_equal(tok.cpu().numpy(), wt)
    assert np.array_equal(sc.cpu().numpy(), ws)   # the same fma of the same fp32 fold
    assert np.array_equal(nx.cpu().numpy(), wn)


@pytest.mark.parametrize("V,B,k", [
    (1, 3, 1), (5, 3, 5), (63, 3, 17), (64, 2, 64), (65, 2, 65), (200, 5, 200), (256, 1030, 256), (257, 4, 33),
    (400, 3, 97), (512, 3, 256), (513, 4, 5), (1024, 7, 64), (1025, 4, 16), (1100, 4, 65), (2048, 3, 256),
    (2049, 3, 9), (2500, 130, 130), (4097, 3, 32), (6145, 2, 256), (8192, 3, 40), (500, 1280, 97), (500, 1281, 97),
    (500, 1025, 33), (300, 8193, 97), (513, 1537, 200), (768, 1025, 96), (769, 1025, 96), (769, 1025, 97),
    (1025, 769, 96), (1280, 769, 1), (1281, 769, 40), (1536, 800, 96), (1536, 800, 97)])
def test_topk_dispatch_edges(V, B, k):
    check_topk(V, B, k, asr_logprobs((B, V + 2), seed=V + k)[:, :V].copy())


@pytest.mark.parametrize("V,k,B", [(100, 70, 6), (300, 40, 6), (512, 200, 6), (1000, 1, 6), (1000, 256, 6),
                                   (1500, 100, 6), (5000, 64, 6), (700, 256, 1538), (1000, 90, 1026), (1200, 90, 770),
                                   (1500, 90, 770)])
def test_topk_ties_beyond_the_list(V, k, B):
    """lam = 0 and few distinct scores: hundreds of tokens share the k-th value, within
    and across wavefronts; rows with fewer than k scores above -inf; a row all at -inf."""
    rng = np.random.default_rng(V + k)
    asr = rng.integers(-2, 1, (B, V)).astype(np.float32)
    asr[1] = 0.0
    asr[2] = -np.inf
    asr[3, rng.permutation(V)[:max(1, V - k // 2)]] = -np.inf
    asr[4] = np.where(np.arange(V) == V - 1, 1.0, -0.0)
    for lam in (0.0, 0.5):
        check_topk(V, B, k, asr, lam)


@pytest.mark.parametrize("V,B,mode", [
    (1, 3, MODE_CTC), (63, 3, MODE_TRANSDUCER), (256, 5, MODE_AED), (257, 5, MODE_CTC), (512, 5, MODE_PLAIN),
    (513, 768, MODE_CTC), (700, 769, MODE_AED), (1024, 900, MODE_TRANSDUCER), (1025, 512, MODE_CTC),
    (1100, 9, MODE_AED), (2048, 513, MODE_PLAIN), (2049, 9, MODE_CTC), (4096, 5, MODE_AED), (4500, 9, MODE_CTC),
    (8192, 3, MODE_TRANSDUCER), (513, 769, MODE_CTC), (768, 769, MODE_AED), (769, 769, MODE_CTC),
    (1025, 257, MODE_TRANSDUCER), (1280, 257, MODE_CTC), (1281, 513, MODE_AED), (1536, 513, MODE_CTC),
    (2049, 513, MODE_CTC), (2560, 513, MODE_AED), (2561, 513, MODE_PLAIN), (3072, 513, MODE_CTC),
    (4097, 129, MODE_CTC), (6144, 129, MODE_AED), (6145, 129, MODE_TRANSDUCER), (8192, 129, MODE_CTC)])
def test_step_dispatch_edges(V, B, mode):
    m, lm, o = model(V, mode == MODE_AED)
    states = uniform_states(m, B, seed=V + 1)
    T = 4
    asr = asr_logprobs((B, T, V + (mode != MODE_PLAIN)), seed=V, blank_boost=4.0 if mode != MODE_PLAIN else 0.0)
    asr[0, 1, :V] = -np.inf
    asr[0, 2, 1:] = -np.inf
    prev = np.random.default_rng(V).choice([0, V - 1, V], B).astype(np.int32)
    want, after = o.decode(asr, mode, 0.5, states, prev=prev, nthreads=8)
    st, pv = torch.from_numpy(states.copy()).cuda(), torch.from_numpy(prev.copy()).cuda()
    rows = torch.from_numpy(asr).cuda()
    print(f"[case] step V={V} B={B} mode={mode}", flush=True)
    for t in range(T):
        got = lm.fused_greedy_step(rows[:, t], 0.5, st, pv if mode == MODE_CTC else None, mode=mode)
        assert np.array_equal(got.cpu().numpy(), want[:, t]), t
        assert np.array_equal(st.cpu().numpy(), after[:, t]), t
    assert lm.check_states() == 0
