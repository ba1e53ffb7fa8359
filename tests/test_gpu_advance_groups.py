"""The query at the edges of its dispatch against the CPU oracle.

The vocabularies and batches sit at changes of the wavefronts per hypothesis,
of the tokens per lane and of the store width; the outputs are also given at
addresses that are not 16-byte aligned, and some states are out of range.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_2505_22857_amd as ng  # noqa: E402
from oracle import Oracle  # noqa: E402
from synth import generate_model, uniform_states  # noqa: E402

_MODELS = {}


def model(V):
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    if V not in _MODELS:
        m = generate_model(V, [V, 4 * V, 3 * V, V], 1.0, seed=V)
        _MODELS[V] = (m, ng.NgpuLM.from_model(m).upload("cuda:0"), Oracle.from_model(m))
    return _MODELS[V]


@pytest.mark.parametrize("V,B", [
    (1, 3), (3, 70), (63, 5), (64, 5), (255, 3), (256, 70), (257, 1024), (400, 1025), (512, 3), (513, 3), (640, 769),
    (700, 9), (768, 800), (999, 769), (1000, 6144), (1000, 6145), (1020, 769), (1024, 768), (1024, 769), (1025, 9),
    (1100, 9), (2048, 5), (2049, 5), (2500, 5), (4096, 3), (4097, 3), (8192, 3)])
def test_advance_dispatch_edges(V, B):
    m, lm, o = model(V)
    states = uniform_states(m, B, seed=B)
    bad = np.arange(B) % 11 == 5
    asked = np.where(bad, m.num_states + 3, states).astype(np.int32)
    want_s, want_n, _ = o.advance(states, nthreads=8)
    st = torch.from_numpy(asked).cuda()
    for shift in (0, 1):   # words past a 16-byte boundary
        sc = torch.full((B * V + 8,), 7.0, device="cuda")
        nx = torch.full((B * V + 8,), 7, dtype=torch.int32, device="cuda")
        print(f"[case] advance V={V} B={B} shift={shift}", flush=True)
        lm.advance(st, sc[shift:shift + B * V], nx[shift:shift + B * V])
        assert lm.check_states() == int(bad.sum())
        s, n = sc.cpu().numpy(), nx.cpu().numpy()
        assert (s[:shift] == 7).all() and (s[shift + B * V:] == 7).all()   # nothing written outside
        assert (n[:shift] == 7).all() and (n[shift + B * V:] == 7).all()
        s, n = s[shift:shift + B * V].reshape(B, V), n[shift:shift + B * V].reshape(B, V)
        assert np.isnan(s[bad]).all() and (n[bad] == -1).all()
        assert np.array_equal(n[~bad], want_n[~bad])
        assert np.array_equal(s[~bad], want_s[~bad])   # the same fp32 fold


def test_advance_grouped_remainder():
    """V = 1024 at the grouped batch size and just past a chunk of it."""
    m, lm, o = model(1024)
    for B in (20480, 20483):
        states = uniform_states(m, B, seed=B)
        asked = states.copy()
        asked[::97] = -1
        sc, nx = lm.advance(torch.from_numpy(asked).cuda())
        assert lm.check_states() == len(asked[::97])
        rows = np.r_[0:40, B - 40:B]
        want_s, want_n, _ = o.advance(states[rows], nthreads=8)
        good = asked[rows] >= 0
        assert np.array_equal(nx.cpu().numpy()[rows][good], want_n[good])
        assert np.array_equal(sc.cpu().numpy()[rows][good], want_s[good])
        assert torch.isnan(sc[::97]).all() and (nx[::97] == -1).all()
