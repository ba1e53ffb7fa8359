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
    (1100, 9), (2048, 5), (2049, 5), (2500, 5), (4096, 3), (4097, 3), (8192, 3), (513, 769), (640, 8193), (700, 4096),
    (700, 4097), (700, 8193),
    (641, 4097), (736, 8193), (768, 768), (768, 8192), (1025, 512), (1025, 513), (1056, 2049),
    (1100, 2049), (1280, 512), (1281, 128), (1281, 129), (1408, 2049), (1536, 128), (1536, 2048), (2049, 1024),
    (2304, 4096), (2304, 4097), (2305, 1024), (2500, 1025), (3072, 1024)])
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


@pytest.mark.parametrize("V", [1024, 1312, 1400, 1501, 1536, 1664, 1800, 2048, 2304, 2500, 4096, 4100])
def test_advance_grouped_remainder(V):
    """The grouped batch size and just past a chunk of it, for each width of the
    grouped mapping, and for odd and other vocabularies that do without it."""
    m, lm, o = model(V)
    for B in (20480, 20483):
        states = uniform_states(m, B, seed=B)
        asked = states.copy()
        asked[::97] = -1
        print(f"[case] advance V={V} B={B}", flush=True)
        sc, nx = lm.advance(torch.from_numpy(asked).cuda())
        assert lm.check_states() == len(asked[::97])
        rows = np.r_[0:40, B - 40:B]
        want_s, want_n, _ = o.advance(states[rows], nthreads=8)
        good = asked[rows] >= 0
        assert np.array_equal(nx[torch.from_numpy(rows).cuda()].cpu().numpy()[good], want_n[good])
        assert np.array_equal(sc[torch.from_numpy(rows).cuda()].cpu().numpy()[good], want_s[good])
        assert torch.isnan(sc[::97]).all() and (nx[::97] == -1).all()
        # every other row was written: scores of one state are the same wherever it stands
        first = {int(s): i for i, s in reversed(list(enumerate(asked)))}
        twin = torch.tensor([first[int(s)] for s in asked], device="cuda")
        assert torch.equal(nx, nx[twin]) and torch.equal(torch.nan_to_num(sc, 7.0), torch.nan_to_num(sc[twin], 7.0))
        del sc, nx
