"""The binding's native per-call path: it answers ordinary calls with the same
results and objects as the Python path, and leaves every other call to it."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2505_22857_amd as ng  # noqa: E402
from synth import tiny_model  # noqa: E402


def test_declines_what_is_not_a_plain_device_tensor():
    """Calls on the CPU never reach the library: None, for the Python path to refuse."""
    fast = ng._load_fast()
    st = torch.zeros(3, dtype=torch.int32)
    asr = torch.zeros(3, 9)
    assert fast.advance(0, 9, st, None, None) is None
    assert fast.advance(0, 9, "states", None, None) is None
    assert fast.advance(0) is None
    assert fast.step(0, 9, asr, 0.5, st, None, 0, None) is None
    assert fast.step(0, 9, asr, 1, st, None, True, None) is None
    assert fast.topk(0, 9, asr, 0.5, 4, st, None, None, None) is None


@pytest.fixture(params=["missing", "no library", "another torch"])
def unusable(request, monkeypatch, tmp_path):
    """No native module, a file that does not load, one built against another torch."""
    monkeypatch.setattr(ng, "_fast", None)
    if request.param == "another torch":
        monkeypatch.setattr(torch, "__version__", "0.1")
    else:
        monkeypatch.setattr(ng, "FAST_PATH", str(tmp_path / "_fastcall.so"))
        if request.param == "no library":
            (tmp_path / "_fastcall.so").write_bytes(b"not a library")


def test_unusable_module_is_left_out(unusable):
    with pytest.warns(RuntimeWarning, match="ctypes"):
        assert ng._fast_or_none() is None
    assert ng._fast is None


@pytest.fixture(scope="module")
def lm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    return ng.NgpuLM.from_model(tiny_model(9, 3, seed=21)).upload("cuda:0")


def both(lm, call):
    """Results of the native path and of the Python path."""
    fast = lm._fast
    got = call()
    lm._fast = None
    try:
        want = call()
    finally:
        lm._fast = fast
    torch.cuda.synchronize()
    return got, want


@pytest.mark.gpu
@pytest.mark.parametrize("B", [0, 1, 5])
def test_same_results_as_the_python_path(lm, B):
    g = torch.Generator(device="cuda").manual_seed(B)
    states = torch.randint(0, lm.num_states, (B,), generator=g, device="cuda").int()
    wide = torch.randn((B, 30), generator=g, device="cuda")
    for asr in (wide[:, :10], wide[:, 3:13], wide[:, ::1][:, :9]):   # row strides and offsets
        k = min(4, lm.vocab_size)
        for call in (lambda: lm.advance(states), lambda: lm.fused_topk(asr, 0.5, k, states),
                     lambda: [lm.fused_greedy_step(asr, 0.5, states.clone())],
                     lambda: lm.fused_topk(asr, np.float64(0.5), k, states),
                     lambda: [lm.fused_greedy_step(asr, 1, states.clone())]):
            got, want = both(lm, call)
            assert len(got) == len(want)
            for x, y in zip(got, want):
                assert x.dtype == y.dtype and x.shape == y.shape and torch.equal(x, y)
    st, pv = states.clone(), torch.full((B,), 9, dtype=torch.int32, device="cuda")
    tok = torch.empty(B + 2, dtype=torch.int32, device="cuda")
    assert lm.fused_greedy_step(wide[:, :10], 0.5, st, pv, mode=ng.NGPU_FUSION_CTC, tokens=tok) is tok
    sc = torch.empty((B, 9), device="cuda")
    assert lm.advance(states, sc)[0] is sc


@pytest.mark.gpu
def test_upload_without_the_module(lm, unusable):
    with pytest.warns(RuntimeWarning, match="ctypes"):
        plain = ng.NgpuLM.from_model(tiny_model(9, 3, seed=21)).upload("cuda:0")
    states = torch.arange(4, dtype=torch.int32, device="cuda")
    got, want = plain.advance(states), lm.advance(states)
    assert plain._fast is None and torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.gpu
def test_other_streams_and_refusals(lm):
    states = torch.zeros(4, dtype=torch.int32, device="cuda")
    asr = torch.zeros((4, 10), device="cuda")
    want = lm.advance(states)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    got = lm.advance(states, stream=side)
    with torch.cuda.stream(side):
        again = lm.advance(states)
    torch.cuda.synchronize()
    for x in (got, again):
        assert torch.equal(x[0], want[0]) and torch.equal(x[1], want[1])
    with pytest.raises(TypeError):
        lm.advance(states.long())
    with pytest.raises(TypeError):
        lm.advance(torch.zeros(8, dtype=torch.int32, device="cuda")[::2])
    with pytest.raises(ValueError):
        lm.advance(states, torch.empty(3, device="cuda"))
    with pytest.raises(TypeError):
        lm.fused_greedy_step(asr.double(), 0.5, states)
    with pytest.raises(ValueError):
        lm.fused_greedy_step(asr[:, :9], 0.5, states, mode=ng.NGPU_FUSION_TRANSDUCER)
    with pytest.raises(ValueError):
        lm.fused_topk(asr, 0.5, 2, states[:3])
    with pytest.raises(ng.NgpuError):
        lm.fused_topk(asr, 0.5, 10, states)          # k above V
    with pytest.raises(ng.NgpuError):
        lm.fused_greedy_step(asr, float("nan"), states)
    with pytest.raises(ng.NgpuError):
        lm.fused_greedy_step(asr, 0.5, states, mode=ng.NGPU_FUSION_AED)   # no </s> in the model


@pytest.mark.gpu
def test_a_failed_allocation_leaves_the_states_alone(lm):
    """The step's result object is made before the step is enqueued: where that
    fails, the native path declines and nothing has moved; the call is then
    made, once, by the Python path."""
    hooks = pytest.importorskip("_testcapi")
    asr = torch.randn((5, 10), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    start = torch.zeros(5, dtype=torch.int32, device="cuda")
    want_st = start.clone()
    want = lm.fused_greedy_step(asr, 0.5, want_st)
    assert (want_st != start).any()
    st = start.clone()
    torch.cuda.synchronize()
    step, args = lm._fast.step, (lm._h.value, lm.vocab_size, asr, 0.5, st, None, 0, None)
    try:
        hooks.set_nomemory(0, 1)   # the first allocation fails, no other
        r = step(*args)
    finally:
        hooks.remove_mem_hooks()
    torch.cuda.synchronize()
    assert r is None and torch.equal(st, start)
    assert torch.equal(lm.fused_greedy_step(asr, 0.5, st), want) and torch.equal(st, want_st)
