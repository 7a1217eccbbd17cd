"""The order between the one-call step's scores and the selection on another stream: by a stored word where kernels of different
queues run side by side, by an event where they may not (a tool in the process, a captured step, a caller that asks for it)."""
import pytest

from paper_2503_16163_amd import binding, synth

pytestmark = pytest.mark.gpu


class Steps:
    """One layer with a prompt, stepped eagerly on the current stream and a side stream."""

    def __init__(self, Hq, Hkv, S=1500, k=32):
        import torch
        self.torch = torch
        self.sc = binding.SpeCache(1, 1, Hq, Hkv, 2, 32, 2048, k, synth.FP16, async_select=2)
        kp, vp = synth.make_kv_device(7, 1, Hkv, S, 128, synth.FP16)
        self.q = synth.make_queries_device(7, 1, 1, Hq, 128, synth.FP16).view(1, Hq, 2, 128).contiguous()
        self.out = torch.empty((1, Hq, 2, 128), dtype=torch.float32, device="cuda")
        self.idx = torch.empty((1, Hkv, k), dtype=torch.int32, device="cuda")
        self.side = torch.cuda.Stream()
        self.sc.quantize_append(0, kp, vp, S)
        torch.cuda.synchronize()

    def score(self, stream=None):
        self.sc.score_attend(0, self.q, 2, None, None, -1, self.out, stream)

    def eager(self, between=lambda: None):
        self.out.zero_()
        self.idx.fill_(-7)
        self.torch.cuda.synchronize()
        self.score()
        between()
        self.sc.select_gather(0, self.idx, -1, self.side)
        self.torch.cuda.synchronize()
        return self.out.clone(), self.idx.clone()


@pytest.fixture
def steps():
    opened = []

    def open_steps(Hq=8, Hkv=2):
        opened.append(Steps(Hq, Hkv))
        return opened[-1]
    yield open_steps
    for s in opened:
        s.torch.cuda.synchronize()
        s.sc.close()


@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (8, 2)])
def test_replayed_step_leaves_later_selections_alone(steps, Hq, Hkv):
    """score_attend captured into a graph, replayed between eager steps and between an eager step's scores and its selection: every
    replay gives the eager output, the captured step goes by the event and the eager ones by the word, and every selection picks
    what it picked before."""
    import torch
    s = steps(Hq, Hkv)
    want = s.eager()
    assert s.sc.debug_scored_by_word(0)
    s.score()                         # the selection's reader is behind: nothing to wait for in the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.score(torch.cuda.current_stream())
    assert not s.sc.debug_scored_by_word(0)
    for between in (lambda: None, g.replay, g.replay):
        s.out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(s.out, want[0])
        got = s.eager(between)
        assert s.sc.debug_scored_by_word(0)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_selection_in_a_capture_behind_scores_outside_it_is_refused(steps):
    """As waiting for an event from outside a capture is: a recorded wait would be for a value long passed."""
    import ctypes
    import torch
    s = steps()
    want = s.eager()
    hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
    s.score()
    torch.cuda.synchronize()
    assert s.sc.debug_scored_by_word(0)
    side, graph = ctypes.c_void_p(s.side.cuda_stream), ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(side, 2) == 0         # relaxed
    try:
        with pytest.raises(binding.SpeCacheError) as e:
            s.sc.select_gather(0, s.idx, -1, s.side)
        assert e.value.code == binding.ESTATE
    finally:
        hip.hipStreamEndCapture(side, ctypes.byref(graph))
        if graph.value:
            hip.hipGraphDestroy(graph)
    got = s.eager()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("variable,value", [("ROCPROF_COUNTERS", "pmc: SQ_WAVES"), ("ROCPROF_ADVANCED_THREAD_TRACE", "1"), ("ROCP_TOOL_LIBRARIES", "/x.so"),
                                            ("HSA_TOOLS_LIB", "/x.so"), ("AMD_DIRECT_DISPATCH", "0")])
def test_steps_beside_a_tool_named_in_the_environment(monkeypatch, steps, variable, value):
    import torch
    want = steps().eager()
    monkeypatch.setenv(variable, value)
    s = steps()
    got = s.eager()
    assert not s.sc.debug_scored_by_word(0)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_steps_while_counters_are_collected(monkeypatch):
    from tests.harness import Case
    monkeypatch.setenv("ROCPROF_COUNTERS", "pmc: SQ_WAVES")
    c = Case(1, 8, 2, 900, synth.BF16, 2, 32, 40, seed=5500, async_select=2, one_pass=True)
    try:
        c.load()
        for t in range(4):
            c.append_token(t)
            c.decode_step(check_logits=False)
            assert not c.sc.debug_scored_by_word(0)
    finally:
        c.close()


def test_steps_beside_a_tool_that_is_loaded_later(steps, tmp_path):
    """A profiler that attaches to the running process brings its library: from then on the event orders the selection."""
    import _ctypes
    import ctypes
    import subprocess
    import torch
    s = steps()
    want = s.eager()
    assert s.sc.debug_scored_by_word(0)
    lib = tmp_path / "librocprofiler-stand-in.so"
    subprocess.run(["gcc", "-shared", "-fPIC", "-x", "c", "/dev/null", "-o", str(lib)], check=True)
    handle = ctypes.CDLL(str(lib))
    try:
        got = s.eager()
        assert not s.sc.debug_scored_by_word(0)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    finally:
        _ctypes.dlclose(handle._handle)


def test_caller_that_wants_events(steps):
    import torch
    s = steps()
    want = s.eager()
    for enable in (True, False):
        s.sc.order_by_events(enable)
        got = s.eager()
        assert s.sc.debug_scored_by_word(0) == (not enable)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
