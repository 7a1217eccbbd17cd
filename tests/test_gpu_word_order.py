"""The order between the one-call step's scores and the selection on another stream, where it cannot go by a stored word:
a captured step (a replay would store an old value) and a profiler that collects counters (kernels run one at a time)."""
import pytest

from paper_2503_16163_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (8, 2)])
def test_replayed_step_leaves_later_selections_alone(Hq, Hkv):
    """score_attend captured into a graph, replayed between eager steps: every replay gives the eager output, and the
    selection of an eager step enqueued after a replay still starts and picks what it picked before."""
    import torch
    S, k = 1500, 32
    sc = binding.SpeCache(1, 1, Hq, Hkv, 2, 32, 2048, k, synth.FP16, async_select=2)
    try:
        kp, vp = synth.make_kv_device(7, 1, Hkv, S, 128, synth.FP16)
        q = synth.make_queries_device(7, 1, 1, Hq, 128, synth.FP16).view(1, Hq, 2, 128).contiguous()
        out = torch.empty((1, Hq, 2, 128), dtype=torch.float32, device="cuda")
        idx = torch.empty((1, Hkv, k), dtype=torch.int32, device="cuda")
        side = torch.cuda.Stream()
        sc.quantize_append(0, kp, vp, S)
        torch.cuda.synchronize()

        def eager():
            out.zero_()
            idx.fill_(-7)
            torch.cuda.synchronize()
            sc.score_attend(0, q, 2, None, None, -1, out)
            sc.select_gather(0, idx, -1, side)
            torch.cuda.synchronize()
            return out.clone(), idx.clone()

        want = eager()
        sc.score_attend(0, q, 2, None, None, -1, out)     # the selection's reader is behind: nothing to wait for in the capture
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            sc.score_attend(0, q, 2, None, None, -1, out, torch.cuda.current_stream())
        for _ in range(3):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want[0])
            got = eager()
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    finally:
        sc.close()


def test_steps_while_counters_are_collected(monkeypatch):
    from tests.harness import Case
    monkeypatch.setenv("ROCPROF_COUNTERS", "pmc: SQ_WAVES")
    c = Case(1, 8, 2, 900, synth.BF16, 2, 32, 40, seed=5500, async_select=2, one_pass=True)
    try:
        c.load()
        for t in range(4):
            c.append_token(t)
            c.decode_step(check_logits=False)
    finally:
        c.close()
