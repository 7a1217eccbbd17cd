"""Waits of the caller's stream for the fetches of its side streams: every step reads the pairs that its own layer fetched, whichever streams
the layers use and however they change, and waits for no other layer's fetch."""
import ctypes
import random

import pytest

from paper_2503_16163_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,sides,change", [(1, 1, False), (2, 2, False), (5, 1, False), (8, 2, False), (12, 3, False), (9, 3, True), (16, 2, True)])
def test_steps_read_what_their_layer_fetched(layers, sides, change):
    import torch
    from paper_2503_16163_amd import binding
    B, H, S, k, steps = 1, 4, 3000, 40, 8
    rng = random.Random(layers * 10 + sides)
    q = synth.make_queries_device(11, steps * layers, B, H, 128, synth.FP16).view(steps, layers, B, H, 2, 128)
    kd, vd = synth.make_kv_device(11, B, H, S, 128, synth.FP16)
    nk, nv = synth.make_kv_device(12, steps * B, H, 1, 128, synth.FP16)
    nk, nv = nk.view(steps, B, H, 1, 128), nv.view(steps, B, H, 1, 128)
    ks, vs = synth.make_kv_device(13, B, H, 1, 128, synth.FP16, n_outlier=0)
    streams = [torch.cuda.Stream() for _ in range(sides)]
    plan = [[rng.randrange(sides) if change else L % sides for L in range(layers)] for _ in range(steps + 1)]
    main = torch.cuda.current_stream()

    def run(free_running):
        sc = binding.SpeCache(layers, B, H, H, 2, 32, (S + 127) // 64 * 64, k, synth.FP16, async_select=2)
        idx = torch.full((2, layers, B, H, k), -1, dtype=torch.int32, device="cuda")
        out = torch.zeros((steps, layers, B, H, 2, 128), dtype=torch.float32, device="cuda")
        try:
            for L in range(layers):
                sc.quantize_append(L, kd, vd, S, main)
                sc.score(L, q[0, L], 2, main)
                sc.select_gather(L, idx[0, L], 0, streams[plan[steps][L]])
            torch.cuda.synchronize()
            for t in range(steps):
                for L in range(layers):
                    side = streams[plan[t][L]]
                    sc.debug_poison_slot(L, (t + 1) % 2, main)      # behind the step that read the slot, ahead of the fetch into it
                    if not free_running:
                        torch.cuda.synchronize()
                    sc.decode_step(L, nk[t], nv[t], q[t, L], ks, vs, t % 2, out[t, L], main, idx[(t + 1) % 2, L], (t + 1) % 2, side)
                    if not free_running:
                        torch.cuda.synchronize()
            torch.cuda.synchronize()
            return out
        finally:
            torch.cuda.synchronize()
            sc.close()

    want = run(False)
    assert torch.isfinite(want).all()
    for _ in range(2):
        got = run(True)
        assert torch.equal(got, want), (got - want).abs().nan_to_num(nan=1e9).amax(dim=(1, 2, 3, 4, 5))


class ThreeLayers:
    """Three layers with a prompt and a list each; a side stream whose kernels run beside those of the caller's stream; sleeps of about 100 ms."""

    def __init__(self):
        import torch
        from paper_2503_16163_amd import binding
        self.torch = torch
        B, H, S, k = 1, 4, 700, 16
        self.sc = binding.SpeCache(3, B, H, H, 2, 32, 768, k, synth.FP16, async_select=2)
        kd, vd = synth.make_kv_device(21, B, H, S, 128, synth.FP16)
        self.q = synth.make_queries_device(21, 1, B, H, 128, synth.FP16).view(B, H, 2, 128).contiguous()
        self.idx = torch.arange(k, dtype=torch.int32, device="cuda").mul(7).expand(B, H, k).contiguous()
        self.out = torch.zeros((B, H, 2, 128), dtype=torch.float32, device="cuda")
        for L in range(3):
            self.sc.quantize_append(L, kd, vd, S)
        self.main = torch.cuda.current_stream()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        torch.cuda._sleep(1000000)
        b.record()
        torch.cuda.synchronize()
        self.cycles = int(1000000 * 100.0 / a.elapsed_time(b))
        self.side = next((s for s in (torch.cuda.Stream() for _ in range(8)) if self.beside(s)), None)
        if self.side is None:
            pytest.skip("every stream shares the caller's hardware queue")

    def sleep(self, stream):
        with self.torch.cuda.stream(stream):
            self.torch.cuda._sleep(self.cycles)
        end = self.torch.cuda.Event(enable_timing=True)
        end.record(stream)
        return end

    def beside(self, stream):
        end = self.sleep(stream)
        self.out.zero_()
        done = self.torch.cuda.Event(enable_timing=True)
        done.record(self.main)
        self.torch.cuda.synchronize()
        return done.elapsed_time(end) > 10.0

    def attend(self):
        self.sc.score_attend(0, self.q, 2, None, None, 0, self.out)

    def want(self):
        """The output with layer 0's pairs staged, everything in turn; then its slot is spoilt."""
        self.sc.gather(0, self.idx, 0, self.side)
        self.torch.cuda.synchronize()
        self.attend()
        self.torch.cuda.synchronize()
        want = self.out.clone()
        self.sc.debug_poison_slot(0, 0, None)
        self.out.zero_()
        self.torch.cuda.synchronize()
        return want


@pytest.fixture
def three_layers():
    t = ThreeLayers()
    yield t
    t.torch.cuda.synchronize()
    t.sc.close()


def test_a_step_does_not_wait_for_later_fetches_of_other_layers(three_layers):
    """A caller may hold its side stream back between two layers' fetches until the first layer's step is through."""
    t = three_layers
    want = t.want()
    t.sc.gather(0, t.idx, 0, t.side)
    held = t.sleep(t.side)
    t.sc.gather(1, t.idx, 0, t.side)
    t.sc.gather(2, t.idx, 0, t.side)
    t.attend()
    done = t.torch.cuda.Event(enable_timing=True)
    done.record(t.main)
    t.torch.cuda.synchronize()
    assert t.torch.equal(t.out, want)
    assert done.elapsed_time(held) > 10.0                  # through long before the side stream goes on


def test_a_step_waits_for_its_fetch_although_others_are_captured_behind_it(three_layers):
    """Fetches of two other layers recorded into a graph on the same side stream, while the layer's own is still to run: no event of the graph
    stands for it."""
    t = three_layers
    want = t.want()
    hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
    side, graph = ctypes.c_void_p(t.side.cuda_stream), ctypes.c_void_p()
    t.sleep(t.side)
    t.sc.gather(0, t.idx, 0, t.side)
    assert hip.hipStreamBeginCapture(side, 2) == 0         # relaxed
    try:
        t.sc.gather(1, t.idx, 0, t.side)
        t.sc.gather(2, t.idx, 0, t.side)
    finally:
        assert hip.hipStreamEndCapture(side, ctypes.byref(graph)) == 0
    try:
        t.attend()
        t.torch.cuda.synchronize()
        assert t.torch.equal(t.out, want)
    finally:
        t.torch.cuda.synchronize()
        hip.hipGraphDestroy(graph)


@pytest.mark.parametrize("calls,k", [("score_topk, gather", 40), ("score, select_gather", 40), ("score, select_gather", 600)])
def test_a_captured_step_with_its_fetch_on_a_side_stream(calls, k):
    """Selection, fetch on a side stream and attention recorded into one graph: the launches' order is the graph's, so that it is whole without
    waits of the caller's, every replay reads the pairs that it fetched, and eager steps between them are as ever."""
    import torch
    from paper_2503_16163_amd import binding
    H, S = 4, 3000                                          # 40 pairs: selected and fetched in one launch; 600: in two
    q = synth.make_queries_device(9, 2, 1, H, 128, synth.FP16).view(2, 1, H, 2, 128)[:, :, :, :1].contiguous()
    kd, vd = synth.make_kv_device(9, 1, H, S, 128, synth.FP16)
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    aside = calls == "score, select_gather"
    sc, reference = (binding.SpeCache(1, 1, H, H, 2, 32, 3072, k, synth.FP16, async_select=2 if aside else 0) for _ in range(2))
    new = lambda: (torch.full((1, H, k), -2, dtype=torch.int32, device="cuda"), torch.zeros((1, H, 1, 128), dtype=torch.float32, device="cuda"))

    def step(c, query, idx, out, stream):
        if aside:
            c.score(0, query, 1, stream)
            c.select_gather(0, idx, 0, side)
        else:
            c.score_topk(0, query, 1, idx, stream)
            c.gather(0, idx, 0, side)
        c.attend(0, query, 1, None, None, 0, out, stream)

    main = torch.cuda.current_stream()
    try:
        for c in (sc, reference):
            c.quantize_append(0, kd, vd, S, main)
        want = [new() for _ in range(2)]
        for i in range(2):
            step(reference, q[i], *want[i], main)
        torch.cuda.synchronize()
        got, graph = new(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step(sc, q[0], *got, torch.cuda.current_stream())
        for _ in range(3):
            got[0].fill_(-2)
            got[1].zero_()
            sc.debug_poison_slot(0, 0, None)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(got[0], want[0][0]) and torch.equal(got[1], want[0][1])
            out = new()[1]
            sc.attend(0, q[0], 1, None, None, 0, out, other)        # the replay's pairs are still there
            torch.cuda.synchronize()
            assert torch.equal(out, want[0][1])
            eager = new()
            step(sc, q[1], *eager, main)
            torch.cuda.synchronize()
            assert torch.equal(eager[0], want[1][0]) and torch.equal(eager[1], want[1][1])
    finally:
        torch.cuda.synchronize()
        sc.close()
        reference.close()


@pytest.mark.parametrize("B,H,S,k", [(1, 1, 300, 5), (1, 3, 900, 33), (3, 5, 700, 200), (5, 30, 400, 31), (1, 1, 1000, 4000)])
def test_fetches_that_read_the_list_ahead_stage_the_same_pairs(B, H, S, k):
    """A fetch on the stream that scored, or between fetches on two streams where little is scored for a pair, reads its list ahead; one on a side
    stream does not.  Fewer pairs than a launch takes at a time, more, none a multiple of it; empty and impossible places in the list."""
    import torch
    from paper_2503_16163_amd import binding
    gen = torch.Generator(device="cpu").manual_seed(S + k)
    q = synth.make_queries_device(14, 1, B, H, 128, synth.FP16).view(B, H, 2, 128)[:, :, :1].contiguous()
    kd, vd = synth.make_kv_device(14, B, H, S, 128, synth.FP16)
    idx = torch.randint(0, S, (B, H, k), generator=gen, dtype=torch.int32)
    idx[torch.rand((B, H, k), generator=gen) < 0.1] = -1
    idx[0, 0, 0] = 1 << 20                                   # beyond the store: nothing is fetched
    idx = idx.cuda()
    sides = [torch.cuda.Stream() for _ in range(2)]
    sc = binding.SpeCache(1, B, H, H, 2, 32, (S + 63) // 64 * 64, k, synth.FP16)
    try:
        sc.quantize_append(0, kd, vd, S)
        own = torch.zeros((B, H, k), dtype=torch.int32, device="cuda")
        outs = []
        for where in (sides[0], None, sides[0], sides[1], sides[0]):     # None: the stream that scores; the last two alternate
            sc.debug_poison_slot(0, 1, None)
            sc.score_topk(0, q, 1, own)
            torch.cuda.synchronize()
            sc.gather(0, idx, 1, where)
            outs.append(torch.zeros((B, H, 1, 128), dtype=torch.float32, device="cuda"))
            sc.attend(0, q, 1, None, None, 1, outs[-1])
            torch.cuda.synchronize()
        assert torch.isfinite(outs[0]).all()
        for out in outs[1:]:
            assert torch.equal(out, outs[0])
    finally:
        torch.cuda.synchronize()
        sc.close()
