"""Waits of the caller's stream for the fetches of its side streams: a wait may cover several layers' fetches, and every step still reads
the pairs that its own layer fetched, whichever streams the layers use and however they change."""
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
