"""The merge of a row's partial results inside the launch that makes them, on both sides of the rule that chooses it (chunks x query
rows up to 64): scoring and attention in one launch, attention alone, one and two query rows, shapes whose slices of the
chunks differ, with steps in a row so that a counter left wrong by one launch shows in the next."""
import pytest

from paper_2503_16163_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,S,bits,g,k,n_rows,one_pass", [
    (2, 2, 200, 2, 32, 16, 2, True), (1, 1, 4096, 2, 32, 64, 2, True), (3, 3, 15872 + 40, 2, 64, 64, 2, True), (3, 3, 15872 + 600, 1, 32, 64, 2, True),
    (2, 2, 3000, 2, 32, 300, 2, False), (2, 2, 3000, 1, 128, 64, 1, False), (4, 2, 1500, 2, 32, 40, 1, False),
    (8, 2, 1700, 2, 32, 48, 2, True), (8, 2, 1990, 2, 64, 48, 2, True), (8, 2, 1700, 1, 32, 48, 2, False), (8, 1, 340, 2, 32, 48, 2, True),
    (8, 1, 600, 2, 32, 48, 2, True), (4, 4, 1500, 4, 32, 32, 2, False), (4, 2, 900, 2, 32, 200, 2, True), (2, 2, 1500, 4, 64, 16, 1, False),
    # as many workgroups as the rule takes, 1024, and one more row of them
    (32, 32, 15700, 2, 32, 64, 1, False), (32, 32, 15700, 2, 64, 64, 2, True), (33, 33, 15700, 2, 64, 64, 2, True), (16, 16, 31600, 1, 64, 64, 1, False),
    # one query row beyond the rule by its workgroups and by its partials, two heads of one row likewise
    (33, 33, 15700, 2, 32, 64, 1, False), (1, 1, 33000, 2, 64, 300, 1, False), (4, 2, 16400, 1, 128, 40, 1, False)])
def test_merge_in_the_launch(Hq, Hkv, S, bits, g, k, n_rows, one_pass):
    from tests.harness import Case
    # the speculative flow with two query rows, the non-speculative one with one
    c = Case(1, Hq, Hkv, S, synth.BF16 if Hq > 4 else synth.FP16, bits, g, k, R=max(64, g), seed=7300 + S + bits, n_rows=n_rows,
             sample=[(0, h) for h in range(min(Hkv, 2))], async_select=2 if n_rows == 2 else 0, one_pass=one_pass, fused_append=one_pass)
    try:
        c.load()
        for t in range(5):
            c.append_token(t)
            if n_rows == 2:
                c.decode_step(check_logits=False)
            else:
                c.nonspec_step()
        assert c.stats["max_out_err"] < 5e-5, c.stats
    finally:
        c.close()


# 20 chunks on 64 rows are the 1280 workgroups of one round; beside them 374 and 405 quantised positions for a pair
@pytest.mark.parametrize("S,k,fetched,bits,g,in_launch", [
    (512 * 19 + 40, 26, True, 2, 32, True), (512 * 20 + 40, 27, True, 2, 32, False), (512 * 20 + 40, 26, True, 1, 64, True),
    (512 * 20 + 40, 27, False, 2, 32, True), (512 * 20 + 40, 27, True, 1, 128, False)])
def test_launches_of_several_rounds_leave_the_merge_where_much_is_fetched(S, k, fetched, bits, g, in_launch):
    """On both sides of the rule: where the merge runs, and the oracle's outputs either way."""
    import torch
    from tests.harness import Case
    c = Case(2, 32, 32, S, synth.FP16, bits, g, k, R=max(64, g), seed=7900 + k, sample=[(0, 0), (1, 31)], async_select=2, one_pass=True, fused_append=True)
    try:
        c.load()
        for t in range(2):
            c.append_token(t)
            c.decode_step(check_logits=False, do_gather=fetched)
        assert c.stats["max_out_err"] < 5e-5, c.stats
        q = synth.make_queries_device(7, 1, 2, 32, 128, synth.FP16).view(2, 32, 2, 128).contiguous()
        out = torch.empty((2, 32, 2, 128), dtype=torch.float32, device="cuda")
        c.sc.timing(True)
        c.sc.score_attend(0, q, 2, None, None, 0 if fetched else -1, out)
        spans = c.sc.timing(False)
        assert spans["score_attend"][1] == 1 and spans["attend_combine"][1] == (0 if in_launch else 1), spans
    finally:
        c.close()


def test_layers_on_streams_of_their_own_keep_their_counters():
    """Every layer counts for itself: layers stepped on different streams, one after the other, and a context opened in between."""
    import torch
    from paper_2503_16163_amd import binding
    H, S, k = 4, 1000, 16
    q = synth.make_queries_device(5, 1, 1, H, 128, synth.FP16).view(1, H, 2, 128).contiguous()
    kd, vd = synth.make_kv_device(5, 1, H, S, 128, synth.FP16)
    want = None
    for rounds in range(2):
        sc = binding.SpeCache(3, 1, H, H, 2, 32, 1024, k, synth.FP16, async_select=2)
        streams = [torch.cuda.Stream() for _ in range(3)]
        try:
            for L in range(3):
                sc.quantize_append(L, kd, vd, S)
            torch.cuda.synchronize()
            for t in range(6):
                for L in range(3):
                    out = torch.zeros((1, H, 2, 128), dtype=torch.float32, device="cuda")
                    torch.cuda.synchronize()
                    sc.score_attend(L, q, 2, None, None, -1, out, streams[(L + t) % 3])
                    torch.cuda.synchronize()
                    want = out if want is None else want
                    assert torch.equal(out, want), (rounds, t, L)
        finally:
            torch.cuda.synchronize()
            sc.close()


def test_attend_from_static_scratch_beside_attend():
    """specache_attend and specache_attend_static of one layer keep their partials apart, so on two streams they may overlap: neither
    counts the other's workgroups."""
    import torch
    from paper_2503_16163_amd import binding
    H, S, k = 4, 6000, 16
    q = synth.make_queries_device(6, 1, 1, H, 128, synth.FP16).view(1, H, 2, 128).contiguous()
    kd, vd = synth.make_kv_device(6, 1, H, S, 128, synth.FP16)
    sc = binding.SpeCache(1, 1, H, H, 2, 32, 6144, k, synth.FP16, async_select=2)
    streams = [torch.cuda.Stream() for _ in range(2)]
    try:
        sc.quantize_append(0, kd, vd, S)
        sc.score(0, q, 2)
        want = [torch.zeros((1, H, 2, 128), dtype=torch.float32, device="cuda") for _ in range(2)]     # each by itself first
        sc.attend(0, q, 2, None, None, -1, want[0])
        sc.attend_static(0, q, 2, None, None, -1, want[1])
        outs = [torch.zeros_like(want[0]) for _ in range(40)]
        torch.cuda.synchronize()
        for i in range(20):
            sc.attend(0, q, 2, None, None, -1, outs[2 * i], streams[0])
            sc.attend_static(0, q, 2, None, None, -1, outs[2 * i + 1], streams[1])
        torch.cuda.synchronize()
        for i, out in enumerate(outs):
            assert torch.equal(out, want[i % 2]), (i, (out - want[i % 2]).abs().max().item())
    finally:
        torch.cuda.synchronize()
        sc.close()


@pytest.mark.parametrize("Hq,Hkv,S,bits,g,k", [
    (1, 1, 600, 2, 32, 16), (3, 3, 5000, 1, 64, 64), (2, 2, 2000, 2, 128, 300),
    # as many rows as leave the merge to the last chunk, and one more
    (4, 4, 600, 2, 32, 16), (5, 5, 600, 2, 32, 16), (6, 6, 3000, 1, 128, 64),
    # as many chunks as the rule takes, 128, and one more; beyond 96 a lane reads its partials in two batches
    (1, 1, 512 * 127 + 40, 2, 32, 64), (1, 1, 512 * 128 + 40, 2, 32, 64), (1, 1, 512 * 96 + 40, 2, 64, 64),
    # 4, 8 and 16 query rows: one share to sixteen, of one query row to eight
    (2, 1, 3000, 2, 32, 48), (4, 1, 900, 2, 64, 48), (8, 1, 300, 2, 32, 16), (8, 1, 20000, 1, 32, 48), (16, 2, 9000, 2, 64, 48), (4, 1, 256 * 127 + 40, 2, 32, 64),
    (4, 1, 256 * 128 + 40, 2, 32, 64), (1, 1, 2000, 4, 32, 32)])
def test_mergers_and_what_they_leave_behind(Hq, Hkv, S, bits, g, k):
    """A share of a row's query rows is merged by a workgroup of its own or, when that stops looking, by the last chunk: the same sums in the
    same order, and counters as the next launch wants them.  attend_static merges in a launch of its own."""
    import torch
    from paper_2503_16163_amd import binding
    q = synth.make_queries_device(7, 1, 1, Hq, 128, synth.FP16).view(1, Hq, 2, 128).contiguous()
    kd, vd = synth.make_kv_device(7, 1, Hkv, S, 128, synth.FP16)
    ks, vs = synth.make_kv_device(8, 1, Hkv, 1, 128, synth.FP16, n_outlier=0)
    idx = torch.full((1, Hkv, k), -1, dtype=torch.int32, device="cuda")
    sc = binding.SpeCache(1, 1, Hq, Hkv, bits, g, (S + 127) // 64 * 64, k, synth.FP16, residual=max(64, g), async_select=2)
    outs = []
    try:
        sc.quantize_append(0, kd, vd, S)
        sc.score(0, q, 2)
        sc.select_gather(0, idx, 0)
        own = torch.zeros((1, Hq, 2, 128), dtype=torch.float32, device="cuda")
        sc.attend_static(0, q, 2, ks, vs, 0, own)
        for polls in (-1, 0, -1, 1, 0, 3, -1):
            binding.debug_merger_polls(polls)
            for fn in (sc.score_attend, sc.attend):
                if fn == sc.attend:
                    sc.score(0, q, 2)
                outs.append((polls, fn.__name__, torch.full((1, Hq, 2, 128), float("nan"), dtype=torch.float32, device="cuda")))
                fn(0, q, 2, ks, vs, 0, outs[-1][2])
        torch.cuda.synchronize()
    finally:
        binding.debug_merger_polls(-1)
        torch.cuda.synchronize()
        sc.close()
    first = {name: out for _, name, out in reversed(outs)}
    for polls, name, out in outs:
        assert torch.equal(out, first[name]), (polls, name, (out - first[name]).abs().max().item())
    # attention alone from other scratch memory: the same kernel, and the merge's own launch adds up in the same order (up to 128 chunks)
    assert torch.equal(first["attend"], own), (first["attend"] - own).abs().max().item()
