"""ArgTopK and the fetch behind it against the scores they were made from: the selection has to be exactly the k largest
keys of the logits that the scoring kernel left (ties to the lower position), at the sizes where the kernel changes its
shape, and the staged pairs those that a fetch of the same index list brings."""
import numpy as np
import pytest

from paper_2503_16163_amd import binding, synth

pytestmark = pytest.mark.gpu


def keys_of(logits):
    u = (logits + np.float32(0.0)).view(np.uint32)
    return np.where(u & 0x80000000, ~u, u | np.uint32(0x80000000)).astype(np.uint32)


def expected(keys, k):
    """Positions of the k largest keys, ascending, -1 padded; key 0 (one NaN pattern) is below everything and stays out of a real choice."""
    keff = min(k, keys.size)
    order = np.lexsort((np.arange(keys.size), -keys.astype(np.int64)))[:keff]
    if keff < keys.size:
        order = order[keys[order] != 0]
    return np.concatenate([np.sort(order), np.full(k - order.size, -1)]).astype(np.int32)


def prompt(pattern, S, H, q):
    rng = np.random.default_rng(S + H)
    K = rng.standard_normal((1, H, S, 128)).astype(np.float32)
    if pattern == "one value":
        K[:] = K[:, :, :1]
    elif pattern == "few values":
        K = K[:, :, np.arange(S) % 64]
    elif pattern == "binades apart":
        K *= np.exp2(-(np.arange(S) // 32 % 12)).astype(np.float32)[None, None, :, None]
    elif pattern == "one far above":
        K[:, :, 40:44] = 30.0 * np.sign(q)[:, :, None, :]
    elif pattern == "negative":
        K = -np.abs(K) * np.sign(q)[:, :, None, :]
    elif pattern == "not numbers":
        K[:, :, 96 % S, 5] = np.nan
        K[:, :, 300 % S, 6] = np.inf
    return K


# positions at the edges of a workgroup's registers: 8, 16, 32 keys for each of 256 threads (in the launches that do not fetch; with so few rows
# those that do have 1024), 16 to 48 for each of 1024, two launches
SIZES = [(64, 16), (64, 256), (320, 300), (2048, 64), (2080, 200), (4096, 256), (4128, 1), (8192, 128), (8224, 64), (8192, 257), (16384, 1024),
         (16416, 64), (24576, 256), (32768, 64), (32800, 500), (40960, 256), (40992, 256), (49152, 256), (49184, 64), (70016, 64), (49152, 4096), (131072, 1024),
         # room for 2048 candidates and for 8192
         (4096, 900), (4096, 1024), (8192, 1200), (8192, 2048), (16384, 1600), (16384, 4095), (24576, 4096), (32768, 2048), (40960, 3000), (70016, 4096),
         # a large share of a short row: a floor, or all keys at once
         (256, 104), (256, 156), (256, 255), (448, 157), (448, 158), (640, 198), (960, 211), (960, 249), (960, 384), (960, 576), (1440, 584), (2048, 512)]
PATTERNS = ["even", "one value", "few values", "binades apart", "one far above", "negative", "not numbers"]


@pytest.mark.parametrize("Nq,k", SIZES)
def test_selected_positions_are_the_largest_keys(Nq, k):
    import torch
    H = 3 if Nq < 40993 else 1
    S = Nq + 32
    q = np.random.default_rng(3).standard_normal((1, H, 2, 128)).astype(np.float32)
    qd = torch.from_numpy(q).half().cuda()
    side = torch.cuda.Stream()
    for pattern in PATTERNS if Nq <= 49184 else PATTERNS[:5]:
        K = prompt(pattern, S, H, q[:, :, 1])
        kd = torch.from_numpy(K).half().cuda()
        vd = torch.from_numpy(np.random.default_rng(4).standard_normal((1, H, S, 128)).astype(np.float32)).half().cuda()
        sc = binding.SpeCache(1, 1, H, H, 2, 32, (S + 63) // 64 * 64, k, synth.FP16, async_select=2)
        try:
            sc.quantize_append(0, kd, vd, S)
            assert sc.counts(0) == (S, Nq)
            idx = [torch.full((1, H, k), -7, dtype=torch.int32, device="cuda") for _ in range(3)]
            out = [torch.empty((1, H, 2, 128), dtype=torch.float32, device="cuda") for _ in range(2)]
            sc.score(0, qd, 2)
            sc.select_gather(0, idx[0], -1, side)           # the selection alone
            sc.select_gather(0, idx[1], 0, side)            # the selection and its pairs
            sc.gather(0, idx[1], 1, side)                   # the pairs of that list again
            sc.score_topk(0, qd, 2, idx[2])
            for slot in (0, 1):
                sc.attend(0, qd, 2, None, None, slot, out[slot])
            torch.cuda.synchronize()
            keys = keys_of(sc.debug_logits(0, 2)[0, :, 1])
            for h in range(H):
                want = expected(keys[h], k)
                for i in range(3):
                    got = idx[i][0, h].cpu().numpy()
                    assert np.array_equal(got, want), (pattern, h, i, got[:8], want[:8])
            assert torch.equal(out[0].view(torch.int32), out[1].view(torch.int32)), pattern
            if pattern != "not numbers":
                assert torch.isfinite(out[0]).all()
        finally:
            torch.cuda.synchronize()
            sc.close()


# rows x quantised positions x k around the rules of the launch that selects and fetches: 256 threads a row (from about 24 rows on) with 8, 16
# and 32 keys a thread, 1024 threads, up to 128 rows; few rows with as many pairs as one launch takes, and one more; two launches
@pytest.mark.parametrize("B,H,Nq,k", [(1, 24, 2048, 64), (3, 8, 2080, 256), (8, 8, 4096, 33), (3, 8, 4128, 200), (4, 32, 8192, 17), (2, 32, 8192, 128), (2, 32, 8224, 64),
                                      (16, 8, 1024, 100), (43, 3, 1024, 16), (1, 33, 64, 256), (1, 1, 4096, 192), (1, 1, 4096, 193), (1, 3, 4096, 256), (1, 3, 4096, 257),
                                      (1, 5, 4096, 385), (1, 6, 8192, 900), (1, 6, 4096, 1000)])
def test_pairs_behind_the_selection_are_those_of_a_fetch_of_its_list(B, H, Nq, k):
    import torch
    S = Nq + 32
    g = torch.Generator(device="cuda")
    g.manual_seed(Nq + k)
    rand = lambda *shape: torch.randn(shape, device="cuda", generator=g).half()
    sc = binding.SpeCache(2, B, H, H, 2, 32, (S + 63) // 64 * 64, k, synth.FP16, async_select=2)
    side = [torch.cuda.Stream() for _ in range(2)]
    idx = torch.full((2, 2, B, H, k), -7, dtype=torch.int32, device="cuda")
    out = torch.empty((2, 2, B, H, 2, 128), dtype=torch.float32, device="cuda")
    q = rand(2, B, H, 2, 128)
    try:
        for L in range(2):
            sc.quantize_append(L, rand(B, H, S, 128), rand(B, H, S, 128), S)
            assert sc.counts(L) == (S, Nq)
        for rounds in range(2):              # (the second fetch on the other stream finds the link shared)
            for L in range(2):
                sc.score(L, q[L], 2)
                sc.select_gather(L, idx[0, L], 0, side[L])
                sc.select_gather(L, idx[1, L], -1, side[L])
                sc.gather(L, idx[1, L], 1, side[L])
                for slot in range(2):
                    sc.attend(L, q[L], 2, None, None, slot, out[L, slot])
            torch.cuda.synchronize()
            sc.score(1, q[1], 2)
            keys = keys_of(sc.debug_logits(1, 2)[:, :, 1])
            for b in range(B):
                for h in range(H):
                    assert np.array_equal(idx[0, 1, b, h].cpu().numpy(), expected(keys[b, h], k)), (b, h)
            assert torch.equal(idx[0], idx[1])
            assert torch.equal(out[:, 0].view(torch.int32), out[:, 1].view(torch.int32)) and torch.isfinite(out).all()
            idx.fill_(-7)
    finally:
        torch.cuda.synchronize()
        sc.close()


def test_rows_of_one_launch_do_not_wait_for_candidate_arrays():
    """A context with room for rows that take two launches has two sets of candidate arrays; while its rows are shorter, a selection
    on a third stream uses neither, and must not wait for the fetches of the streams that did the first two."""
    import torch
    k, S = 64, 600
    sc = binding.SpeCache(3, 1, 1, 1, 2, 32, 65536, k, synth.FP16, async_select=2)
    idx = torch.full((3, k), -1, dtype=torch.int32, device="cuda")
    kv = torch.randn((2, 1, 1, S, 128), device="cuda").half()
    q = torch.randn((1, 1, 1, 128), device="cuda").half()

    def event_on(stream, timing=False):
        e = torch.cuda.Event(enable_timing=timing)
        e.record(stream)
        return e

    try:
        for L in range(3):
            sc.quantize_append(L, kv[0], kv[1], S)
            sc.score(L, q, 1)
        held = [torch.cuda.Stream() for _ in range(2)]
        torch.cuda._sleep(1000)
        torch.cuda.synchronize()
        begin = event_on(held[0], True)
        with torch.cuda.stream(held[0]):
            torch.cuda._sleep(1000000)
        end = event_on(held[0], True)
        torch.cuda.synchronize()
        cycles = int(1000000 * 30.0 / max(begin.elapsed_time(end), 0.1))      # 30 ms

        def hold():
            for stream in held:
                with torch.cuda.stream(stream):
                    torch.cuda._sleep(cycles)

        # streams share a few hardware queues: one whose work runs beside that of the held ones
        free = None
        for stream in [torch.cuda.Stream() for _ in range(8)]:
            hold()
            blocked = [event_on(s) for s in held]
            event_on(stream).synchronize()
            if not any(e.query() for e in blocked):
                free = stream
            torch.cuda.synchronize()
            if free is not None:
                break
        if free is None:
            pytest.skip("every stream shares a hardware queue with the held ones")
        hold()
        for L, stream in enumerate(held):
            sc.select_gather(L, idx[L], 0, stream)
        blocked = [event_on(s) for s in held]
        sc.select_gather(2, idx[2], 0, free)
        event_on(free).synchronize()
        waited = any(e.query() for e in blocked)
        torch.cuda.synchronize()
        assert not waited
        assert torch.equal(idx[0], idx[1]) and torch.equal(idx[0], idx[2]) and (idx >= 0).all()
    finally:
        torch.cuda.synchronize()
        sc.close()


def test_selection_captured_between_eager_ones():
    """score_topk lets its launch carry the event that a gather waits for; captured, it records it: replays give the eager positions and
    outputs, and an eager selection behind them orders a gather on another stream as before."""
    import torch
    from paper_2503_16163_amd import binding
    H, S, k = 4, 3000, 40
    q = synth.make_queries_device(9, 2, 1, H, 128, synth.FP16).view(2, 1, H, 2, 128)[:, :, :, :1].contiguous()
    kd, vd = synth.make_kv_device(9, 1, H, S, 128, synth.FP16)
    sc = binding.SpeCache(1, 1, H, H, 2, 32, 3072, k, synth.FP16)
    new = lambda: (torch.full((1, H, k), -2, dtype=torch.int32, device="cuda"), torch.zeros((1, H, 1, 128), dtype=torch.float32, device="cuda"))
    side = torch.cuda.Stream()
    try:
        sc.quantize_append(0, kd, vd, S)
        want = [new() for _ in range(2)]
        for i in range(2):
            sc.score_topk(0, q[i], 1, want[i][0])
            sc.attend(0, q[i], 1, None, None, -1, want[i][1])
        torch.cuda.synchronize()
        got, graph = new(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            st = torch.cuda.current_stream()
            sc.score_topk(0, q[0], 1, got[0], st)
            sc.attend(0, q[0], 1, None, None, -1, got[1], st)
        for _ in range(3):
            got[0].fill_(-2)
            got[1].zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(got[0], want[0][0]) and torch.equal(got[1], want[0][1])
            eager = new()
            sc.score_topk(0, q[1], 1, eager[0])
            sc.gather(0, eager[0], 0, side)
            sc.attend(0, q[1], 1, None, None, -1, eager[1])
            torch.cuda.synchronize()
            assert torch.equal(eager[0], want[1][0]) and torch.equal(eager[1], want[1][1])
    finally:
        torch.cuda.synchronize()
        sc.close()
