"""Several query rows per KV head on the f16 matrix cores (rows_kernel): scoring and attention in one launch and as two,
at the sizes where units of tokens, waves and chunks end."""
import numpy as np
import pytest

from paper_2503_16163_amd import binding, synth

pytestmark = pytest.mark.gpu

# Multipliers and p s are hi + lo f16, each rounded to nearest: 2^-23 of a product, and sums of 128 in binary32 are good for about
# the same.  The products of a logit add up to at most about ten times the largest logit of a row (128 channels, outlier
# channels included), so 3e-6 of it, 5e-6 with the zero-point term; an output is a convex combination of such errors in numerator
# and softmax: four times that.
LOGITS, OUTPUTS = 5e-6, 2e-5


@pytest.mark.parametrize("B,Hq,Hkv,S,dtype,bits,g,R,k", [
    (1, 4, 1, 90, synth.FP16, 2, 32, 64, 16),       # 32 quantised positions: half a unit, three empty waves
    (1, 4, 1, 130, synth.BF16, 2, 32, 64, 300),     # one unit and a half; more pairs asked for than there are
    (1, 8, 2, 1700, synth.BF16, 2, 64, 64, 48),     # a token group is a unit
    (2, 8, 2, 2100, synth.FP16, 2, 128, 128, 300),  # a token group is two units
    (1, 8, 2, 1300, synth.BF16, 1, 32, 64, 40),
    (1, 8, 2, 1500, synth.FP16, 1, 128, 256, 40),
    (1, 8, 1, 100, synth.FP16, 2, 32, 64, 16),      # 16 rows: a unit is 32 positions
    (1, 16, 2, 1700, synth.BF16, 2, 64, 64, 130),   # 16 rows, a token group is two units, two chunks of 16-bit pairs
    (1, 16, 2, 1300, synth.FP16, 1, 32, 64, 40),
    (3, 24, 3, 2600, synth.BF16, 2, 128, 128, 64),  # 16 rows, a token group is four units
])
@pytest.mark.parametrize("calls", ["one-pass", "carry", "split"])
def test_rows_kernel(B, Hq, Hkv, S, dtype, bits, g, R, k, calls):
    from tests.harness import Case
    binding.debug_kernel_choice(binding.KEEP_ONE_PASS_LOGITS)
    c = Case(B, Hq, Hkv, S, dtype, bits, g, k, R=R, seed=5100 + Hq + g + bits + S, async_select=2, one_pass=calls != "split",
             fused_append=calls == "carry")
    try:
        c.load()
        c.decode_step()                      # nothing staged yet
        for t in range(36):                  # across a flush
            c.append_token(t)
            c.decode_step(check_logits=(t % 6 == 0))
        assert c.sc.counts(0)[0] == S + 36
        print(c.stats)
        assert c.stats["max_logit_err"] < LOGITS and c.stats["max_out_err"] < OUTPUTS
    finally:
        c.close()
        binding.debug_kernel_choice(0)


@pytest.mark.parametrize("S", [40000, 70000])
def test_rows_kernel_with_several_units_per_wave(S):
    """Long rows: every wave walks several units (running maximum, prefetched loads), the last chunk is short."""
    from tests.harness import Case
    binding.debug_kernel_choice(binding.KEEP_ONE_PASS_LOGITS)
    c = Case(2, 64, 16, S, synth.BF16, 2, 32, 64, seed=5200, async_select=2, one_pass=True, sample=[(0, 0), (1, 15)])
    try:
        c.load()
        for t in range(3):
            c.append_token(t)
            c.decode_step()
        print(c.stats)
        assert c.stats["max_logit_err"] < LOGITS and c.stats["max_out_err"] < OUTPUTS
    finally:
        c.close()
        binding.debug_kernel_choice(0)


@pytest.mark.parametrize("B,Hq,Hkv,S,dtype,g,R,k,n_rows", [
    (1, 2, 2, 100, synth.FP16, 32, 64, 16, 1),      # one row per KV head, 64 quantised positions: one unit
    (2, 3, 3, 1500, synth.FP16, 32, 128, 300, 2),   # two rows, three chunks of 16-bit pairs
    (1, 4, 2, 90, synth.BF16, 32, 64, 40, 2),       # four rows, half a unit
    (1, 4, 1, 1300, synth.BF16, 64, 64, 48, 1),     # four rows, one of each head
    (2, 8, 2, 2100, synth.FP16, 128, 128, 64, 2),   # eight rows, a token group is two units
    (1, 16, 2, 1300, synth.BF16, 32, 96, 40, 2),    # sixteen rows
    (1, 8, 1, 900, synth.FP16, 128, 256, 40, 2),
])
@pytest.mark.parametrize("calls", ["split", "fused append"])
def test_rows_kernel_on_four_bit_codes(B, Hq, Hkv, S, dtype, g, R, k, n_rows, calls):
    """4-bit codes take the kernel with any number of rows: with fewer than 8 some of its columns have no row."""
    from tests.harness import Case
    c = Case(B, Hq, Hkv, S, dtype, 4, g, k, R=R, seed=5300 + Hq + g + S, n_rows=n_rows, async_select=2, fused_append=calls != "split")
    try:
        c.load()
        c.check_quantized()
        c.decode_step(use_spec=n_rows == 2)
        for t in range(36):
            c.append_token(t)
            c.decode_step(use_spec=n_rows == 2, check_logits=(t % 6 == 0))
        c.check_quantized()
        print(c.stats)
        assert c.stats["max_logit_err"] < LOGITS and c.stats["max_out_err"] < OUTPUTS
    finally:
        c.close()


@pytest.mark.parametrize("B,Hq,Hkv,S,dtype,bits,g,R,k,n_rows", [
    (1, 2, 1, 90, synth.FP16, 2, 32, 64, 16, 2),       # 32 quantised positions: half a unit, three empty waves
    (1, 4, 2, 130, synth.BF16, 1, 32, 64, 300, 2),     # one unit and a half; more pairs asked for than there are
    (1, 4, 2, 1700, synth.BF16, 2, 64, 64, 48, 2),     # a token group is a unit
    (2, 6, 3, 2100, synth.FP16, 2, 128, 128, 300, 2),  # a token group is two units, three chunks of 16-bit pairs
    (1, 4, 2, 1500, synth.FP16, 1, 128, 256, 40, 2),
    (1, 8, 2, 1300, synth.BF16, 2, 32, 64, 40, 1),     # one row of each of four heads
    (1, 4, 1, 1500, synth.FP16, 1, 64, 64, 130, 1),
])
@pytest.mark.parametrize("calls", ["one-pass", "carry", "split"])
def test_rows_kernel_with_four_rows(B, Hq, Hkv, S, dtype, bits, g, R, k, n_rows, calls):
    """Four rows of 1- and 2-bit codes run as eight, of which four do not exist."""
    from tests.harness import Case
    binding.debug_kernel_choice(binding.KEEP_ONE_PASS_LOGITS)
    c = Case(B, Hq, Hkv, S, dtype, bits, g, k, R=R, seed=5500 + Hq + g + bits + S, n_rows=n_rows, async_select=2,
             one_pass=calls != "split", fused_append=calls == "carry")
    try:
        c.load()
        c.decode_step(use_spec=n_rows == 2)
        for t in range(36):                  # across a flush
            c.append_token(t)
            c.decode_step(use_spec=n_rows == 2, check_logits=(t % 6 == 0))
        print(c.stats)
        assert c.stats["max_logit_err"] < LOGITS and c.stats["max_out_err"] < OUTPUTS
    finally:
        c.close()
        binding.debug_kernel_choice(0)


def test_attend_after_the_one_launch_call():
    """The one launch of grouped-query heads leaves no logits; an attend of the same cache state behind it still works
    (it scores again) and gives the same output up to the rounding of other partial sums."""
    import torch
    from tests.harness import Case, to_dev
    c = Case(1, 8, 2, 1700, synth.BF16, 2, 64, 48, seed=5400, async_select=2, one_pass=True)
    try:
        c.load()
        _, out = c.decode_step(use_spec=False, check_logits=False, do_gather=False)
        again = torch.empty((1, 8, 2, 128), dtype=torch.float32, device="cuda")
        c.sc.attend(0, to_dev(c.last_q_bits, c.dtype), 2, None, None, -1, again, torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert abs(again.cpu().numpy() - out).max() <= OUTPUTS * abs(out).max()
    finally:
        c.close()


def _spread(c, kind, rng):
    """Keys and values of the case with scales far apart, in place."""
    M = 128 // c.g
    for b, h in c.sample:
        k, v = synth.from_bits(c.k_bits[b, h], c.dtype).copy(), synth.from_bits(c.v_bits[b, h], c.dtype).copy()
        S = v.shape[0]
        if kind in ("value groups", "large token"):
            v *= np.where(np.arange(128) // c.g < M // 2, 2.0 ** -12, 1.0).astype(np.float32)[None] if M > 1 else 1.0
        if kind == "large token":             # the first tokens of a wave's walk, and one in the middle
            v[[3, 40, S // 2]] *= 256.0
        if kind == "tokens":
            v *= np.exp2(rng.integers(-6, 7, size=S)).astype(np.float32)[:, None]
        if kind == "key channels":
            k *= np.exp2(rng.permutation(np.linspace(-6, 6, 128).round())).astype(np.float32)[None]
        if kind == "key groups":
            k *= np.exp2(rng.integers(-10, 1, size=-(-S // 32))).astype(np.float32).repeat(32)[:S, None]
        if kind == "huge key":                # (its query is as small, below)
            k[3::97, 5] = 2.0 ** 40
        if kind == "nothing":
            k[:, 7] = 0.0
            v[:, :32] = 0.5
        c.k_bits[b, h], c.v_bits[b, h] = synth.to_bits(k, c.dtype), synth.to_bits(v, c.dtype)


@pytest.mark.parametrize("kind,dtype", [("value groups", synth.FP16), ("large token", synth.BF16), ("tokens", synth.FP16), ("key channels", synth.BF16),
                                        ("key groups", synth.FP16), ("huge key", synth.BF16), ("nothing", synth.FP16)])
@pytest.mark.parametrize("B,Hq,Hkv,S,bits,g,n_rows", [
    (1, 4, 2, 2500, 2, 32, 2),         # four rows
    (1, 8, 2, 2500, 2, 64, 2),
    (1, 8, 2, 2500, 1, 32, 2),
    (1, 16, 2, 2500, 2, 32, 2),        # sixteen rows: a value group's scales lie in every other or every fourth lane
    (1, 16, 2, 2500, 1, 64, 2),
    (1, 3, 3, 2500, 4, 32, 2),
    (2, 64, 16, 40000, 2, 64, 2),      # waves of several units
])
def test_rows_kernel_with_scales_far_apart(kind, dtype, B, Hq, Hkv, S, bits, g, n_rows):
    """Value groups of a token, tokens, key channels and token groups up to 4096 apart, single tokens far above the rest, a key channel
    2^40 above the others that the query all but ignores, a zero query and constant channels: the f16 operands keep what binary32
    kept.  Outputs are compared per value group, so that small channels count as much as large ones."""
    import torch
    from tests.harness import Case, to_dev
    binding.debug_kernel_choice(binding.KEEP_ONE_PASS_LOGITS)
    c = Case(B, Hq, Hkv, S, dtype, bits, g, 16, R=max(64, g), seed=5600 + Hq + bits, n_rows=n_rows, async_select=2,
             sample=[(0, 0)] if S > 10000 else None)
    try:
        _spread(c, kind, np.random.default_rng(17))
        c.load()
        q_bits = synth.make_queries(c.seed, B, Hq, 128, dtype, n_rows=n_rows)
        if kind in ("huge key", "nothing"):
            q = synth.from_bits(q_bits, dtype).copy()
            if kind == "huge key":
                q[..., 5] *= 2.0 ** -44
            else:
                q[:, ::2] = 0.0
            q_bits = synth.to_bits(q, dtype).reshape(q_bits.shape)
        q, stream = to_dev(q_bits, dtype), torch.cuda.current_stream()
        out = torch.empty((B, Hq, n_rows, 128), dtype=torch.float32, device="cuda")
        c.sc.score_attend(0, q, n_rows, None, None, -1, out, stream)
        torch.cuda.synchronize()
        logits, got = c.sc.debug_logits(0, n_rows), out.cpu().numpy().astype(np.float64)
        for b, h in c.sample:
            heads = slice(h * c.G, (h + 1) * c.G)
            want_logits, _ = c.oc[(b, h)].scores(q_bits[b, heads], c.sm_scale)
            err = np.abs(logits[b, heads] - want_logits).max(-1) / np.maximum(np.abs(want_logits).max(-1), 1e-30)
            assert err.max() < LOGITS, (b, h, err.max())
            want = c.oc[(b, h)].attend(q_bits[b, heads], c.sm_scale).reshape(c.G, n_rows, 128 // g, g)
            diff = got[b, heads].reshape(want.shape) - want
            err = np.sqrt((diff ** 2).sum(-1) / (want ** 2).sum(-1))
            print(kind, (b, h), "outputs", err.max())
            assert err.max() < OUTPUTS, (b, h, err.max())
    finally:
        c.close()
        binding.debug_kernel_choice(0)


@pytest.mark.parametrize("Hq,Hkv,bits,n_rows", [(8, 2, 2, 2), (4, 2, 1, 2), (8, 1, 2, 2), (8, 2, 1, 1)])
def test_logits_after_the_one_launch_call(Hq, Hkv, bits, n_rows):
    """The one launch of grouped-query heads keeps its queries in place of the logits: specache_debug_logits works them out from those,
    also when the caller's buffer holds something else by then and the cache has grown."""
    import torch
    from tests.harness import Case, to_dev
    c = Case(1, Hq, Hkv, 1700, synth.BF16, bits, 32, 48, seed=5700 + Hq, n_rows=n_rows, async_select=2, one_pass=True)
    try:
        c.load()
        q_bits = synth.make_queries(c.seed, 1, Hq, 128, c.dtype, n_rows=n_rows)
        q = to_dev(q_bits, c.dtype)
        out = torch.empty((1, Hq, n_rows, 128), dtype=torch.float32, device="cuda")
        want = [c.oc[0, h].scores(q_bits[0, h * c.G:(h + 1) * c.G], c.sm_scale)[0] for h in range(Hkv)]
        c.sc.score_attend(0, q, n_rows, None, None, -1, out, torch.cuda.current_stream())
        q.zero_()
        c.append_token(0)
        got = c.sc.debug_logits(0, n_rows)
        for h in range(Hkv):
            err = np.abs(got[0, h * c.G:(h + 1) * c.G] - want[h]).max(-1) / np.abs(want[h]).max(-1)
            assert err.max() < LOGITS
    finally:
        c.close()
