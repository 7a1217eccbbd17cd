"""Several query rows per KV head on the f16 matrix cores (rows_kernel): scoring and attention in one launch and as two,
at the sizes where units of tokens, waves and chunks end."""
import pytest

from paper_2503_16163_amd import binding, synth

pytestmark = pytest.mark.gpu

# Multipliers and p s are hi + lo f16, each truncated: 2^-21 of a product.  The products of a logit add up to at most
# about ten times the largest logit of a row (128 channels, outlier channels included), so 5e-6 of it; an output is a
# convex combination of such errors in numerator and softmax: four times that.
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
