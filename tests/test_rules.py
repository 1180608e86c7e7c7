"""The rules by which a call takes one kernel or another (csrc/gss_rules.h), on the host."""

import random


def test_istft_plan_covers_every_block(rules):
    """Every block of 256 samples belongs to one workgroup and none is without a block, whatever the call's sizes."""
    rng = random.Random(1)
    for _ in range(20000):
        S, T = round(10 ** rng.uniform(0, 3.5)), 3 + round(10 ** rng.uniform(0, 5))
        waves, steps, per_seg = rules.istft(S, T, rng.choice([64, 256, 304]))
        per_wg = waves * steps - 3
        assert waves in (8, 16) and 1 <= steps <= (8 if waves == 8 else 32)
        assert per_seg * per_wg >= T - 3 and (per_seg - 1) * per_wg < T - 3, (S, T)


def test_istft_short_calls_take_8_wavefronts(rules):
    """An enhanced utterance of up to 20 s does not fill the compute units once with single steps of 8 wavefronts; these take two
    thirds of the time of 16.  The same for batches of short pieces."""
    for seconds in (1, 2, 5, 10, 18, 20):
        assert rules.istft(1, seconds * 16000 // 256 + 4)[:2] == (8, 1), seconds
    for S, T in ((8, 9), (60, 20), (128, 8), (168, 18), (277, 11), (3, 300)):
        assert rules.istft(S, T)[0] == 8, (S, T)


def test_istft_long_calls_keep_16_wavefronts(rules):
    """A workgroup of 16 wavefronts per compute unit, in full rounds: 128 segments of 18 s are 512 workgroups, two rounds."""
    for S, T, steps in ((128, 1129, 18), (10, 1566, 5), (30, 566, 5), (1, 62503, 16)):
        assert rules.istft(S, T)[:2] == (16, steps), (S, T)
