"""The rules by which a call takes one kernel or another (csrc/gss_rules.h), on the host."""

import random

import pytest


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


@pytest.mark.parametrize("D,K,S,T,iters,ragged,one,four", [
    (4, 3, 1, 64, 15, False, 39.6, 35.2), (2, 3, 1, 64, 8, False, 16.7, 14.6), (4, 2, 1, 52, 8, False, 23.3, 18.1),
    (2, 8, 1, 60, 15, False, 40.1, 52.0), (2, 5, 2, 125, 10, False, 37.0, 41.0), (2, 3, 3, 46, 10, False, 22.9, 32.3),
    (3, 3, 3, 271, 15, False, 86.4, 118.0), (4, 2, 3, 346, 5, False, 44.3, 55.0), (3, 4, 3, 397, 15, True, 113.2, 145.3),
    (3, 3, 4, 381, 5, True, 42.2, 53.4), (1, 3, 8, 1296, 15, True, 208.1, 210.8), (4, 3, 6, 636, 15, False, 335.8, 315.1),
    (3, 6, 5, 999, 15, False, 452.7, 399.8), (3, 2, 1, 296, 15, True, 54.5, 47.3), (4, 6, 2, 140, 12, True, 99.6, 88.5),
    (2, 6, 7, 1431, 20, True, 375.3, 433.4), (4, 2, 5, 893, 5, False, 105.1, 118.1),
    (4, 2, 3, 779, 10, True, 103.0, 118.0), (4, 2, 5, 1356, 19, True, 309.1, 349.8)])
def test_em_four_wavefronts_where_measured(rules, D, K, S, T, iters, ragged, one, four):
    """Calls measured with one and with four wavefronts per problem (us, 513 bins, 256 compute units): the one that is
    chosen takes at most a tenth longer than the other."""
    assert (four if rules.em_four_wavefronts(D, K, S, T, iters, ragged) else one) <= 1.1 * min(one, four)


def test_em_four_wavefronts_for_one_short_segment(rules):
    """One segment of one tile: a launch less, and faster or as fast whatever the channels and classes, but for the two kernels
    that keep registers in scratch memory."""
    for D in (1, 2, 3, 4):
        for K in range(1, 9):
            for T in (1, 40, 64):
                assert rules.em_four_wavefronts(D, K, 1, T, 8) == (D != 2 or K < 7), (D, K, T)
                assert rules.em_four_wavefronts(D, K, 1, T, 1), (D, K, T)


@pytest.mark.parametrize("D,K,S,T,F,one,chunks", [
    (8, 5, 1, 348, 65, 132.8, 97.6), (8, 3, 1, 383, 65, 127.0, 104.5), (8, 2, 1, 346, 65, 115.5, 97.5), (8, 6, 3, 333, 65, 286.9, 228.4),
    (7, 1, 1, 673, 65, 201.1, 131.0), (6, 4, 1, 300, 513, 0.92, 1.0), (8, 5, 1, 330, 513, 0.92, 1.0), (8, 5, 4, 701, 513, 0.95, 1.0),
    (8, 5, 2, 1875, 513, 1.33, 1.0)])
def test_em_one_launch_where_measured(rules, D, K, S, T, F, one, chunks):
    """Calls of 5 to 8 channels measured in one launch and in chunks (us, or relative; 256 compute units): the faster one is chosen."""
    assert rules.em_one_launch(D, S, T, False, F) == (one < chunks)
