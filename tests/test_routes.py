"""Which kernel a call takes, on both sides of every line that is drawn by size (CPU: the rules are host code)."""
import math

import pytest

from gpu_common import fine_chunks, kernel_of, listed_slots

WIDE, SIXTEEN, EIGHT, GENERIC, REFUSED = "wide rows", "16 rows", "8 rows", "generic", "refused"

# heads, KV heads, query tokens, call, the last length on the kernel for wide rows (one sequence), the kernel past it.
# 256 compute units: a load of L tokens per unit and 32-row block ends at (L + 1) * 256 / KV heads / blocks of 32 rows - 1 tokens.
LINES_128 = [
    (64, 8, 4, "step", 40031, SIXTEEN), (64, 8, 4, "decode", 19231, SIXTEEN), (64, 8, 4, "lengths", 51231, SIXTEEN),
    (64, 8, 5, "step", 20031, SIXTEEN), (64, 8, 5, "decode", 9631, SIXTEEN),
    (128, 8, 1, "step", 35231, SIXTEEN), (128, 8, 1, "decode", 28831, SIXTEEN), (128, 8, 1, "lengths", 51231, SIXTEEN),
    (64, 8, 2, "step", 57631, SIXTEEN), (64, 8, 2, "decode", 38431, SIXTEEN),
    (32, 8, 2, "step", 30751, EIGHT), (16, 8, 2, "step", 16031, EIGHT), (4, 4, 2, "step", 32063, EIGHT),
]


@pytest.mark.parametrize("heads,kv,nq,call,last,other", LINES_128)
def test_lines_by_load_at_128(heads, kv, nq, call, last, other):
    assert kernel_of(1, heads, kv, 128, last, call, n_queries=nq) == WIDE
    assert kernel_of(1, heads, kv, 128, last + 1, call, n_queries=nq) == other
    assert kernel_of(1, heads, kv, 128, last + 5000, call, n_queries=nq, window=last - nq + 1) == WIDE     # (what is attended counts)
    assert kernel_of(1, heads, kv, 128, last + 5000, call, n_queries=nq, window=last - nq + 2) == other
    for variant, group, scale in ((1, 32, 1.0), (0, 64, 1.0), (0, 32, 0.0), (0, 32, -1.0), (0, 32, math.inf), (0, 32, math.nan)):
        assert kernel_of(1, heads, kv, 128, 64, call, n_queries=nq, variant=variant, group=group, scale=scale) != WIDE


@pytest.mark.parametrize("heads,nq,other", [(128, 1, SIXTEEN), (64, 2, SIXTEEN), (64, 8, SIXTEEN), (32, 2, EIGHT)])
def test_lines_by_sequences_at_128(heads, nq, other):
    for call in ("decode", "step", "lengths"):
        first = kernel_of(16, heads, 8, 128, 300, call, n_queries=nq)
        rows = heads // 8 * nq
        assert first == (other if (rows <= 8 and call != "step") or (rows > 16 and call == "decode") else WIDE)
        assert kernel_of(17, heads, 8, 128, 300, call, n_queries=nq) == other
    assert kernel_of(8, 64, 8, 128, 300, "decode", n_queries=4) == WIDE and kernel_of(9, 64, 8, 128, 300, "decode", n_queries=4) == SIXTEEN


def test_one_query_token_of_up_to_eight_rows_at_128():
    for heads, kv in ((8, 1), (64, 8), (32, 8), (32, 32), (3, 1)):
        for S in (1, 300, 8191, 131072):
            for call in ("decode", "step", "lengths"):
                assert kernel_of(1, heads, kv, 128, S, call) == EIGHT
    assert kernel_of(1, 64, 8, 128, 300, n_queries=4, scale=0.0) == REFUSED


def test_lines_at_256():
    for call in ("decode", "step", "lengths"):
        assert kernel_of(1, 32, 4, 256, 3072, call) == WIDE and kernel_of(1, 32, 4, 256, 3071, call) == EIGHT
        assert kernel_of(1, 16, 4, 256, 131072, call) == EIGHT and kernel_of(1, 20, 4, 256, 131072, call) == WIDE   # four rows, five
        assert kernel_of(1, 16, 8, 256, 33, call, n_queries=2) == WIDE and kernel_of(1, 8, 8, 256, 33, call, n_queries=2) == EIGHT
        line = 1024 if call == "lengths" else 512
        for batch, S, kernel in ((32, 100, WIDE), (33, line - 1, EIGHT), (33, line, WIDE)):
            assert kernel_of(batch, 16, 4, 256, S, call, n_queries=2) == kernel
        assert kernel_of(33, 32, 4, 256, line - 1, call) == EIGHT and kernel_of(33, 32, 4, 256, line, call) == WIDE
        for variant, group, scale in ((1, 32, 1.0), (0, 64, 1.0), (0, 32, 0.0), (0, 32, -1.0), (0, 32, math.inf)):
            assert kernel_of(1, 32, 4, 256, 8192, call, variant=variant, group=group, scale=scale) != WIDE


def test_always_at_512():
    for call in ("decode", "step", "lengths"):
        for scale in (1.0, 0.0, -2.0, 1e-40):
            assert kernel_of(3, 32, 1, 512, 1, call, scale=scale) == WIDE
        assert kernel_of(1, 32, 1, 512, 300, call, variant=1) == GENERIC
        assert kernel_of(1, 32, 1, 512, 300, call, group=64) == GENERIC
        assert kernel_of(1, 32, 1, 512, 300, call, scale=math.inf) == GENERIC
        assert kernel_of(1, 32, 1, 512, 300, call, variant=2, scale=0.0) == REFUSED


# (sequences, heads, KV heads, head dim, the longest bound that does not deal its waves to the sequences; 0: every bound does)
@pytest.mark.parametrize("B,heads,kv,d,last", [
    (63, 64, 8, 128, 0), (64, 64, 8, 128, 3072), (65, 64, 8, 128, 1024), (85, 64, 8, 128, 1024), (86, 64, 8, 128, 4096),
    (88, 64, 8, 128, 4096), (88, 32, 8, 128, 1024), (44, 64, 16, 128, 1024), (22, 32, 32, 128, 1024), (129, 64, 8, 128, 2048), (192, 64, 8, 128, 2048),
    (48, 32, 32, 128, 2048), (31, 32, 16, 256, 0), (32, 32, 16, 256, 2048), (33, 32, 16, 256, 256), (42, 32, 16, 256, 256),
    (44, 32, 16, 256, 256), (45, 32, 16, 256, 2048), (65, 32, 16, 256, 2048), (109, 32, 16, 256, 2048), (8, 72, 72, 128, 1024), (5, 96, 96, 128, 0), (3, 129, 129, 128, 0)])
def test_lengths_that_are_dealt_to_waves(B, heads, kv, d, last):
    slots = 256 // kv * 8
    assert listed_slots(B, heads, kv, d, last + 1) == slots and (last == 0 or listed_slots(B, heads, kv, d, last) == 0)
    for more in (dict(window=100), dict(n_splits=2), dict(variant=1), dict(n_queries=2)):
        assert listed_slots(B, heads, kv, d, 5000, **more) == 0


# (sequences, heads, KV heads, head dim, group, the longest bound that deals its waves to the sequences): beyond it the slots are too few
@pytest.mark.parametrize("B,heads,kv,d,group,most", [
    (193, 64, 8, 128, 32, 3072), (213, 64, 8, 128, 32, 3072), (193, 32, 8, 128, 64, 3072), (205, 32, 8, 128, 32, 4096), (219, 32, 8, 128, 32, 4096),
    (52, 32, 32, 128, 32, 4096), (54, 32, 32, 128, 32, 4096), (109, 64, 16, 128, 32, 4096)])
def test_slots_that_are_enough_up_to_a_bound(B, heads, kv, d, group, most):
    assert [listed_slots(B, heads, kv, d, bound, group) > 0 for bound in (2048, 2049, most, most + 1, 50000)] == [False, True, True, False, False]


# too few slots to a sequence, at any bound, or half the chip without a block
@pytest.mark.parametrize("B,heads,kv,d", [
    (89, 64, 8, 128), (128, 64, 8, 128), (214, 64, 8, 128), (55, 32, 32, 128), (56, 32, 32, 128), (220, 64, 8, 128), (110, 64, 16, 128),
    (28, 64, 64, 128), (110, 32, 16, 256), (6, 96, 96, 128), (4, 129, 129, 128), (4, 256, 256, 128)])
def test_too_few_slots_to_deal(B, heads, kv, d):
    assert all(listed_slots(B, heads, kv, d, bound) == 0 for bound in (100, 1500, 2500, 3500, 8000, 131072))


def test_lengths_that_are_not_dealt_to_waves():
    assert listed_slots(192, 8, 1, 128, 5000) == 2048
    assert listed_slots(256, 8, 1, 128, 5000) == 2048 and listed_slots(257, 8, 1, 128, 5000) == 0
    assert listed_slots(4, 128, 8, 128, 60000) == 0 and listed_slots(4, 32, 4, 256, 5000) == 0   # 16-row tile, rows in several blocks
    assert listed_slots(4, 32, 1, 512, 5000) == 0


# (heads, KV heads, head dim, group, query tokens, the longest sequence that stays one chunk): the merge is dearer than a wave's second tile
# in the 4-row tile and outside the plain instances of head_dim 128
@pytest.mark.parametrize("heads,kv,d,group,nq,last", [
    (8, 1, 128, 32, 1, 256), (64, 8, 128, 32, 1, 256), (32, 8, 128, 32, 1, 384), (32, 32, 128, 32, 1, 384), (64, 8, 128, 64, 1, 384),
    (32, 8, 128, 128, 1, 384), (32, 8, 128, 32, 2, 384), (32, 16, 256, 32, 1, 256), (32, 16, 256, 64, 1, 256)])
def test_short_sequences_that_stay_one_chunk(heads, kv, d, group, nq, last):
    assert fine_chunks(1, heads, kv, d, last, group, nq) == 1
    assert fine_chunks(1, heads, kv, d, last + 1, group, nq) == (last // 32 + 2) // 2
    assert fine_chunks(1, heads, kv, d, 480, group, nq) == 8
    assert fine_chunks(256 // kv, heads, kv, d, 480, group, nq) == 1              # (no compute units for a second chunk)
