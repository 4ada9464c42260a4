"""Which decode calls run in one launch, without a GPU: the rule on sizes, and that a test may set it for its own thread."""
import threading

import pytest

from paper_2404_09526_amd import binding as esp


# requests of one length that fill the chip, (query heads, KV heads): the last length that was measured to gain, and one that was not
@pytest.mark.parametrize("Hq,Hkv,gains,not_any_more", [(4, 4, 2000, 4000), (32, 32, 2000, 8000), (8, 4, 8000, 16000), (64, 32, 8000, 32000),
                                                        (32, 1, 16000, 131072), (32, 4, 2000, 16000), (32, 8, 4000, 16000), (12, 12, 2000, 8000)])
def test_long_requests_are_cut_into_ranges(Hq, Hkv, gains, not_any_more):
    B = 256 // Hkv
    for n, plan in ((gains, 2), (not_any_more, 1), (131072, 1)):
        assert esp.esp_debug_decode_plan(B, B * n, n, Hq, Hkv) == plan, n
    # the longest one walks alone, half the chip is idle (8 of 1000, 16 / 8 heads), and a bound beyond all
    assert esp.esp_debug_decode_plan(64, 260980, 7000, 32, 4) == 1 and esp.esp_debug_decode_plan(8, 8000, 1000, 16, 8) == 1
    assert esp.esp_debug_decode_plan(64, 2 ** 31 - 1, 2 ** 25, 8, 4) == 1


@pytest.mark.parametrize("sizes,plan", [
    ((4, 1283, 485, 4, 4), 2), ((1, 200, 200, 32, 8), 2), ((30, 30000, 1000, 32, 8), 2), ((250, 130000, 520, 32, 1), 2),
    ((8, 8000, 1000, 64, 32), 2), ((256, 256, 1, 32, 1), 2), ((1, 64, 64, 66, 1), 2),
    ((257, 257, 1, 32, 1), 1), ((5, 5, 1, 64, 64), 1), ((129, 129, 1, 40, 1), 1),            # more workgroups than CUs (40 / 1: two chunks each)
    ((16, 14312, 3077, 32, 8), 1), ((3, 2100, 700, 32, 8), 1), ((12, 12000, 1000, 4, 4), 1),   # the longest request's walk
    ((64, 887489, 88062, 32, 32), 1), ((1, 2 ** 31 - 1, 2 ** 31 - 1, 32, 1), 1), ((2 ** 31 - 1, 2 ** 31 - 1, 1, 64, 32), 1),
    ((0, 0, 0, 8, 8), 1), ((5, 0, 0, 8, 8), 1), ((3, 10, 10, 8, 3), 0), ((-1, 10, 10, 8, 8), 0)])
def test_which_calls_run_in_one_launch(sizes, plan):
    assert esp.esp_debug_decode_plan(*sizes) == plan


def test_a_plan_is_set_for_the_thread_that_asks():
    sizes = (4, 1283, 485, 4, 4)
    for plan in (1, 2):
        assert esp.esp_debug_set_decode_plan(plan) == 0
        try:
            there = []
            t = threading.Thread(target=lambda: there.append(esp.esp_debug_decode_plan(64, 887489, 88062, 32, 32)))
            t.start()
            t.join()
            assert esp.esp_debug_decode_plan(*sizes) == plan and there == [1]
        finally:
            assert esp.esp_debug_set_decode_plan(0) == plan
    assert esp.esp_debug_set_decode_plan(3) == 0 and esp.esp_debug_set_decode_plan(0) == 0
