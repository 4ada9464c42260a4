"""Which prefill kernel a call runs on, and in how many parts (host code; no GPU)."""
import ctypes
import math
import random
import threading

import pytest


@pytest.fixture(scope="module")
def esp():
    from paper_2404_09526_amd import binding
    return binding


def test_a_forced_plan_holds_for_its_thread_and_for_the_workspaces_it_asks_for(esp):
    sizes = (40, 3000, 1, 40, 3000, 8, 2)
    by_estimate, room = esp.esp_debug_prefill_plan(*sizes), esp.esp_prefill_workspace_bytes(40, 3000, 1, 8, 2, 128)
    assert by_estimate != 0
    part = 40 * 8 * (128 + 1) * 4
    for plan in (1, 5, -1, -7):                                   # (room for fewer parts than were forced: one)
        assert esp.esp_debug_set_prefill_plan(plan) == 0
        try:
            need = 256 + (abs(plan) * part if abs(plan) > 1 else 0)
            assert esp.esp_debug_prefill_plan(*sizes) == plan and esp.esp_prefill_workspace_bytes(40, 3000, 1, 8, 2, 128) == need
            assert esp.esp_debug_prefill_plan(*sizes, workspace_bytes=256) == (1 if plan > 0 else -1)
            there = []
            t = threading.Thread(target=lambda: there.append((esp.esp_debug_prefill_plan(*sizes), esp.esp_prefill_workspace_bytes(40, 3000, 1, 8, 2, 128))))
            t.start(); t.join()
            assert there == [(by_estimate, room)]
        finally:
            assert esp.esp_debug_set_prefill_plan(0) == plan
    assert esp.esp_debug_prefill_plan(*sizes) == by_estimate
    assert esp.esp_debug_set_prefill_plan(17) == 0 and esp.esp_debug_set_prefill_plan(0) == 0            # beyond ESP_MAX_PARTIALS: none
    assert esp.esp_debug_prefill_plan(40, 3000, 1, 40, 3000, 8, 3) == 0                                  # Hq % Hkv


def room_for(parts, Tq, Hq):
    return 256 + (parts * (Tq * Hq * 512 + (Tq * Hq * 4 + 255) // 256 * 256) if parts > 1 else 0)


@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (4, 4), (32, 8), (64, 8), (12, 12)])
def test_one_request_asks_for_the_room_that_its_parts_take(esp, Hq, Hkv):
    for Tq, Tkv in ((1, 1), (1100, 1100), (1024, 1024), (256, 512), (40, 3000), (300, 20300), (31, 70195), (2000, 9000), (1488, 210407)):
        parts = abs(esp.esp_debug_prefill_plan(Tq, Tkv, 1, Tq, Tkv, Hq, Hkv))
        assert esp.esp_prefill_workspace_bytes(Tq, Tkv, 1, Hq, Hkv, 128) == room_for(parts, Tq, Hq), (Tq, Tkv, parts)


# (new tokens, tokens in the shard) of the requests, query heads, KV heads, least parts that the longest request has to be cut in: uncut,
# or cut as the average request would be, its walk by one workgroup set the time of the call (us, cut by the average -> by the longest)
UNEVEN = [([(16, 8192)] + [(16, 512)] * 7, 32, 8, 3),           # 64 -> 32
          ([(32, 16384)] + [(32, 512)] * 7, 8, 8, 4),            # 70 -> 35
          ([(32, 60000)] + [(32, 64)] * 31, 4, 4, 8),            # 408 -> 68
          ([(8, 200000)] + [(8, 512)] * 63, 32, 8, 6),           # 2210 -> 480
          ([(300, 20300)] + [(300, 600)] * 3, 32, 8, 3)]         # 324 -> 161


@pytest.mark.parametrize("requests,Hq,Hkv,parts", UNEVEN)
def test_the_longest_request_of_a_batch_is_cut(esp, requests, Hq, Hkv, parts):
    new, rows = zip(*requests)
    sizes, heads = (sum(new), sum(rows), len(requests)), (Hq, Hkv)
    room = esp.esp_prefill_workspace_bytes(*sizes, *heads, 128)
    plan = esp.esp_debug_prefill_plan(*sizes, max(new), max(rows), *heads, workspace_bytes=room)
    assert abs(plan) >= parts and room_for(abs(plan), sum(new), Hq) <= room
    assert esp.esp_debug_prefill_plan(*sizes, max(new), max(rows), *heads) == plan          # no other in a larger workspace
    # requests of one length are cut as their average says, whether or not the bound on it is a row or two too high
    even = -(-sum(rows) // len(requests))
    assert esp.esp_debug_prefill_plan(*sizes, max(new), even, *heads) == esp.esp_debug_prefill_plan(*sizes, max(new), 0, *heads)


# lengths of prompts, heads, the plans that were within 10 % of the best measured (us, best of these; the others)
UNEVEN_PROMPTS = [([2000] + [32] * 15, 8, 8, {-1}),                                               # 30.3; uncut on the main kernel 34.3
                  ([4000] + [32] * 7, 4, 4, {-1, 3}),                                             # 44.7; uncut 55.3
                  ([6000] + [32] * 15, 4, 4, {2, 3, 4}),                                          # 67.9; uncut 75.4, the kernel for few rows 88.0
                  ([8000] + [64] * 7, 4, 4, {1, 2, 3, 5}),                                        # 89.2; the kernel for few rows 144.1
                  ([102, 105, 115, 231, 235, 250, 266, 276, 378, 616, 815, 1228], 4, 4, {-1})]    # 23.6; uncut 27.1


@pytest.mark.parametrize("prompts,Hq,Hkv,good", UNEVEN_PROMPTS)
def test_one_long_prompt_beside_short_ones(esp, prompts, Hq, Hkv, good):
    """A batch takes no less than its longest request does: neither where that is the paired sweep of a call of one round nor where
    the kernel for few rows has most of its blocks there."""
    sizes = (sum(prompts), sum(prompts), len(prompts))
    plan = esp.esp_debug_prefill_plan(*sizes, max(prompts), max(prompts), Hq, Hkv, workspace_bytes=esp.esp_prefill_workspace_bytes(*sizes, Hq, Hkv, 128))
    assert plan in good


# tokens, rows, heads, the plans within 10 % of the best measured: with a causal mask, where rows may see a triangle of the shard or, lying
# behind it, all (within 10 % in either; us, worse of the two, best of these and the triangle's own choice); without a mask
NEAR = [(4088, 4088, 4, 4, {3, 4}, {3, 4}),                     # 51, 61 on the kernel for few rows
        (2427, 3640, 4, 4, {5, 6}, {4, 5, 6}),                  # 37, 51 on the kernel for few rows
        (1715, 2572, 12, 12, {2, 3}, {2, 3}),                   # 44, 54 uncut
        (2427, 2427, 8, 8, {3}, {2, 3}),                        # 41, 50 uncut
        (510, 1275, 32, 8, {-1}, {-1}),                         # 26, 32 uncut on the main kernel
        (472, 472, 40, 8, {1}, {1, -1}),                        # 20, 22 on the kernel for few rows
        (2048, 2048, 32, 8, {1}, {1}), (1000, 1000, 32, 32, {1}, {1}), (4000, 4000, 16, 16, {1}, {1}), (6000, 6000, 8, 8, {1}, {1})]   # pairs


@pytest.mark.parametrize("Tq,Tkv,Hq,Hkv,causal,full", NEAR)
def test_a_chunk_may_lie_behind_its_shard_or_have_no_mask(esp, Tq, Tkv, Hq, Hkv, causal, full):
    assert esp.esp_debug_prefill_plan(Tq, Tkv, 1, Tq, Tkv, Hq, Hkv) in causal
    assert esp.esp_debug_prefill_plan(Tq, Tkv, 1, Tq, Tkv, Hq, Hkv, causal=False) in full


def test_the_plan_of_a_call_that_keeps_rows_is_told(esp):
    """Such calls are not paired: 1500 on 1500, 12 / 12 heads, runs on one kernel or the other."""
    plan = lambda kept: esp.esp_debug_prefill_plan(1500, 1500, 1, 1500, 1500, 12, 12, kept=kept)
    assert plan(False) == 1 and plan(True) == -1


def test_the_workspace_holds_the_parts_of_every_kind_of_call(esp):
    rng = random.Random(9)
    for _ in range(1000):
        Hkv, batch, Tkv = rng.choice((1, 4, 8, 12, 32)), rng.choice((1, 1, 3, 20)), int(math.exp(rng.uniform(0, math.log(60000))))
        Hq, Tq = Hkv * rng.choice((1, 2, 4, 8)), max(1, int(Tkv * rng.uniform(0.1, 1.2)))
        room = esp.esp_prefill_workspace_bytes(Tq, Tkv, batch, Hq, Hkv, 128)
        for causal in (True, False):
            for kept in (True, False):
                plan = lambda **kw: esp.esp_debug_prefill_plan(Tq, Tkv, batch, Tq, Tkv, Hq, Hkv, causal=causal, kept=kept, **kw)
                assert room_for(abs(plan()), Tq, Hq) <= room and plan(workspace_bytes=room) == plan()


def test_a_batch_never_runs_in_more_parts_than_its_workspace_holds(esp):
    rng = random.Random(7)
    size = lambda top: int(math.exp(rng.uniform(0, math.log(top))))
    for _ in range(2000):
        Hkv = rng.choice((1, 2, 4, 8, 12, 32))
        Hq, batch = Hkv * rng.choice((1, 2, 4, 8)), rng.randint(1, 64)
        new, rows = [size(3000) for _ in range(batch)], [size(100000) for _ in range(batch)]
        sizes = (sum(new), sum(rows), batch)
        room = esp.esp_prefill_workspace_bytes(*sizes, Hq, Hkv, 128)
        for longest in (max(rows), sum(rows)) if batch > 1 else (sum(rows),):
            q = max(new) if batch > 1 else sum(new)
            plan = esp.esp_debug_prefill_plan(*sizes, q, longest, Hq, Hkv)
            assert room_for(abs(plan), sum(new), Hq) <= room and 1 <= abs(plan) <= 16
            assert esp.esp_debug_prefill_plan(*sizes, q, longest, Hq, Hkv, workspace_bytes=room) == plan


def test_a_smaller_workspace_holds_as_many_parts_as_fit(esp):
    """... and not none at once: the call with room for fewer parts than it would like runs in the best number of those."""
    sizes, Hq = (300, 20300, 1, 300, 20300, 32, 8), 32
    want = esp.esp_debug_prefill_plan(*sizes)
    assert want >= 4
    for n in range(1, want + 1):
        for spare in (0, 255):
            plan = abs(esp.esp_debug_prefill_plan(*sizes, workspace_bytes=room_for(n, 300, Hq) + spare))
            assert plan <= n and (plan > 1) == (n > 1), (n, plan)
    assert esp.esp_debug_prefill_plan(*sizes, workspace_bytes=room_for(want, 300, Hq) - 1) == want - 1


def test_the_size_of_a_call_that_would_be_refused_is_zero_for_pool_rows_too(esp):
    """No KV heads divided by zero."""
    for Tq, Tkv, batch, Hq, Hkv, D in ((4, 4, 1, 4, 0, 128), (4, 4, 0, 4, 2, 128), (4, 4, 1, 5, 2, 128), (-1, 4, 1, 4, 2, 128), (4, 4, 1, 4, 2, 64)):
        assert esp.esp_prefill_pool_workspace_bytes(Tq, Tkv, batch, Hq, Hkv, D) == esp.esp_prefill_workspace_bytes(Tq, Tkv, batch, Hq, Hkv, D) == 0
    assert esp.esp_prefill_pool_workspace_bytes(4, 5, 1, 4, 2, 128) == 256 + 2 * 5 * 2 * 256


def test_a_forced_plan_whose_launch_would_not_fit_is_refused(esp):
    one, nul = ctypes.c_void_p(256), ctypes.c_void_p(0)             # never dereferenced: refused before anything is launched
    Tq = 1 << 30
    assert esp.esp_debug_set_prefill_plan(-16) == 0
    try:
        st = esp.lib.esp_partial_attn_prefill(one, one, one, one, one, nul, nul, 1, Tq, 64, Tq, 64, 8, 1, 128, ctypes.c_float(0.1), 1, one, one,
                                              one, 1 << 62, nul)
        assert st == esp.ESP_ERR_UNSUPPORTED and "too many rows" in esp.last_error()
    finally:
        esp.esp_debug_set_prefill_plan(0)
