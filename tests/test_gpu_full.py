"""GPU parity at the benchmark's full sizes (configs 2-5), in the launch configuration bench.py times.
The oracle cannot evaluate these in full, so it computes a seeded sample of outputs one by one:
(request, head, row) triples for prefill (all heads, chunk and tile edges, rows with an empty visible set,
random rows), whole requests for decode.  Per-shard partials and the merged result are both checked."""
import numpy as np
import pytest
import torch

import oracle
from esp_checks import check_o_lse
from paper_2404_09526_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def esp(cuda):
    from paper_2404_09526_amd import binding
    return binding


def say(msg):
    print(f"[case] {msg}", flush=True)


def check_prefill_sampled(esp, pc, n_total, seed):
    """The launch configuration bench.py times: one shard -> bf16 output; several shards -> fp32 partials, merged once."""
    rows, heads, reqs = wl.prefill_parity_samples(pc, n_total, seed)
    assert set(heads.tolist()) == set(range(pc.Hq))
    qb, qp = wl.bits(pc.q), wl.host_i32(pc.q_pos)
    single = pc.batch == 1
    several = len(pc.shards) > 1
    ri, hi = torch.from_numpy(rows).to(pc.q.device), torch.from_numpy(heads).to(pc.q.device)
    parts, refs = [], []
    for si, s in enumerate(pc.shards):
        say(f"{pc.name} shard {si}: Tq={pc.Tq} Tkv={s.k.shape[0]} Hq={pc.Hq} Hkv={pc.Hkv} batch={pc.batch} samples={len(rows)}")
        # outputs start as NaN, so that the no-NaN check below also proves every row was written by this launch
        O = torch.full(pc.q.shape, float("nan"), dtype=torch.float32 if several else torch.bfloat16, device=pc.q.device)
        LSE = torch.full((pc.Tq, pc.Hq), float("nan"), dtype=torch.float32, device=pc.q.device)
        esp.esp_partial_attn_prefill(pc.q, s.k, s.v, pc.q_pos, s.kv_pos,
                                     None if single else pc.cu_q, None if single else s.cu_kv,
                                     None if single else pc.max_q, None if single else s.max_kv,
                                     softmax_scale=pc.scale, causal=pc.causal, O=O, LSE=LSE)
        torch.cuda.synchronize()
        cu_kv = wl.host_i32(s.cu_kv)
        Or, Lr = oracle.partial_attn(qb, wl.bits(s.k), wl.bits(s.v), qp, wl.host_i32(s.kv_pos), pc.scale, pc.causal,
                                     rows, heads, cu_kv[reqs], cu_kv[reqs + 1])
        st = check_o_lse(O[ri, hi].float().cpu().numpy(), LSE[ri, hi].cpu().numpy(), Or, Lr, f"{pc.name} shard {si}")
        say(f"  ok: {st}; rows with an empty visible set among the samples: {int(np.isneginf(Lr).sum())}")
        # properties that hold at any size: no NaN anywhere, LSE finite or -inf
        assert not torch.isnan(O).any() and not torch.isnan(LSE).any()
        if several and si == len(pc.shards) - 1:
            # the bf16 output of the same call at this size: the fp32 one rounded, bit for bit
            Ob = torch.full_like(pc.q, float("nan")); Lb = torch.full_like(LSE, float("nan"))
            esp.esp_partial_attn_prefill(pc.q, s.k, s.v, pc.q_pos, s.kv_pos, None if single else pc.cu_q, None if single else s.cu_kv,
                                         None if single else pc.max_q, None if single else s.max_kv, softmax_scale=pc.scale,
                                         causal=pc.causal, O=Ob, LSE=Lb)
            torch.cuda.synchronize()
            assert torch.equal(Ob.view(torch.int16), O.to(torch.bfloat16).view(torch.int16)) and torch.equal(Lb.view(torch.int32), LSE.view(torch.int32))
            del Ob, Lb
        parts.append((O, LSE)); refs.append((Or, Lr))
    if several:
        Om, Lm = esp.esp_merge_partials([p[0] for p in parts], [p[1] for p in parts])
        torch.cuda.synchronize()
        Oref, Lref = oracle.merge_partials(np.stack([r[0] for r in refs]), np.stack([r[1] for r in refs]))
        st = check_o_lse(Om[ri, hi].float().cpu().numpy(), Lm[ri, hi].cpu().numpy(), Oref, Lref, f"{pc.name} merged")
        say(f"  merged ok: {st}")
        # causal striped layout with r_q = 0: every row sees at least its own token in shard 0
        assert torch.isfinite(Lm).all() and not torch.isnan(Om.float()).any()


def test_config2_prefill_striped_4_shards(esp, cuda):
    pc = wl.config2_prefill(cuda)
    assert pc.visible_pairs_per_head == 2 * 8192 * 8192 - 8192
    check_prefill_sampled(esp, pc, *wl.PARITY_SAMPLES[pc.name])


def test_config2_prefill_with_retention(esp, cuda):
    """Config 2's shards 0 and 3 through esp_partial_attn_prefill_retain, every row kept at a random slot of a pool with
    room for twice as many: the pool rows against the oracle's scatter (every kept row, bit for bit, plus the sum of
    all 16-bit patterns of the pool: nothing else was touched), O and LSE against the oracle on the parity samples."""
    pc = wl.config2_prefill(cuda)
    rows, heads, reqs = wl.prefill_parity_samples(pc, *wl.PARITY_SAMPLES[pc.name])
    ri, hi = torch.from_numpy(rows).to(cuda), torch.from_numpy(heads).to(cuda)
    rng = np.random.default_rng(5)
    S = 2 * 8192
    for si in (0, 3):
        s = pc.shards[si]
        slots = rng.permutation(S)[:8192].astype(np.int32)
        slots[rng.random(8192) > 0.9] = -1
        kp = torch.zeros((S, pc.Hkv, pc.D), dtype=torch.bfloat16, device=cuda); vp = torch.zeros_like(kp)
        O = torch.full(pc.q.shape, float("nan"), dtype=torch.float32, device=cuda)
        LSE = torch.full((pc.Tq, pc.Hq), float("nan"), dtype=torch.float32, device=cuda)
        say(f"{pc.name} shard {si} with retention: kept {int((slots >= 0).sum())} of 8192 rows, pool {S} slots")
        esp.esp_partial_attn_prefill_retain(pc.q, s.k, s.v, pc.q_pos, s.kv_pos, torch.from_numpy(slots).to(cuda), kp, vp,
                                            softmax_scale=pc.scale, causal=True, O=O, LSE=LSE)
        torch.cuda.synchronize()
        kh = np.zeros((S, pc.Hkv, pc.D), np.uint16); vh = np.zeros_like(kh)
        oracle.kv_append(wl.bits(s.k), wl.bits(s.v), slots, kh, vh)
        assert np.array_equal(wl.bits(kp), kh) and np.array_equal(wl.bits(vp), vh)
        Or, Lr = oracle.partial_attn(wl.bits(pc.q), wl.bits(s.k), wl.bits(s.v), wl.host_i32(pc.q_pos), wl.host_i32(s.kv_pos), pc.scale,
                                     True, rows, heads)
        check_o_lse(O[ri, hi].cpu().numpy(), LSE[ri, hi].cpu().numpy(), Or, Lr, f"{pc.name} shard {si} (retain)")
        assert not torch.isnan(O).any() and not torch.isnan(LSE).any()


def test_config4_prefill_long_context(esp, cuda):
    pc = wl.config4_prefill(cuda)
    assert pc.visible_pairs_per_head == 32768 * 262144
    check_prefill_sampled(esp, pc, *wl.PARITY_SAMPLES[pc.name])


@pytest.mark.parametrize("ticks", [None, 0])
def test_chunk_against_a_long_prefix_with_round_start_waits(esp, cuda, ticks):
    """A 4096-token chunk against 32768 earlier tokens: long, alike items, so the workgroups that share a KV head wait
    for each other at the start of every dealt round.  Run as is, and with the longest wait set to nothing, so that
    every wait gives up at once (what a missing workgroup causes): the results must not depend on it."""
    was = esp.esp_debug_set_prefill_sync_ticks(ticks) if ticks is not None else None
    try:
        pc = wl.contiguous_prefill("chunk-vs-prefix", 4096, 32768 - 4096, [(0, 32768)], 32, 32, 33, cuda)
        check_prefill_sampled(esp, pc, 256, 7)
    finally:
        if was is not None:
            esp.esp_debug_set_prefill_sync_ticks(was)


def test_round_start_waits_replayed_from_a_graph(esp, cuda):
    """The same shape recorded into a graph: replays carry the recorded launch's tag, so the arrival counts of the
    round-start waits must have been cleared by the launch before (the arrival that completes a count clears it).
    Replays alternate with eager calls on the same workspace; every result must equal the eager one bit for bit."""
    pc = wl.contiguous_prefill("chunk-vs-prefix-graph", 4096, 32768 - 4096, [(0, 32768)], 32, 32, 34, cuda)
    s = pc.shards[0]
    ws = torch.zeros(esp.esp_prefill_workspace_bytes(pc.Tq, 32768, 1, 32, 32, 128), dtype=torch.uint8, device=cuda)
    run = lambda O, L: esp.esp_partial_attn_prefill(pc.q, s.k, s.v, pc.q_pos, s.kv_pos, softmax_scale=pc.scale, O=O, LSE=L, workspace=ws)
    O_ref = torch.empty_like(pc.q); L_ref = torch.empty((pc.Tq, pc.Hq), dtype=torch.float32, device=cuda)
    run(O_ref, L_ref)
    torch.cuda.synchronize()
    O_g, L_g = torch.empty_like(O_ref), torch.empty_like(L_ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run(O_g, L_g)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run(O_g, L_g)
    for rep in range(4):
        say(f"graph replay {rep}")
        O_g.copy_(torch.full_like(O_g, float("nan"))); L_g.copy_(torch.full_like(L_g, float("nan")))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(O_g.view(torch.int16), O_ref.view(torch.int16)) and torch.equal(L_g.view(torch.int32), L_ref.view(torch.int32)), rep
        if rep % 2 == 0:
            O_e, L_e = torch.empty_like(O_ref), torch.empty_like(L_ref)
            run(O_e, L_e)
            torch.cuda.synchronize()
            assert torch.equal(O_e.view(torch.int16), O_ref.view(torch.int16))
    # the counts are clear again: nothing of this launch's tag is left behind the pool counter
    words = ws.view(torch.int64)
    assert int((words[2:2 + 2 * 32] != 0).sum()) == 0


@pytest.mark.parametrize("ticks,Tq,Tkv", [(None, 4096, 32768), (0, 4096, 32768), (None, 4500, 36864), (0, 4500, 36864)])
def test_round_start_waits_and_an_item_pool(esp, cuda, main_prefill_kernel, ticks, Tq, Tkv):
    """Eight rounds of alike items, or eight and 26 of 32 (4096 or 4500 tokens, 16 query heads to each of eight KV heads): seven are dealt and start
    together, the others are drawn from the pool.  Against the oracle; bit for bit the two halves of the chunk, which have no pool; and replayed from
    a graph between eager calls, which the pool's counter and the arrival counts must survive."""
    was = esp.esp_debug_set_prefill_sync_ticks(ticks) if ticks is not None else None
    try:
        pc = wl.contiguous_prefill("chunk-and-pool", Tq, Tkv - Tq, [(0, Tkv)], 128, 8, 35, cuda)
        check_prefill_sampled(esp, pc, 256, 5)
        s = pc.shards[0]
        ws = torch.zeros(esp.esp_prefill_workspace_bytes(pc.Tq, Tkv, 1, 128, 8, 128), dtype=torch.uint8, device=cuda)
        run = lambda q, pos, O, L: esp.esp_partial_attn_prefill(q, s.k, s.v, pos, s.kv_pos, softmax_scale=pc.scale, O=O, LSE=L, workspace=ws)
        O_ref = torch.empty_like(pc.q); L_ref = torch.empty((pc.Tq, pc.Hq), dtype=torch.float32, device=cuda)
        for half in (slice(0, 2048), slice(2048, Tq)):             # (whole query tiles of 16 tokens)
            run(pc.q[half], pc.q_pos[half], O_ref[half], L_ref[half])
        O, L = torch.empty_like(O_ref), torch.empty_like(L_ref)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            run(pc.q, pc.q_pos, O, L)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            run(pc.q, pc.q_pos, O, L)
        for rep in range(4):
            O.fill_(float("nan")); L.fill_(float("nan"))
            g.replay() if rep % 2 == 0 else run(pc.q, pc.q_pos, O, L)
            torch.cuda.synchronize()
            assert torch.equal(O.view(torch.int16), O_ref.view(torch.int16)) and torch.equal(L.view(torch.int32), L_ref.view(torch.int32)), rep
            assert int((ws[:256].view(torch.int64) != 0).sum()) == 0
    finally:
        if was is not None:
            esp.esp_debug_set_prefill_sync_ticks(was)


def test_config5_prefill_varlen_gqa(esp, cuda):
    pc = wl.config5_prefill(cuda)
    assert pc.visible_pairs_per_head == 2994661376
    check_prefill_sampled(esp, pc, *wl.PARITY_SAMPLES[pc.name])


def check_decode_sampled(esp, dc, sample, heads_per_req=None):
    say(f"{dc.name}: B={dc.B} total={dc.total_tokens} max={int(dc.lens.max())} Hq={dc.Hq} Hkv={dc.Hkv} S={dc.num_slots} requests checked={len(sample)}")
    slots, off = wl.host_i32(dc.slot_idx), wl.host_i32(dc.seq_offsets)
    assert len(np.unique(slots)) == len(slots)                      # unique, non-contiguous slots
    kp = np.zeros((dc.num_slots, dc.Hkv, dc.D), np.uint16); vp = np.zeros_like(kp)   # lazily paged host image
    for b in sample:
        kr, vr = dc.host_rows[b]
        oracle.kv_append(kr, vr, slots[off[b]:off[b + 1]], kp, vp)
    O, LSE = esp.esp_partial_attn_decode(dc.q, dc.k_pool, dc.v_pool, dc.slot_idx, dc.seq_offsets, int(dc.lens.max()),
                                         softmax_scale=dc.scale)
    torch.cuda.synchronize()
    hs_all = np.arange(dc.Hq, dtype=np.int64) if heads_per_req is None else heads_per_req
    reqs = np.repeat(np.asarray(sample, np.int64), len(hs_all)); hs = np.tile(hs_all, len(sample))
    Or, Lr = oracle.partial_attn_decode(wl.bits(dc.q), kp, vp, slots, off, dc.scale, reqs, hs)
    st = check_o_lse(O.float().cpu().numpy()[reqs, hs], LSE.cpu().numpy()[reqs, hs], Or, Lr, dc.name)
    say(f"  ok: {st}")
    assert torch.isfinite(LSE).all() and not torch.isnan(O.float()).any()
    # merge with the 3 synthetic peer partials (kernel test on the arrays the GPU merged)
    Om, Lm = esp.esp_merge_partials([O] + list(dc.peer_O), [LSE] + list(dc.peer_LSE))
    torch.cuda.synchronize()
    Op = np.stack([oracle.bf16_bits_to_f64(wl.bits(t)) for t in [O] + list(dc.peer_O)])
    Lp = np.stack([t.cpu().numpy().astype(np.float64) for t in [LSE] + list(dc.peer_LSE)])
    Oref, Lref = oracle.merge_partials(Op, Lp)
    check_o_lse(Om.float().cpu().numpy().reshape(-1, dc.D), Lm.cpu().numpy().reshape(-1), Oref.reshape(-1, dc.D),
                Lref.reshape(-1), f"{dc.name} merge")
    # the same step as one call (what the benchmark times): the oracle's OWN local partials, never rounded, with the peers
    Of, Lf = esp.esp_partial_attn_decode_merge(dc.q, dc.k_pool, dc.v_pool, dc.slot_idx, dc.seq_offsets, int(dc.lens.max()),
                                               list(dc.peer_O), list(dc.peer_LSE), softmax_scale=dc.scale)
    torch.cuda.synchronize()
    Op = np.stack([Or] + [oracle.bf16_bits_to_f64(wl.bits(t))[reqs, hs] for t in dc.peer_O])
    Lp = np.stack([Lr] + [t.cpu().numpy().astype(np.float64)[reqs, hs] for t in dc.peer_LSE])
    Oref, Lref = oracle.merge_partials(Op, Lp)
    check_o_lse(Of.float().cpu().numpy()[reqs, hs], Lf.cpu().numpy()[reqs, hs], Oref, Lref, f"{dc.name} decode + merge in one call")
    # append to random free slots: appended rows + 4096 random untouched rows on the host, whole-pool checksum on device
    new_slots = wl.host_i32(dc.new_slots)
    rng = np.random.default_rng(7)
    probe = np.setdiff1d(rng.integers(0, dc.num_slots, 4096), new_slots)
    pi = torch.from_numpy(probe).to(dc.k_pool.device)
    before_k, before_v = wl.bits(dc.k_pool[pi]), wl.bits(dc.v_pool[pi])
    sum_before = [int(p.view(torch.int16).sum(dtype=torch.int64).item()) for p in (dc.k_pool, dc.v_pool)]
    esp.esp_kv_append(dc.new_k, dc.new_v, dc.new_slots, dc.k_pool, dc.v_pool)
    torch.cuda.synchronize()
    ni = torch.from_numpy(new_slots.astype(np.int64)).to(dc.k_pool.device)
    assert np.array_equal(wl.bits(dc.k_pool[ni]), wl.bits(dc.new_k)) and np.array_equal(wl.bits(dc.v_pool[ni]), wl.bits(dc.new_v))
    assert np.array_equal(wl.bits(dc.k_pool[pi]), before_k) and np.array_equal(wl.bits(dc.v_pool[pi]), before_v)
    added = [int(t.view(torch.int16).sum(dtype=torch.int64).item()) for t in (dc.new_k, dc.new_v)]
    sum_after = [int(p.view(torch.int16).sum(dtype=torch.int64).item()) for p in (dc.k_pool, dc.v_pool)]
    assert sum_after[0] == sum_before[0] + added[0] and sum_after[1] == sum_before[1] + added[1]   # free slots were zero


def test_config3_decode_pool_4M_slots(esp, cuda):
    """Every request, every head."""
    dc = wl.config3_decode(cuda)
    assert dc.Hkv * dc.D * 2 * 2 == 16384                           # bytes per resident token (K and V rows)
    check_decode_sampled(esp, dc, list(range(dc.B)))


def test_config5_decode_pool_16M_slots_gqa(esp, cuda):
    """Every request, nine query heads that cover all eight KV heads."""
    dc = wl.config5_decode(cuda)
    check_decode_sampled(esp, dc, list(range(dc.B)), heads_per_req=np.array([0, 5, 10, 15, 17, 22, 27, 28, 31], np.int64))

