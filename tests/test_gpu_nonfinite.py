"""Scores that are not finite, and partial results that mark "nothing" with a large negative number: a NaN key must show in O
and in LSE of every row that sees it, whichever way a call is cut into parts, and nowhere else."""
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


def nan_pattern(O, LSE, hit, what):
    """O and LSE are NaN throughout where `hit` [rows, heads] is set, and hold no NaN anywhere else."""
    O, LSE = np.isnan(O.float().cpu().numpy()), np.isnan(LSE.cpu().numpy())
    wrong = [np.argwhere(hit & ~O.all(2)).tolist(), np.argwhere(hit & ~LSE).tolist(), np.argwhere(~hit & (O.any(2) | LSE)).tolist()]
    assert not any(wrong), f"{what}, (row, head) pairs: finite O {wrong[0]}, LSE without NaN {wrong[1]}, NaN without a reason {wrong[2]}"


# ------------------------------------------------------------------ prefill whose keys are cut into parts
@pytest.mark.parametrize("out", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("at", [100, 2980])
@pytest.mark.parametrize("room", ["split", "whole"])
@pytest.mark.usefixtures("each_prefill_cut")
def test_prefill_nan_key_shows_however_the_keys_are_cut(esp, cuda, room, at, out):
    """40 tokens at the end of 3000: one NaN key that all rows see, in the first part, and one on the diagonal.  The dense
    call, the call that keeps rows and the one on pool rows; a workspace for the parts and one without room for them."""
    Tq, Tkv, Hq, Hkv = 40, 3000, 8, 2
    pc = wl.contiguous_prefill("nan-key", Tq, Tkv - Tq, [(0, Tkv)], Hq, Hkv, 50, cuda)
    s = pc.shards[0]
    s.k[at, 1] = float("nan")
    size = esp.esp_prefill_workspace_bytes(Tq, Tkv, 1, Hq, Hkv, 128)
    least = esp.esp_prefill_workspace_bytes(Tq, 0, 1, Hq, Hkv, 128)
    assert size > least                                                   # this call does split where it has the room
    ws = torch.empty(size if room == "split" else least, dtype=torch.uint8, device=cuda)
    q_pos = wl.host_i32(pc.q_pos)
    hit = (q_pos[:, None] >= at) & (np.arange(Hq) >= Hq // Hkv)[None, :]
    rows, heads = np.nonzero(~hit)
    Or, Lr = oracle.partial_attn(wl.bits(pc.q), wl.bits(s.k), wl.bits(s.v), q_pos, wl.host_i32(s.kv_pos), pc.scale, True,
                                 rows, heads, np.zeros(len(rows), np.int64), np.full(len(rows), Tkv, np.int64))
    slots = torch.randperm(Tkv, generator=torch.Generator(device=cuda).manual_seed(51), device=cuda).to(torch.int32)
    kp, vp = torch.zeros_like(s.k), torch.zeros_like(s.v)
    esp.esp_kv_append(s.k, s.v, slots, kp, vp)
    common = dict(softmax_scale=pc.scale, workspace=ws)
    for what, call in (
            ("dense", lambda o: esp.esp_partial_attn_prefill(pc.q, s.k, s.v, pc.q_pos, s.kv_pos, O=o, **common)),
            ("kept", lambda o: esp.esp_partial_attn_prefill_retain(pc.q, s.k, s.v, pc.q_pos, s.kv_pos, slots, torch.zeros_like(kp),
                                                                   torch.zeros_like(vp), O=o, **common)),
            ("pool", lambda o: esp.esp_partial_attn_prefill_pool_direct(pc.q, kp, vp, slots, pc.q_pos, s.kv_pos, O=o, **common))):
        print(f"[case] nan key at {at}, {room}, {what}, {out}", flush=True)
        O, LSE = call(torch.zeros(pc.q.shape, dtype=out, device=cuda))
        torch.cuda.synchronize()
        nan_pattern(O, LSE, hit, what)
        check_o_lse(O.float().cpu().numpy()[rows, heads], LSE.cpu().numpy()[rows, heads], Or, Lr, f"{what}, rows without the key")


@pytest.mark.usefixtures("each_prefill_cut")
def test_prefill_nan_query_row_in_a_split_call(esp, cuda):
    """Every part's result of such a row is NaN, and so is their combination."""
    pc = wl.contiguous_prefill("nan-query", 40, 2960, [(0, 3000)], 8, 2, 52, cuda)
    s = pc.shards[0]
    pc.q[7, 3] = float("nan")
    hit = np.zeros((40, 8), bool)
    hit[7, 3] = True
    O, LSE = esp.esp_partial_attn_prefill(pc.q, s.k, s.v, pc.q_pos, s.kv_pos, softmax_scale=pc.scale)
    torch.cuda.synchronize()
    nan_pattern(O, LSE, hit, "NaN query row")


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("P", [1, 3])
def test_merge_keeps_a_nan_partial(esp, cuda, P, dtype):
    """A NaN log-sum-exp beside finite ones, beside -inf ones, and in every partial."""
    g = torch.Generator(device=cuda).manual_seed(53)
    Os = [torch.randn((6, 4, 128), generator=g, device=cuda).to(dtype) for _ in range(P)]
    Ls = [torch.randn((6, 4), generator=g, device=cuda) for _ in range(P)]
    hit = np.zeros((6, 4), bool)
    Ls[0][1] = float("nan"); hit[1] = True
    for L in Ls:
        L[2] = float("nan"); L[4] = float("-inf")
    hit[2] = True
    for L in Ls[1:]:
        L[3] = float("-inf")
    Ls[0][3] = float("nan"); hit[3] = True
    O, LSE = esp.esp_merge_partials(Os, Ls)
    torch.cuda.synchronize()
    nan_pattern(O, LSE, hit, f"merge of {P}")
    assert torch.isneginf(LSE[4]).all() and (O[4] == 0).all()


# ------------------------------------------------------------------ decode
@pytest.mark.parametrize("peers", [0, 3])
@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (8, 8), (16, 16), (32, 32), (8, 4), (8, 2), (32, 8), (6, 3)])
def test_decode_nan_key_stays_with_its_request_and_head(esp, cuda, Hq, Hkv, peers):
    """One NaN key in one KV head of a request of one token, of one that fits a range and of one across several: that
    request's query heads are NaN, everything else is bit for bit what it is without the NaN."""
    lens = [1, 40, 0, 9000, 1, 700]
    dc = wl.decode_pool(f"decode-nan ({Hq}/{Hkv})", lens, 16384, Hq, Hkv, 54, cuda, n_new=0)
    off, slots = wl.host_i32(dc.seq_offsets), wl.host_i32(dc.slot_idx)

    def call():
        if peers:
            return esp.esp_partial_attn_decode_merge(dc.q, dc.k_pool, dc.v_pool, dc.slot_idx, dc.seq_offsets, max(lens),
                                                     list(dc.peer_O)[:peers], list(dc.peer_LSE)[:peers], softmax_scale=dc.scale)
        return esp.esp_partial_attn_decode(dc.q, dc.k_pool, dc.v_pool, dc.slot_idx, dc.seq_offsets, max(lens), softmax_scale=dc.scale)

    O0, L0 = call()
    hit = np.zeros((len(lens), Hq), bool)
    G = Hq // Hkv
    for r, t, h in ((0, 0, 0), (1, 17, 1), (3, 4321, Hkv - 1)):
        dc.k_pool[int(slots[off[r] + t]), h] = float("nan")
        hit[r, h * G:(h + 1) * G] = True
    O, LSE = call()
    torch.cuda.synchronize()
    nan_pattern(O, LSE, hit, dc.name)
    keep = torch.from_numpy(~hit).to(cuda)
    assert torch.equal(O[keep].view(torch.int16), O0[keep].view(torch.int16)) and torch.equal(LSE[keep].view(torch.int32), L0[keep].view(torch.int32))


@pytest.mark.parametrize("nothing", [-1e30, float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("longest", [60, 30000])
@pytest.mark.parametrize("Hq,Hkv,n_peers", [(8, 8, 2), (8, 2, 15), (32, 32, 9)])
def test_decode_peers_that_mark_nothing_with_a_finite_number(esp, cuda, Hq, Hkv, n_peers, longest, nothing):
    """Peers whose LSE is the lowest there is, finite, and whose O was never written: weight 0, whichever peers they are,
    with and without tokens of the request on this instance, whether a pair is combined by a wavefront or a workgroup."""
    lens = [longest, 0, 1, 700]
    dc = wl.decode_pool(f"decode-nothing ({Hq}/{Hkv})", lens, 32768, Hq, Hkv, 55, cuda, n_new=0, n_peers=n_peers)
    kp, vp = wl.bits(dc.k_pool), wl.bits(dc.v_pool)
    marked = np.random.default_rng(56).random((n_peers, len(lens))) < 0.6
    marked[0, 1], marked[1, 1] = False, True                              # request 1: one peer that holds something, one that does not
    marked[:, 3] = True                                                   # request 3: this instance alone
    for p in range(n_peers):
        m = torch.from_numpy(marked[p]).to(cuda)
        dc.peer_LSE[p][m] = nothing
        dc.peer_O[p][m] = float("nan")
    O, LSE = esp.esp_partial_attn_decode_merge(dc.q, dc.k_pool, dc.v_pool, dc.slot_idx, dc.seq_offsets, max(lens),
                                               list(dc.peer_O), list(dc.peer_LSE), softmax_scale=dc.scale)
    torch.cuda.synchronize()
    Or, Lr = oracle.partial_attn_decode_all(wl.bits(dc.q), kp, vp, wl.host_i32(dc.slot_idx), wl.host_i32(dc.seq_offsets), dc.scale)
    Op = np.stack([Or] + [np.nan_to_num(oracle.bf16_bits_to_f64(wl.bits(t)), nan=0.0) for t in dc.peer_O])
    Lp = np.stack([Lr] + [np.where(marked[p][:, None], -np.inf, dc.peer_LSE[p].cpu().numpy().astype(np.float64)) for p in range(n_peers)])
    Oref, Lref = oracle.merge_partials(Op, Lp)
    check_o_lse(O.float().cpu().numpy().reshape(-1, dc.D), LSE.cpu().numpy().reshape(-1), Oref.reshape(-1, dc.D), Lref.reshape(-1), dc.name)
