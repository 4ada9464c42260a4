"""Calls with more work-items than a launch counts in one dimension (2^32): every row of them is written.  Values are small whole numbers,
so the results are exact.  The largest takes 140 GiB."""
import pytest
import torch

pytestmark = pytest.mark.gpu
CHUNK = 1 << 18


@pytest.fixture(scope="module")
def esp(cuda):
    from paper_2404_09526_amd import binding
    return binding


@pytest.fixture(autouse=True)
def memory(cuda):
    torch.cuda.empty_cache()
    yield
    torch.cuda.empty_cache()


def value(first, last, cuda):
    """1 .. 251 by the row: whole numbers that bf16 holds."""
    return (torch.arange(first, last, device=cuda) % 251 + 1).view(-1, 1, 1)


def by_row(T, H, dtype, cuda):
    x = torch.empty((T, H, 128), dtype=dtype, device=cuda)
    for i in range(0, T, CHUNK):
        x[i:i + CHUNK] = value(i, min(i + CHUNK, T), cuda).to(dtype)
    return x


@pytest.mark.parametrize("dtype,T", [(torch.float32, (1 << 22) + 3), (torch.bfloat16, (1 << 23) + 3)], ids=["fp32", "bf16"])
def test_merge_of_more_pairs_than_a_grid_dimension_holds(esp, cuda, dtype, T):
    H = 32                                                          # 32 lanes a pair of fp32 partials, 16 of bf16: just above 2^32
    print(f"[case] merge {T} x {H} {dtype}", flush=True)
    x, lse = by_row(T, H, dtype, cuda), torch.zeros((T, H), device=cuda)
    O = torch.zeros((T, H, 128), dtype=torch.bfloat16, device=cuda)
    esp.esp_merge_partials([x, x], [lse, lse], O=O, want_lse=False)
    torch.cuda.synchronize()
    for i in range(0, T, CHUNK):
        n = min(i + CHUNK, T)
        assert (O[i:n] == value(i, n, cuda).to(torch.bfloat16)).all(), i


def test_append_and_gather_of_more_pieces_than_a_grid_dimension_holds(esp, cuda):
    H, T, S = 32, (1 << 23) + 3, 1024                               # 512 pieces of 16 bytes a row: just above 2^32
    print(f"[case] append, gather {T} x {H}", flush=True)
    k_pool = torch.zeros((S, H, 128), dtype=torch.bfloat16, device=cuda)
    v_pool = torch.zeros_like(k_pool)
    x = by_row(T, H, torch.bfloat16, cuda)
    kept = torch.cat([torch.arange(100), torch.arange(T // 2, T // 2 + 100), torch.arange(T - 100, T)]).to(cuda)
    slots = torch.full((T,), -1, dtype=torch.int32, device=cuda)
    slots[kept] = torch.arange(300, dtype=torch.int32, device=cuda) * 3
    esp.esp_kv_append(x, x, slots, k_pool, v_pool)
    torch.cuda.synchronize()
    want = torch.zeros_like(k_pool)
    want[slots[kept].long()] = x[kept]
    assert torch.equal(k_pool, want) and torch.equal(v_pool, want)
    del x

    k_pool.copy_(value(0, S, cuda).to(torch.bfloat16))
    v_pool.copy_(value(7, S + 7, cuda).to(torch.bfloat16))
    slots = (torch.arange(T, device=cuda) % S).to(torch.int32)
    k, v = esp.esp_kv_gather(k_pool, v_pool, slots)
    torch.cuda.synchronize()
    for i in range(0, T, CHUNK):
        s = slots[i:i + CHUNK].long()
        assert torch.equal(k[i:i + CHUNK], k_pool[s]) and torch.equal(v[i:i + CHUNK], v_pool[s]), i


def test_decode_of_more_pairs_than_a_grid_dimension_holds(esp, cuda):
    """A workgroup of the combination to each of 2^24 and more (request, head) pairs: one long request, the others of one token."""
    Hq, B, long, S = 32, (1 << 19) + 5, 600_000, 1024
    print(f"[case] decode {B} x {Hq}/1", flush=True)
    lens = torch.ones(B, dtype=torch.int64)
    lens[1] = long
    offsets = torch.cat([torch.zeros(1, dtype=torch.int64), lens.cumsum(0)]).to(torch.int32).to(cuda)
    rows = torch.arange(B, device=cuda) % S                         # a request's tokens are all in one row
    slots = rows.repeat_interleave(lens.to(cuda)).to(torch.int32)
    k_pool = torch.zeros((S, 1, 128), dtype=torch.bfloat16, device=cuda)
    v_pool = torch.empty_like(k_pool)
    v_pool.copy_(value(0, S, cuda).to(torch.bfloat16))
    q = torch.ones((B, Hq, 128), dtype=torch.bfloat16, device=cuda)
    before = esp.esp_debug_set_decode_plan(1)
    try:
        O, LSE = esp.esp_partial_attn_decode(q, k_pool, v_pool, slots, offsets, long, softmax_scale=1.0)
        torch.cuda.synchronize()
    finally:
        esp.esp_debug_set_decode_plan(before)
    assert (LSE.view(B, Hq) - lens.to(cuda).log().view(-1, 1)).abs().max() < 1e-4
    for i in range(0, B, CHUNK):
        assert (O[i:i + CHUNK] == v_pool[rows[i:i + CHUNK]]).all(), i
