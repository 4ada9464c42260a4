"""Decode calls whose token list is as long as an int32 counts: what is looked ahead to lies past 2^31.  A request's tokens share a row of the
pool, but for the very last token of the list, which outweighs all others of its request."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


TOTAL = 2 ** 31 - 1


def check(cuda, plan, Hq, Hkv, at, longest):
    """Requests at[b] .. at[b + 1] - 1 of the list, none longer than `longest` by what the call is told."""
    from paper_2404_09526_amd import binding as esp
    torch.cuda.empty_cache()
    B = len(at) - 1
    print(f"[case] {TOTAL} tokens, {B} requests, {Hq}/{Hkv}, plan {plan}", flush=True)
    slots = torch.empty(TOTAL, dtype=torch.int32, device=cuda)
    for b in range(B):
        slots[at[b]:at[b + 1]] = b
    slots[-1] = B
    k_pool = torch.zeros((B + 1, Hkv, 128), dtype=torch.bfloat16, device=cuda)
    k_pool[B] = 30 / 128                                            # (exact in bf16)
    v_pool = (1 + torch.arange((B + 1) * Hkv * 128, device=cuda) % 2).to(torch.bfloat16).view(B + 1, Hkv, 128)   # sums of 1 and 2 are exact
    v_pool[B] = 64
    q = torch.ones((B, Hq, 128), dtype=torch.bfloat16, device=cuda)
    offsets = torch.tensor(at, dtype=torch.int64).to(torch.int32).to(cuda)
    before = esp.esp_debug_set_decode_plan(plan)
    try:
        O, LSE = esp.esp_partial_attn_decode(q, k_pool, v_pool, slots, offsets, longest, softmax_scale=1.0)
        torch.cuda.synchronize()
    finally:
        esp.esp_debug_set_decode_plan(before)
    lens = torch.tensor([b - a for a, b in zip(at, at[1:])], dtype=torch.float64)
    want = lens.log()
    want[-1] = math.log(math.exp(30) + float(lens[-1]) - 1)
    assert (LSE.view(B, Hq).double().cpu() - want.view(-1, 1)).abs().max() < 1e-4   # fp32 of 17 and of 30: 2e-6, sums of whole numbers
    assert torch.equal(O[:-1], v_pool[:B - 1].repeat_interleave(Hq // Hkv, 1))
    assert (O[-1] == 64).all()                                      # (the others of its request weigh 4e-6 in all)


@pytest.mark.parametrize("Hq,Hkv,B", [(4, 4, 50), (8, 4, 50), (32, 1, 200)])
@pytest.mark.parametrize("plan", [1, 2], ids=["ranges", "one-launch"])
def test_decode_of_a_token_list_of_int32_length(cuda, plan, Hq, Hkv, B):
    at = [TOTAL * b // B for b in range(B + 1)]
    check(cuda, plan, Hq, Hkv, at, max(b - a for a, b in zip(at, at[1:])))


@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (8, 4), (32, 1)])
def test_decode_of_parts_that_a_short_request_at_the_end_does_not_have(cuda, Hq, Hkv):
    """Six ranges of 2^22 tokens for each of 77 requests, by a length bound that says less than they have (the sixth takes the rest): those of the
    last request, of 99 tokens, would start past 2^31."""
    at = [(TOTAL - 99) * b // 76 for b in range(77)] + [TOTAL]
    check(cuda, 1, Hq, Hkv, at, 6 << 22)
