"""Calls with more work-items than a launch counts in one dimension (2^32): every row of them is written.  Values are small whole numbers,
so the results are exact.  The largest takes 130 GiB."""
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
