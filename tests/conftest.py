import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


# Which of the two prefill kernels a call runs on, and whether its keys are cut, follows from its sizes: tests of small calls that are
# about a kernel, or about both, say so.  (1, 3: the main kernel, uncut and in three parts; -1, -3: the one for few rows.)
def on_plan(plan):
    from paper_2404_09526_amd import binding
    before = binding.esp_debug_set_prefill_plan(plan)
    assert binding.esp_debug_prefill_plan(40, 3000, 1, 40, 3000, 8, 2) == plan
    yield plan
    assert binding.esp_debug_set_prefill_plan(before) == plan


@pytest.fixture(params=[1, 3, -1, -3], ids=["main", "main-cut", "short", "short-cut"])
def each_prefill_plan(request, cuda):
    yield from on_plan(request.param)


@pytest.fixture(params=[3, -3], ids=["main-cut", "short-cut"])
def each_prefill_cut(request, cuda):
    yield from on_plan(request.param)


@pytest.fixture
def main_prefill_kernel(cuda):
    yield from on_plan(1)


# The same of decode: in ranges and a combination (1), or in one launch (2).  What the decode tests claim, they claim of both.
@pytest.fixture
def decode_plan(request, cuda):
    from paper_2404_09526_amd import binding
    before = binding.esp_debug_set_decode_plan(request.param)
    assert binding.esp_debug_decode_plan(4, 4000, 1000, 8, 2) == request.param
    yield request.param
    assert binding.esp_debug_set_decode_plan(before) == request.param


def pytest_generate_tests(metafunc):
    if metafunc.module.__name__ in ("test_gpu_small", "test_gpu_nonfinite") and metafunc.definition.name.startswith("test_decode_"):
        metafunc.fixturenames.append("decode_plan")
        metafunc.parametrize("decode_plan", [1, 2], ids=["ranges", "one-launch"], indirect=True)
