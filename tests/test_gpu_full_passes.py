"""The full rotation at the sizes where its plan of passes changes: the longest single pass (11
stages behind the chunk kernels, 16-float rows), its neighbours on both sides, and gradients that
fill only part of the blocks; odd lengths end inside a stored pair."""
import pytest
import torch

import paper_2407_01378_amd as thc

from test_gpu_full import _full_pipeline

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available()
    thc.lib()


@pytest.mark.parametrize("l,n,bits,dtype", [
    (20, (1 << 19) + 3, 4, torch.bfloat16),      # 6 stages: no LDS
    (21, (1 << 20) + 16_385, 8, torch.float32),  # 7: two waves
    (24, (1 << 23) + 777_777, 4, torch.float32),
    (25, (1 << 24) + 5, 4, torch.bfloat16),      # 11
    (25, 40_001, 2, torch.float32),              # 11, almost all padding
    (26, (1 << 25) + 99_999, 8, torch.float32),  # 6 + 6
])
def test_passes_around_the_longest_one(l, n, bits, dtype):
    _full_pipeline(l, n, 1, bits, dtype)
