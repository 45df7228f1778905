"""The full rotation of 2^25 coordinates, whose first pass covers chunks of 2^15 from a length of 9/16 on (and
of 2^26, with chunks of 2^14 and a pass more): the whole pipeline against the oracle on both sides of that length, with one- and two-byte
sums, and the rotated values against the stages one by one, so that a wrong unit of the exchange is
seen where the oracle would take too long."""
import pytest
import torch

import paper_2407_01378_amd as thc

from test_gpu_full import _full_pipeline
from test_gpu_full_passes import _stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bits,dtype", [
    (20_000_001, 4, torch.float32), ((9 << 21) + 1, 8, torch.bfloat16), (9 << 21, 2, torch.bfloat16),
])
def test_pipeline(n, bits, dtype):
    _full_pipeline(25, n, 2, bits, dtype)


@pytest.mark.parametrize("l,n,dtype", [
    (25, (1 << 25) - 1, torch.bfloat16), (26, (1 << 15) + 1, torch.float32), (26, 1, torch.bfloat16),
    (25, 1 << 25, torch.float32), (26, (1 << 26) - 3, torch.float32), (26, (1 << 25) + 32_767, torch.bfloat16),
])
def test_forward_and_inverse_match_the_stages_one_by_one(l, n, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(l + n % 97)
    x = torch.randn(n, generator=g, device="cuda").mul_(1e-3).to(dtype)
    factor = torch.tensor(2.0 ** (-l / 2), dtype=torch.float64).float().item()
    y = torch.full((1 << l,), float("nan"), device="cuda")
    thc.rht_forward_full(x, l, 7, y)
    P = thc.thc_num_chunks(n, 14)
    ref = torch.zeros(1 << l, device="cuda")
    thc.rht_forward(x, 14, 7, ref[:P << 14])
    ref[:P << 14] *= 128.0   # (exact: the chunks' own factor is a power of two)
    _stages(ref, 14, l)
    assert torch.equal(y, ref * factor)
    back = torch.full((n,), float("nan"), device="cuda")
    thc.rht_inverse_full(y.clone(), n, l, 7, back)
    # the inverse: all stages on the rotated values and the factor give the magnitudes bit for bit; the signs are
    # those of x (the round trip is off by at most some l * 2^-24 of the largest value)
    inv = _stages(y, 0, l)[:n] * factor
    assert torch.equal(back.abs(), inv.abs())
    assert torch.allclose(back, x.float(), rtol=0, atol=float(x.float().abs().max()) * 1e-5)


@pytest.mark.parametrize("rest", [1, 2, 255, 257, 1025, 1535, 1537, 1791, 1793, 2049])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_a_short_last_chunk_is_padded_with_zeros_whatever_lies_behind_it(rest, dtype):
    """Of the last chunk of 2^15 only `rest` coordinates exist; the memory behind them is the caller's and
    holds large values.  The bounds of its loads are those of the gradient for every run of a wave (2^9
    bf16 or 2^8 fp32 coordinates apart)."""
    l, n = 25, (600 << 15) + rest
    g = torch.Generator(device="cuda")
    g.manual_seed(rest)
    whole = torch.full((n + (1 << 15),), 1e6, device="cuda", dtype=dtype)
    x = whole[:n]
    x.copy_(torch.randn(n, generator=g, device="cuda"))
    y = torch.full((1 << l,), float("nan"), device="cuda")
    absmax = torch.empty(1, device="cuda")
    thc.rht_forward_full_absmax(x, l, 7, y, absmax)
    P = thc.thc_num_chunks(n, 14)
    ref = torch.zeros(1 << l, device="cuda")
    thc.rht_forward(x.clone(), 14, 7, ref[:P << 14])
    ref[:P << 14] *= 128.0   # (exact: the chunks' own factor is a power of two)
    _stages(ref, 14, l)
    ref *= torch.tensor(2.0 ** (-l / 2), dtype=torch.float64).float().item()
    assert torch.equal(y, ref)
    assert torch.equal(absmax[0], ref.abs().max())
