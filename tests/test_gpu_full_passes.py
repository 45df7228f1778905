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


def _stages(y, first, last):
    """Stages first .. last - 1 on y in place, one separately rounded addition and subtraction each."""
    for s in range(first, last):
        v = y.view(-1, 2, 1 << s)
        d = v[:, 0] - v[:, 1]
        v[:, 0] += v[:, 1]
        v[:, 1] = d
    return y


@pytest.mark.parametrize("l,n,dtype", [
    (27, (1 << 26) + 12_345, torch.float32),     # 13 high stages: 6 + 7
    (28, (1 << 14) + 1, torch.bfloat16),         # 7 + 7, almost all padding
    (29, (1 << 28) + 77_777, torch.bfloat16),    # 8 + 7
    (31, (1 << 27) + 3, torch.float32),          # 9 + 8
])
def test_two_passes_match_the_stages_one_by_one(l, n, dtype):
    """Sizes beyond what the oracle takes in reasonable time, against the same stages in torch on the
    GPU, bit for bit; the stored, range-only and quantizing forms of the last pass, and the inverse."""
    print(f"two passes l={l} n={n} dtype={dtype}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(l)
    x = torch.randn(n, generator=g, device="cuda").mul_(1e-3).to(dtype)
    factor = torch.tensor(2.0 ** (-l / 2), dtype=torch.float64).float().item()
    y = torch.full((1 << l,), float("nan"), device="cuda")
    thc.rht_forward_full(x, l, 7, y)
    ref = torch.zeros(1 << l, device="cuda")
    thc.rht_forward(x, 14, 7, ref[:thc.thc_num_chunks(n, 14) << 14])
    ref[:thc.thc_num_chunks(n, 14) << 14] *= 128.0   # (exact: the chunks' own factor is a power of two)
    _stages(ref, 14, l).mul_(factor)
    assert torch.equal(y, ref)
    scale, ranged = torch.empty(1, device="cuda"), torch.empty(1, device="cuda")
    thc.thc_full_absmax(y, l, scale)
    assert float(scale) == float(torch.stack([ref.max(), -ref.min()]).max())
    stored, deferred = (torch.empty((1 << l) // 2, dtype=torch.uint8, device="cuda") for _ in range(2))
    thc.thc_full_encode(y, l, 7, 1, 4, scale, stored)
    thc.rht_forward_full_deferred(x, l, 7, y.fill_(float("nan")), ranged)
    thc.thc_full_encode_deferred(y, n, l, 7, 1, 4, scale, deferred)
    assert float(ranged) == float(scale) and torch.equal(stored, deferred)
    back = torch.full((n,), float("nan"), device="cuda")
    y.copy_(ref)
    thc.rht_inverse_full(y, n, l, 7, back)
    _stages(ref, 0, l).mul_(factor)
    assert torch.equal(back.abs(), ref[:n].abs())      # (the diagonal changes signs only, which the input has)
    assert float((back - x.float()).norm()) <= 1e-5 * float(x.float().norm())


@pytest.mark.parametrize("l,frac", [
    (17, 1.0), (18, 0.9), (20, 0.6),   # passes of 3 .. 6 stages: few workgroups, in order or in eighths
    (23, 0.8), (24, 0.8),              # 9 and 10 stages, one round of workgroups: eighths
    (25, 0.5), (25, 0.8),              # 11 stages: eighths; 10: runs of a payload line's worth
    (26, 0.51), (27, 0.51),            # 6 stages: eighths; 7: eighths at 2 bits, runs otherwise
])
def test_quantizing_pass_takes_every_tile_once_in_any_order(l, frac):
    """The deferred payload is that of the stored rotation, whatever order the tiles are dealt out in."""
    n = int(frac * (1 << l)) - 1
    g = torch.Generator(device="cuda")
    g.manual_seed(l)
    x = torch.randn(n, generator=g, device="cuda")
    y, work = torch.empty(1 << l, device="cuda"), torch.empty(1 << l, device="cuda")
    scale, ranged = torch.empty(1, device="cuda"), torch.empty(1, device="cuda")
    thc.rht_forward_full_absmax(x, l, 7, y, scale)
    thc.rht_forward_full_deferred(x, l, 7, work, ranged)
    assert float(ranged) == float(scale)
    for bits in (2, 4, 8):
        stored = torch.full(((bits << l) // 8,), 0xAA, dtype=torch.uint8, device="cuda")
        deferred = torch.full_like(stored, 0x55)
        thc.thc_full_encode(y, l, 7, 1, bits, scale, stored)
        thc.thc_full_encode_deferred(work, n, l, 7, 1, bits, scale, deferred)
        assert torch.equal(stored, deferred), bits
