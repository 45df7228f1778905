"""The tuned kernels for chunks of 2^5 .. 2^13 coordinates against the CPU oracle: every chunk
size, worker counts around the edges of a workgroup (16 waves, several workgroups beyond),
odd and ragged sizes, one-pass and per-call forms, and the signed grid's centre rule."""
import numpy as np
import pytest
import torch

import paper_2407_01378_amd as thc
from oracle import thc as O
from oracle import thc_sat as S
from synth import to_numpy_bits

from gpu_util import DEV, check_against_oracle, run_path, run_path_fused, run_path_timed

pytestmark = pytest.mark.gpu


def _grads(W, n, dtype, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    xs = []
    for _ in range(W):
        x = torch.randn(n, generator=g, device=DEV) / torch.sqrt((torch.randn(3, n, generator=g, device=DEV) ** 2).mean(dim=0))
        x = x * torch.exp(torch.randn(n // 512 + 1, generator=g, device=DEV) * 3 - 6).repeat_interleave(512)[:n]
        x[n // 3:n // 3 + n // 8] = 0.0   # whole chunks of zeros among the small sizes
        xs.append(x.to(dtype))
    return xs


CASES = [  # (l, W, bits, n): a lone ragged chunk, edges of a wave's 2^11, several workgroups, regions
    (5, 8, 4, 33), (5, 3, 2, 40_001), (6, 1, 8, 70_000), (7, 16, 4, 10_243), (8, 17, 8, 5_001), (9, 2, 4, 131_072),
    (9, 33, 2, 6_145), (10, 4, 4, 100_003), (10, 8, 8, 2_047), (10, 64, 4, 4_099), (11, 1, 4, 200_001), (11, 5, 2, 40_961),
    (11, 18, 4, 8_191), (12, 8, 8, 60_001), (12, 3, 4, 4_097), (12, 9, 2, 12_289), (12, 1, 4, 300_001), (13, 4, 4, 90_003),
    (13, 8, 2, 40_000), (13, 5, 8, 8_193), (13, 2, 4, 7),
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("l,W,bits,n", CASES)
def test_small_chunks_match_the_oracle(l, W, bits, n, dtype):
    print(f"small l={l} W={W} bits={bits} n={n} {dtype}", flush=True)
    xs = _grads(W, n, dtype, 7 * l + W)
    fused = run_path_fused(xs, l, 5, bits)
    check_against_oracle(xs, fused, l, 5, bits)
    per_call = run_path(xs, l, 5, bits)
    check_against_oracle(xs, per_call, l, 5, bits)
    timed = run_path_timed(xs, l, 5, bits)
    assert torch.equal(timed["out"], fused["out"])
    own = torch.empty_like(fused["payloads"][0])   # the worker's own range as the grid
    scale = torch.empty_like(fused["scale"])
    thc.thc_encode(xs[W - 1], l, 5, W - 1, bits, None, own, scale)
    torch.cuda.synchronize()
    bf = dtype == torch.bfloat16
    y = O.rht_forward(to_numpy_bits(xs[W - 1]), l, 5, dtype=np.float32, bf16=bf)
    s = O.chunk_absmax(y, l)
    assert (scale.cpu().numpy() == s).all()
    assert (own.cpu().numpy() == O.pack(O.quantize(y, s, l, W - 1, 5, bits, dtype=np.float32), bits)).all()


@pytest.mark.parametrize("l,W,bits,dtype", [(5, 4, 4, torch.float32), (10, 8, 2, torch.bfloat16), (12, 9, 8, torch.bfloat16),
                                            (13, 3, 4, torch.float32)])
@pytest.mark.parametrize("magnitude", [1.0, 2.0 ** -118, 2.0 ** -112, 2.0 ** 104])
def test_small_chunks_outside_the_folded_range(l, W, bits, dtype, magnitude):
    n = 3 * (1 << l) + 77
    print(f"small folded l={l} W={W} bits={bits} {dtype} {magnitude}", flush=True)
    xs = [(x.float().clamp(-4, 4) * magnitude).to(dtype) for x in _grads(W, n, dtype, 3)]
    check_against_oracle(xs, run_path_fused(xs, l, 9, bits), l, 9, bits)


@pytest.mark.parametrize("l,W,bits", [(5, 2, 2), (11, 8, 4), (13, 7, 8)])
def test_small_chunks_on_the_signed_grid(l, W, bits):
    n = 2 * (1 << l) + 1001
    xs = _grads(W, n, torch.bfloat16, 11)
    xs = [torch.where(torch.arange(n, device=DEV) < (1 << l), torch.zeros_like(x), x) for x in xs]   # an empty chunk
    P = thc.thc_num_chunks(n, l)
    scale = torch.empty(P, device=DEV)
    pay = [torch.empty(thc.thc_payload_bytes(n, l, bits), dtype=torch.uint8, device=DEV) for _ in range(W)]
    ws = torch.empty(thc.thc_encode_all_workspace_bytes(W, n, l), dtype=torch.uint8, device=DEV)
    thc.thc_sat_encode_all(xs, l, 5, bits, pay, scale, ws)
    ref = [torch.empty_like(pay[0]) for _ in range(W)]
    for w in range(W):
        thc.thc_sat_encode(xs[w], l, 5, w, bits, scale, ref[w])
    torch.cuda.synchronize()
    want = S.sat_pipeline([to_numpy_bits(x) for x in xs], l, 5, bits, dtype=np.float32, bf16=True)
    for w in range(W):
        assert (pay[w].cpu().numpy() == want["payloads"][w]).all()
        assert torch.equal(ref[w], pay[w])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("l,W,bits,n", [(5, 3, 4, 20_001), (6, 1, 8, 33), (7, 8, 2, 40_961), (8, 2, 4, 16_384), (9, 17, 8, 5_001),
                                        (10, 4, 4, 100_003), (11, 5, 2, 2_047), (12, 8, 8, 12_289), (13, 2, 4, 70_000)])
def test_gradients_off_the_16_byte_grid_match_the_oracle(l, W, bits, n, dtype):
    """These take the generic kernels, one launch per step and worker (test_launch_shapes_host.py)."""
    print(f"unaligned l={l} W={W} bits={bits} n={n} {dtype}", flush=True)
    xs = [torch.empty(n + 1, dtype=dtype, device=DEV)[1:].copy_(x) for x in _grads(W, n, dtype, 5 * l + W)]
    assert all(x.data_ptr() % 16 for x in xs)
    check_against_oracle(xs, run_path(xs, l, 6, bits), l, 6, bits)
    fused = run_path_fused(xs, l, 6, bits)
    check_against_oracle(xs, fused, l, 6, bits)
    timed = run_path_timed(xs, l, 6, bits)
    assert torch.equal(timed["out"], fused["out"])
    mixed = [xs[0]] + [x.clone() for x in xs[1:]]   # one gradient off the grid is enough
    again = run_path_fused(mixed, l, 6, bits)
    assert all(torch.equal(a, b) for a, b in zip(again["payloads"], fused["payloads"]))
    own = torch.empty_like(fused["payloads"][0])    # the worker's own range as the grid
    scale = torch.empty_like(fused["scale"])
    thc.thc_encode(xs[0], l, 6, 0, bits, None, own, scale)
    torch.cuda.synchronize()
    bf = dtype == torch.bfloat16
    y = O.rht_forward(to_numpy_bits(xs[0]), l, 6, dtype=np.float32, bf16=bf)
    s = O.chunk_absmax(y, l)
    assert (scale.cpu().numpy() == s).all()
    assert (own.cpu().numpy() == O.pack(O.quantize(y, s, l, 0, 6, bits, dtype=np.float32), bits)).all()


def _one_pass(xs, l, bits, ws, cleared=True):
    W, n = len(xs), xs[0].numel()
    scale = torch.full((thc.thc_num_chunks(n, l),), float("nan"), device=DEV)
    pay = [torch.full((thc.thc_payload_bytes(n, l, bits),), 0xAA, dtype=torch.uint8, device=DEV) for _ in range(W)]
    (thc.thc_encode_all_cleared if cleared else thc.thc_encode_all)(xs, l, 5, bits, pay, scale, ws)
    return scale, pay


def _matches_the_per_worker_calls(xs, l, bits, scale, pay):
    W, P = len(xs), scale.numel()
    absmax, want, own = torch.empty(W * P, device=DEV), torch.empty_like(scale), torch.empty_like(pay[0])
    for w in range(W):
        thc.thc_chunk_absmax(xs[w], l, 5, absmax[w * P:(w + 1) * P])
    thc.thc_scale_reduce(absmax, W, P, want)
    assert torch.equal(want, scale)
    for w in range(W):
        thc.thc_encode(xs[w], l, 5, w, bits, want, own)
        assert torch.equal(own, pay[w]), w


SPREAD = [  # (l, W, bits, n): the fewest and the most workers of several workgroups, more items than the chip holds
    (5, 17, 4, 33), (5, 64, 2, 4_100), (5, 24, 8, 700_001), (8, 33, 4, 30_000), (10, 17, 2, 1_500_001), (11, 64, 4, 200_001),
    (12, 9, 8, 4_097), (12, 64, 4, 300_001), (13, 5, 4, 8_193), (13, 8, 8, 2_000_001), (13, 64, 2, 250_001), (13, 33, 4, 1),
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("l,W,bits,n", SPREAD)
def test_workers_spread_over_workgroups(l, W, bits, n, dtype):
    """Against the one-call-per-worker route, on a workspace that has to come back clear, twice; and on one in any state."""
    print(f"spread l={l} W={W} bits={bits} n={n} {dtype}", flush=True)
    xs = _grads(W, n, dtype, l + W)
    ws = torch.zeros(thc.thc_encode_all_workspace_bytes(W, n, l), dtype=torch.uint8, device=DEV)
    for cleared in (True, True, False):
        if not cleared:
            ws.fill_(0xFF)
        scale, pay = _one_pass(xs, l, bits, ws, cleared)
        torch.cuda.synchronize()
        assert not thc.thc_encode_all_timed_out(ws) and (not cleared or int(ws.count_nonzero()) == 0)
        _matches_the_per_worker_calls(xs, l, bits, scale, pay)


ROUNDS = [  # (l, W, bits, n): two to four rounds of workers, fewer and more items than CUs, a worker too few for the last round
    (5, 17, 4, 500_001), (5, 64, 2, 700_001), (5, 33, 8, 1_100_003), (6, 31, 4, 524_287), (7, 33, 8, 1_048_001), (8, 17, 2, 524_288),
    (9, 23, 4, 520_001), (10, 17, 8, 500_001), (11, 18, 4, 524_000), (12, 9, 2, 1_000_003), (12, 10, 8, 1 << 20), (12, 12, 4, 1_048_001),
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("l,W,bits,n", ROUNDS)
def test_workers_taken_in_rounds(l, W, bits, n, dtype):
    """Against the one-call-per-worker route, twice: no workspace is needed, a clear one stays clear, the error word of any
    other is cleared."""
    print(f"rounds l={l} W={W} bits={bits} n={n} {dtype}", flush=True)
    xs = _grads(W, n, dtype, l + W)
    ws = torch.zeros(thc.thc_encode_all_workspace_bytes(W, n, l), dtype=torch.uint8, device=DEV)
    for cleared in (True, False):
        if not cleared:
            ws.fill_(0xFF)
        scale, pay = _one_pass(xs, l, bits, ws, cleared)
        torch.cuda.synchronize()
        assert not thc.thc_encode_all_timed_out(ws) and (not cleared or int(ws.count_nonzero()) == 0)
        _matches_the_per_worker_calls(xs, l, bits, scale, pay)


@pytest.mark.parametrize("l,W,n", [(8, 24, 900_001), (13, 64, 250_001), (13, 64, 2_000_001)])
def test_expired_wait_of_spread_workers(l, W, n):
    """Failure handling forced from the host: with a poll limit of zero a wait gives up after one read.  Every wave still
    ends, the error word is set, and a cleared workspace is good again.  (In a launch of few rounds every word may be there
    at the first read: one of up to fifty launches has to report an expired wait.)"""
    print(f"expired wait l={l} W={W} n={n}", flush=True)
    xs = _grads(W, n, torch.bfloat16, l + W)
    ws = torch.zeros(thc.thc_encode_all_workspace_bytes(W, n, l), dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    try:
        thc.thc_set_spin_limit(0)
        for launch in range(50):
            thc.thc_workspace_clear(ws)
            _one_pass(xs, l, 4, ws)
            torch.cuda.synchronize()
            expired = thc.thc_encode_all_timed_out(ws)
            if expired:
                break
    finally:
        thc.thc_set_spin_limit(1 << 22)
    print(f"reported by launch {launch}", flush=True)
    assert expired
    thc.thc_workspace_clear(ws)
    scale, pay = _one_pass(xs, l, 4, ws)
    torch.cuda.synchronize()
    assert int(ws.count_nonzero()) == 0
    _matches_the_per_worker_calls(xs, l, 4, scale, pay)
