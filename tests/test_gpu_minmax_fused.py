"""One-pass forms of the min/max-range variant (thc_encode_all_minmax,
thc_aggregate_decode_minmax) on the GPU: shared ranges and payloads bit-identical to the
oracle and to the one-call-per-step entry points; fp32 output bit-identical to the fp32
canonical order and within 1e-5 relative L2 of the float64 definition; error paths."""
import numpy as np
import pytest
import torch

import paper_2407_01378_amd as thc
from oracle import thc as O
from oracle import thc_minmax as M
from synth import to_numpy_bits

from gpu_util import DEV
from test_gpu_minmax import _rand, run_minmax

pytestmark = pytest.mark.gpu
L14 = 14


def run_fused(xs, seed, bits, rotate, fill=0x5A):
    W, n = len(xs), xs[0].numel()
    P = thc.thc_num_chunks(n, L14)
    rng = torch.full((P * 2,), float("nan"), device=DEV)
    nb = thc.thc_payload_bytes(n, L14, bits)
    payloads = [torch.full((nb,), 0xAA, dtype=torch.uint8, device=DEV) for _ in range(W)]
    out = torch.full((n,), float("nan"), device=DEV)
    ws = torch.full((thc.thc_encode_all_minmax_workspace_bytes(W, n, L14),), fill, dtype=torch.uint8, device=DEV)
    thc.thc_encode_all_minmax(xs, L14, seed, bits, rotate, payloads, rng, ws)
    thc.thc_aggregate_decode_minmax(payloads, rng, n, L14, seed, bits, rotate, out)
    torch.cuda.synchronize()
    assert not thc.thc_encode_all_timed_out(ws)
    # the workspace comes back clear: header, range words and arrival counters
    assert int(ws.view(torch.int32).abs().max().item()) == 0
    return dict(range=rng.view(P, 2), payloads=payloads, out=out)


@pytest.mark.parametrize("bits,W,dtype,n,rotate", [
    (4, 8, torch.bfloat16, (5 << 14) + 8193, True),
    (4, 8, torch.bfloat16, (5 << 14) + 8193, False),
    (4, 3, torch.float32, (3 << 14) + 5, True),
    (4, 3, torch.float32, (3 << 14) + 5, False),
    (2, 17, torch.bfloat16, (2 << 14) + 77, True),        # odd bf16 count, more workers than a wave has bytes
    (2, 17, torch.bfloat16, (2 << 14) + 77, False),
    (8, 2, torch.bfloat16, (2 << 14) + 100, True),
    (8, 5, torch.float32, 1 << 14, False),
    (4, 1, torch.float32, 40, True),                      # one worker, one ragged chunk
    (4, 64, torch.bfloat16, (1 << 14) + 2, False),        # the largest worker count
    (4, 20, torch.bfloat16, (2 << 14) + 2, True),         # sums of 20 workers need 16-bit accumulators
    (4, 8, torch.bfloat16, 700 << 14, True),              # more chunks than resident workgroups: several rounds
    (4, 8, torch.bfloat16, (700 << 14) + 3, False),
    # even bf16 counts without rotation take the pipelined kernel: one item per workgroup,
    # one or two, two or three, and about eleven
    (4, 8, torch.bfloat16, (5 << 14) + 8194, False),
    (4, 8, torch.bfloat16, (100 << 14) + 2, False),
    (2, 8, torch.bfloat16, (150 << 14) + 6, False),
    (8, 2, torch.bfloat16, (300 << 14) + 10, False),
    (4, 8, torch.bfloat16, (700 << 14) + 4, False),
])
def test_one_pass_minmax_matches_the_oracle_and_the_per_step_calls(bits, W, dtype, n, rotate):
    print(f"minmax one-pass bits={bits} W={W} dtype={dtype} n={n} rotate={rotate}", flush=True)
    xs = [_rand(n, dtype, 31 * bits + w, scale=10.0 ** (-2 - (w % 3)), shift=3e-3) for w in range(W)]
    got = run_fused(xs, 23, bits, rotate)
    # the per-step entry points on the same inputs
    if thc.thc_sum_bytes(W, bits):
        ref_gpu = run_minmax(xs, L14, 23, bits, rotate, torch.float32)
        assert torch.equal(got["range"], ref_gpu["range"]), "shared ranges differ from the per-step calls"
        for w in range(W):
            assert torch.equal(got["payloads"][w], ref_gpu["payloads"][w]), f"payload {w} differs from thc_encode_minmax"
        assert torch.equal(got["out"], ref_gpu["out"]), "output differs from thc_decode_minmax"
    if n > (9 << 14):
        return   # the big shapes are covered by the comparison above and by sampled chunks below
    ref = M.pipeline_minmax([to_numpy_bits(x) for x in xs], L14, 23, bits, rotate=rotate, dtype=np.float32,
                            bf16=dtype == torch.bfloat16, out_bf16=False)
    assert (got["range"].cpu().numpy() == ref["range"]).all(), "shared ranges differ"
    for w in range(W):
        same = got["payloads"][w].cpu().numpy() == ref["payloads"][w]
        assert same.all(), f"payload {w} differs at bytes {np.flatnonzero(~same)[:8]}"
    out = got["out"].cpu().numpy()
    assert (out == ref["out"]).all(), "output differs from the fp32 canonical order"
    d64 = M.decode_minmax(ref["sums"], ref["range"].astype(np.float64), W, n, L14, 23, bits, rotate)
    assert np.linalg.norm(out - d64) <= 1e-5 * np.linalg.norm(d64)


@pytest.mark.parametrize("rotate", [True, False])
def test_one_pass_minmax_sampled_chunks_of_a_large_gradient(rotate):
    """700 chunks per worker (several rounds of the persistent grid): the first, the last
    (ragged) and a few chunks in between against the oracle run on those chunks alone."""
    bits, W, l = 4, 8, L14
    n = (700 << l) + 1234
    xs = [_rand(n, torch.bfloat16, 900 + w, scale=10.0 ** (-1 - (w % 4)), shift=-2e-3) for w in range(W)]
    got = run_fused(xs, 5, bits, rotate)
    P = thc.thc_num_chunks(n, l)
    per = (1 << l) * bits // 8
    for p in (0, 1, 255, 256, 511, 512, 513, 698, 699, P - 1):
        g0, g1 = p << l, min(n, (p + 1) << l)
        ref = M.pipeline_minmax([to_numpy_bits(x[g0:g1]) for x in xs], l, 5, bits, rotate=rotate, dtype=np.float32,
                                bf16=True, out_bf16=False, g0=g0)
        assert (got["range"][p].cpu().numpy() == ref["range"][0]).all(), f"range of chunk {p}"
        for w in range(W):
            assert (got["payloads"][w][p * per:(p + 1) * per].cpu().numpy() == ref["payloads"][w]).all(), (p, w)
        assert (got["out"][g0:g1].cpu().numpy() == ref["out"]).all(), f"output of chunk {p}"


def test_one_pass_minmax_constant_and_zero_chunks():
    """A constant chunk has an empty range: every index 0, decoded exactly; an all-zero
    gradient likewise."""
    bits, W, n = 4, 4, (2 << 14) + 10
    xs = [torch.zeros(n, device=DEV) for _ in range(W)]
    for x in xs:
        x[:1 << 14] = 0.375
    got = run_fused(xs, 1, bits, False)
    assert torch.equal(got["range"][0], torch.tensor([0.375, 0.375], device=DEV))
    assert torch.equal(got["range"][1], torch.zeros(2, device=DEV))
    assert all(int(p.max().item()) == 0 for p in got["payloads"])
    assert torch.equal(got["out"], xs[0])
    got = run_fused([torch.zeros(n, device=DEV) for _ in range(W)], 1, bits, True)
    assert int(got["range"].abs().max().item()) == 0 and int(got["out"].abs().max().item()) == 0


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rotate", [True, False])
def test_one_pass_minmax_zeros_have_the_sign_that_the_per_step_calls_give_them(rotate, dtype):
    """Ranges bit for bit (== does not tell -0 from 0): all-zero chunks of either sign, chunks that
    rotate into one value and zeros (the sign diagonal itself, and its negative), and zeros whose
    signs add up to a -0."""
    W, c, seed = 3, 1 << 14, 29
    n = 7 * c + 4001                                       # the ragged end is all zeros
    diagonal = 1.0 - 2.0 * torch.from_numpy(O.sign_bits(0, n, seed).astype(np.float32)).to(DEV)
    xs = []
    for w in range(W):
        x = torch.zeros(n, device=DEV)
        x[c:2 * c] = diagonal[c:2 * c]
        x[2 * c:3 * c] = -diagonal[2 * c:3 * c]
        x[3 * c:4 * c] = -0.0
        x[4 * c:5 * c] = diagonal[4 * c:5 * c] * -0.0
        x[5 * c:6 * c] = _rand(c, torch.float32, 70 + w)
        xs.append(x.to(dtype))
    print(f"minmax signs of zeros rotate={rotate} dtype={dtype}", flush=True)
    got = run_fused(xs, seed, 4, rotate)
    ref = run_minmax(xs, L14, seed, 4, rotate, torch.float32)
    same = got["range"].view(torch.int32) == ref["range"].view(torch.int32)
    assert bool(same.all()), (got["range"].tolist(), ref["range"].tolist())
    for w in range(W):
        assert torch.equal(got["payloads"][w], ref["payloads"][w])
    assert torch.equal(got["out"].view(torch.int32), ref["out"].view(torch.int32))
    if rotate:
        zeros = got["range"].view(torch.int32)[[0, 3, 4, 6, 7]]
        assert int(zeros.abs().max()) == 0, got["range"].tolist()
        # a gradient at an odd address (other kernels), and the chunk sizes that only they take
        odd = torch.empty(n + 1, dtype=dtype, device=DEV)[1:].copy_(xs[0])
        for l in (14, 9):
            per = 2 * thc.thc_num_chunks(n, l)
            a, b = torch.empty(per, device=DEV), torch.empty(per, device=DEV)
            thc.thc_chunk_minmax(xs[0], l, seed, True, a)
            thc.thc_chunk_minmax(odd, l, seed, True, b)
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))
            assert not bool((a.view(torch.int32) == -(1 << 31)).any())


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rotate", [True, False])
@pytest.mark.parametrize("bits", [2, 4, 8])
def test_minmax_ranges_too_narrow_for_the_reciprocal_step(bits, rotate, dtype):
    """Chunks whose range is narrower than and around 2^-119 (L / (hi - lo) is not finite in
    fp32 much below that): sent like constant chunks; one-pass and per-step forms against
    the oracle and each other."""
    W, c = 3, 1 << 14
    n = 4 * c + 6
    xs = []
    for w in range(W):
        x = _rand(n, torch.float32, 800 + w, scale=1.0, shift=0.0)
        x[:c] *= 2.0 ** -131
        x[c:2 * c] *= 2.0 ** -123
        x[2 * c:3 * c] *= 2.0 ** -121
        xs.append(x.to(dtype))
    print(f"minmax tiny ranges bits={bits} rotate={rotate} dtype={dtype}", flush=True)
    got = run_fused(xs, 6, bits, rotate)
    ref_gpu = run_minmax(xs, L14, 6, bits, rotate, torch.float32)
    assert torch.equal(got["range"], ref_gpu["range"])
    for w in range(W):
        assert torch.equal(got["payloads"][w], ref_gpu["payloads"][w])
    assert torch.equal(got["out"], ref_gpu["out"])
    ref = M.pipeline_minmax([to_numpy_bits(x) for x in xs], L14, 6, bits, rotate=rotate, dtype=np.float32,
                            bf16=dtype == torch.bfloat16, out_bf16=False)
    assert (got["range"].cpu().numpy() == ref["range"]).all()
    for w in range(W):
        assert (got["payloads"][w].cpu().numpy() == ref["payloads"][w]).all(), f"payload {w}"
    assert (got["out"].cpu().numpy() == ref["out"]).all()
    width = got["range"][0, 1] - got["range"][0, 0]
    assert 0 < float(width) < 2.0 ** -119
    assert all(int(p[: c * bits // 8].max()) == 0 for p in got["payloads"])


def test_one_pass_minmax_refuses_what_it_does_not_cover():
    n, W = 1 << 14, 4
    xs = [torch.zeros(n, device=DEV) for _ in range(W)]
    pay = [torch.empty(n // 2, dtype=torch.uint8, device=DEV) for _ in range(W)]
    rng = torch.empty(2, device=DEV)
    out = torch.empty(n, device=DEV)
    ws = torch.empty(thc.thc_encode_all_minmax_workspace_bytes(W, n, L14), dtype=torch.uint8, device=DEV)
    assert thc.thc_encode_all_minmax_workspace_bytes(W, n, 10) == 0
    with pytest.raises(thc.ThcError) as e:
        thc.thc_encode_all_minmax(xs, 10, 0, 4, True, pay, rng, ws)
    assert e.value.status == -3
    with pytest.raises(thc.ThcError) as e:
        thc.thc_encode_all_minmax(xs, L14, 0, 4, True, pay, rng, ws[:64])
    assert e.value.status == -6
    with pytest.raises(thc.ThcError) as e:
        thc.thc_aggregate_decode_minmax(pay, rng, n, 10, 0, 4, True, out)
    assert e.value.status == -3
    with pytest.raises(thc.ThcError) as e:                 # more workers than the one-launch forms take
        thc.thc_aggregate_decode_minmax(pay * 17, rng, n, L14, 0, 4, True, out)
    assert e.value.status == -4
    with pytest.raises(thc.ThcError) as e:
        thc.thc_aggregate_decode_minmax(pay, rng, n, L14, 0, 4, True, torch.empty(n + 1, device=DEV)[1:])
    assert e.value.status == -8
    torch.cuda.synchronize()


@pytest.mark.parametrize("rotate", [True, False])
def test_one_pass_minmax_expired_wait_sets_the_error_word_and_every_wave_exits(rotate):
    """Failure handling forced from the host, as for thc_encode_all: with a poll limit of
    zero the waits between workgroups give up at once; the kernels (the rotated one and the
    pipelined unrotated one) must still finish and report it, and with the limit restored
    the same call on the same workspace is correct again."""
    bits, W = 4, 8
    n = 600 << 14
    xs = [_rand(n, torch.bfloat16, 60 + w, scale=1e-2, shift=1e-3) for w in range(W)]
    P = thc.thc_num_chunks(n, L14)
    pay = [torch.empty(thc.thc_payload_bytes(n, L14, bits), dtype=torch.uint8, device=DEV) for _ in range(W)]
    rng = torch.empty(2 * P, device=DEV)
    ws = torch.empty(thc.thc_encode_all_minmax_workspace_bytes(W, n, L14), dtype=torch.uint8, device=DEV)
    print(f"minmax one-pass expired wait rotate={rotate}", flush=True)
    try:
        thc.thc_set_spin_limit(0)
        thc.thc_encode_all_minmax(xs, L14, 9, bits, rotate, pay, rng, ws)
        torch.cuda.synchronize()            # returns: nothing hangs
        expired = thc.thc_encode_all_timed_out(ws)
    finally:
        thc.thc_set_spin_limit(1 << 22)
    assert expired                           # 4800 items: some wave had to wait at least once
    got = run_fused(xs, 9, bits, rotate)
    ref = run_minmax(xs, L14, 9, bits, rotate, torch.float32)
    assert torch.equal(got["range"], ref["range"])
    for w in range(W):
        assert torch.equal(got["payloads"][w], ref["payloads"][w])


@pytest.mark.parametrize("dtype,bits", [(torch.bfloat16, 4), (torch.float32, 8), (torch.bfloat16, 2)])
@pytest.mark.parametrize("W,chunks", [(8, 48), (8, 49), (8, 64), (8, 65), (17, 30), (17, 31)])   # 384 and 512 places, and beyond
def test_one_pass_minmax_around_one_round_of_workgroups(W, chunks, dtype, bits):
    n = (chunks << 14) - 4097
    print(f"minmax one round W={W} chunks={chunks} {dtype} {bits} bits", flush=True)
    xs = [_rand(n, dtype, 7 * w + chunks, scale=10.0 ** (-2 - (w % 3)), shift=3e-3) for w in range(W)]
    got, ref = run_fused(xs, 23, bits, True), run_minmax(xs, L14, 23, bits, True, torch.float32)
    assert torch.equal(got["range"], ref["range"])
    assert all(torch.equal(got["payloads"][w], ref["payloads"][w]) for w in range(W))
    assert torch.equal(got["out"], ref["out"])


@pytest.mark.parametrize("W,chunks,dtype", [(8, 3, torch.bfloat16), (8, 60, torch.float32), (17, 30, torch.bfloat16)])
def test_expired_wait_in_one_round_leaves_a_workspace_that_can_be_cleared(W, chunks, dtype):
    """The form of one item per workgroup with a poll limit of zero: the launch ends, whether or not a wait had to be
    given up, and the same call on the same workspace is right again with the limit restored."""
    bits, n = 4, (chunks << 14) - 4097
    print(f"minmax one round, expired wait W={W} chunks={chunks} {dtype}", flush=True)
    xs = [_rand(n, dtype, 5 * w + chunks, scale=1e-2, shift=1e-3) for w in range(W)]
    pay = [torch.empty(thc.thc_payload_bytes(n, L14, bits), dtype=torch.uint8, device=DEV) for _ in range(W)]
    rng = torch.empty(2 * thc.thc_num_chunks(n, L14), device=DEV)
    ws = torch.empty(thc.thc_encode_all_minmax_workspace_bytes(W, n, L14), dtype=torch.uint8, device=DEV)
    try:
        thc.thc_set_spin_limit(0)
        thc.thc_encode_all_minmax(xs, L14, 9, bits, True, pay, rng, ws)
        torch.cuda.synchronize()            # returns: nothing hangs
    finally:
        thc.thc_set_spin_limit(1 << 22)
    thc.thc_encode_all_minmax(xs, L14, 9, bits, True, pay, rng, ws)
    torch.cuda.synchronize()
    assert not thc.thc_encode_all_timed_out(ws)
    ref = run_minmax(xs, L14, 9, bits, True, torch.float32)
    assert torch.equal(rng.view(-1, 2), ref["range"])
    assert all(torch.equal(pay[w], ref["payloads"][w]) for w in range(W))
