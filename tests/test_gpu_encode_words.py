"""The one-pass encoder's forms of agreement (a word per wave, per workgroup, one reader per workgroup, each also
for launches of one item per workgroup), on both sides of the worker counts where they change, with one item
per workgroup, a few and more than eight rounds: scales and payloads are those of the per-worker calls, and
the workspace comes back clear."""
import pytest
import torch

import paper_2407_01378_amd as thc

pytestmark = pytest.mark.gpu
GRID = 512   # workgroups that are resident at once


@pytest.mark.parametrize("W", [1, 2, 15, 16, 17, 32, 33, 36, 64])
@pytest.mark.parametrize("rounds,dtype,bits", [(0, torch.bfloat16, 4), (0, torch.float32, 8), (3, torch.bfloat16, 2),
                                               (3, torch.float32, 4), (6, torch.bfloat16, 4), (7, torch.bfloat16, 4), (10, torch.bfloat16, 4), (10, torch.float32, 8)])
def test_agreement_matches_the_per_worker_calls(W, rounds, dtype, bits):
    per_round = GRID // W
    chunks = min(rounds * per_round + 1, 256) if W == 1 else rounds * per_round + 1
    n = (chunks << 14) - 1234   # even and ragged
    if rounds == 0:
        n -= 1                  # odd
    print(f"W={W} chunks={chunks} n={n} {dtype} {bits} bits", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W)
    xs = [torch.randn(n, generator=gen, device="cuda").mul_(10.0 ** (w % 3)).to(dtype) for w in range(W)]
    P, nb = thc.thc_num_chunks(n, 14), thc.thc_payload_bytes(n, 14, bits)
    ws = torch.empty(thc.thc_encode_all_workspace_bytes(W, n, 14), dtype=torch.uint8, device="cuda")
    thc.thc_workspace_clear(ws)
    scale = torch.full((P,), float("nan"), device="cuda")
    payloads = [torch.full((nb,), 0xAA, dtype=torch.uint8, device="cuda") for _ in range(W)]
    thc.thc_encode_all_cleared(xs, 14, 7, bits, payloads, scale, ws)
    torch.cuda.synchronize()
    assert int(ws.count_nonzero()) == 0
    _matches_the_per_worker_calls(xs, bits, scale, payloads)


def _matches_the_per_worker_calls(xs, bits, scale, payloads):
    W, P = len(xs), scale.numel()
    absmax = torch.empty(W * P, device="cuda")
    for w in range(W):
        thc.thc_chunk_absmax(xs[w], 14, 7, absmax[w * P:(w + 1) * P])
    shared = torch.empty(P, device="cuda")
    thc.thc_scale_reduce(absmax, W, P, shared)
    assert torch.equal(scale, shared)
    ref = torch.empty_like(payloads[0])
    for w in range(W):
        thc.thc_encode(xs[w], 14, 7, w, bits, shared, ref)
        assert torch.equal(payloads[w], ref), w


@pytest.mark.parametrize("W,chunks", [(8, 640), (8, 641), (64, 81)])
def test_streamed_fp32_gradients_match_the_per_worker_calls(W, chunks):
    """fp32 gradients of more than 5120 chunks in all are read as for the last time: both sides of the line, ragged."""
    n, bits = (chunks << 14) - 4321, 4
    xs = [torch.randn(n, generator=torch.Generator(device="cuda").manual_seed(w), device="cuda") for w in range(W)]
    P, nb = thc.thc_num_chunks(n, 14), thc.thc_payload_bytes(n, 14, bits)
    ws = torch.empty(thc.thc_encode_all_workspace_bytes(W, n, 14), dtype=torch.uint8, device="cuda")
    scale = torch.full((P,), float("nan"), device="cuda")
    payloads = [torch.full((nb,), 0xAA, dtype=torch.uint8, device="cuda") for _ in range(W)]
    thc.thc_encode_all(xs, 14, 7, bits, payloads, scale, ws)
    _matches_the_per_worker_calls(xs, bits, scale, payloads)


@pytest.mark.parametrize("W,rounds,dtype,bits", [
    (20, 3, torch.bfloat16, 4), (20, 10, torch.float32, 2),     # a word per workgroup, every wave reads
    (64, 3, torch.bfloat16, 4),                                 # the same beyond 32 workers
    (64, 3, torch.float32, 4), (64, 10, torch.bfloat16, 8),     # one reader, few rounds and the late pause
    (2, 0, torch.bfloat16, 4), (8, 0, torch.float32, 8),        # one item per workgroup: a word per wave
    (20, 0, torch.bfloat16, 4), (32, 0, torch.float32, 8),      # a word per workgroup
    (33, 0, torch.float32, 2), (64, 0, torch.bfloat16, 4),      # one reader
])
def test_expired_wait_of_every_form_of_agreement(W, rounds, dtype, bits):
    """Failure handling forced from the host: with a poll limit of zero a wait gives up after one read.  Every wave
    still ends, over several rounds the error word is set (a word takes longer from one workgroup to another
    than the pause in front of that read), and a cleared workspace is good again."""
    n = ((rounds * (GRID // W) + 1) << 14) - 1234
    print(f"expired wait W={W} n={n} {dtype} {bits} bits", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W)
    xs = [torch.randn(n, generator=gen, device="cuda").mul_(10.0 ** (w % 3)).to(dtype) for w in range(W)]
    P, nb = thc.thc_num_chunks(n, 14), thc.thc_payload_bytes(n, 14, bits)
    ws = torch.empty(thc.thc_encode_all_workspace_bytes(W, n, 14), dtype=torch.uint8, device="cuda")
    thc.thc_workspace_clear(ws)
    scale = torch.full((P,), float("nan"), device="cuda")
    payloads = [torch.full((nb,), 0xAA, dtype=torch.uint8, device="cuda") for _ in range(W)]
    torch.cuda.synchronize()
    try:
        thc.thc_set_spin_limit(0)
        thc.thc_encode_all_cleared(xs, 14, 7, bits, payloads, scale, ws)
        torch.cuda.synchronize()            # returns: nothing hangs
    finally:
        thc.thc_set_spin_limit(1 << 22)
    assert rounds == 0 or thc.thc_encode_all_timed_out(ws)
    thc.thc_workspace_clear(ws)
    thc.thc_encode_all_cleared(xs, 14, 7, bits, payloads, scale, ws)
    torch.cuda.synchronize()
    assert int(ws.count_nonzero()) == 0
    _matches_the_per_worker_calls(xs, bits, scale, payloads)


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("W,chunks,rest", [(3, 1, 1), (3, 2, 31), (8, 4, 33), (8, 3, 16383), (24, 2, 8191), (40, 1, 16351),   # one round
                                           (2, 300, 1), (8, 70, 65), (24, 25, 16383), (40, 14, 32769 - 16384)])
def test_odd_counts_of_bf16(W, chunks, rest, bits):
    """The last coordinate of an odd count, by the thread of the last chunk that owns it; in launches of one round and of
    several, for every form of agreement."""
    n = ((chunks - 1) << 14) + rest
    print(f"odd W={W} n={n} {bits} bits", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W + rest)
    xs = [torch.randn(n, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(W)]
    for w in range(W):
        xs[w][-1] = 40.0 + w          # it decides the range of its chunk
    P, nb = thc.thc_num_chunks(n, 14), thc.thc_payload_bytes(n, 14, bits)
    ws = torch.empty(thc.thc_encode_all_workspace_bytes(W, n, 14), dtype=torch.uint8, device="cuda")
    scale = torch.full((P,), float("nan"), device="cuda")
    payloads = [torch.full((nb,), 0xAA, dtype=torch.uint8, device="cuda") for _ in range(W)]
    thc.thc_encode_all(xs, 14, 7, bits, payloads, scale, ws)
    _matches_the_per_worker_calls(xs, bits, scale, payloads)
