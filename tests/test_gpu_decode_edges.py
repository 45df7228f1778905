"""The decoders store through buffer descriptors: the coordinates behind a ragged end stay untouched, the
last ones in front of it are written, with 1, 2, 3 and 0 coordinates of the last 16 bytes, in the one-launch
forms and in thc_decode.  The payload sums run in groups of workers: 1 .. 64 workers, so that every
number of whole groups and every rest occurs, against the sum of the payloads in numpy."""
import numpy as np
import pytest
import torch

import paper_2407_01378_amd as thc
from oracle import thc as O

pytestmark = pytest.mark.gpu
GUARD = 64


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 2047, 16381, 16383, 16384, 16385, 16386, 40003])
def test_nothing_is_written_behind_a_ragged_end(n):
    W, l, bits, seed = 3, 14, 4, 5
    P = thc.thc_num_chunks(n, l)
    rng = np.random.default_rng(n)
    payloads = [torch.from_numpy(rng.integers(0, 256, thc.thc_payload_bytes(n, l, bits), dtype=np.uint8)).cuda()
                for _ in range(W)]
    scale = torch.from_numpy(rng.uniform(0.5, 2.0, P).astype(np.float32)).cuda()
    sums = torch.empty(P << l, dtype=torch.uint8, device="cuda")
    thc.thc_aggregate(payloads, n, l, bits, sums)
    outs = []
    for form in ("fused", "fused_batch_like", "decode", "sat"):
        whole = torch.full((n + GUARD,), 7.0, dtype=torch.float32, device="cuda")
        out = whole[:n]
        if form == "decode":
            thc.thc_decode(sums, scale, W, n, l, seed, bits, out)
        elif form == "sat":
            thc.thc_sat_aggregate_decode(payloads, scale, n, l, seed, bits, None, None, out)
        else:
            thc.thc_aggregate_decode(payloads, scale, n, l, seed, bits, sums if form == "fused" else None, out)
        torch.cuda.synchronize()
        assert torch.equal(whole[n:], torch.full((GUARD,), 7.0, device="cuda")), (form, n)
        assert not bool((out == 7.0).any()), (form, n)
        if form != "sat":
            outs.append(out)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    want = O.decode(sums.cpu().numpy(), scale.cpu().numpy().astype(np.float64), W, n, l, seed, bits)
    # (the rotation's own rounding, relative to the whole rotated chunk: 14 stages of 2^-24)
    err = np.abs(outs[0].cpu().numpy() - want).max() / np.sqrt(np.mean(want ** 2) + 1e-30)
    assert err < 1e-4, (n, err)


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 8, 11, 12, 13, 15, 16, 17, 18, 19, 20, 31, 32, 33, 47, 63, 64])
@pytest.mark.parametrize("l", [10, 14])
def test_sums_of_every_number_of_workers(W, bits, l):
    n = 3 * (1 << 14) + 77   # (with more chunks than a device holds at once: test_gpu_timed_path.py)
    rng = np.random.default_rng(W * 10 + bits)
    count = thc.thc_payload_bytes(n, l, bits)
    raw = rng.integers(0, 256, (W, count), dtype=np.uint8)
    raw[:, : count // 4] = 255   # the largest sums
    payloads = [torch.from_numpy(r.copy()).cuda() for r in raw]
    P = thc.thc_num_chunks(n, l)
    scale = torch.ones(P, dtype=torch.float32, device="cuda")
    one = thc.thc_sum_bytes(W, bits) == 1
    sums = torch.empty(P << l, dtype=torch.uint8 if one else torch.int16, device="cuda")
    out = torch.empty(n, dtype=torch.float32, device="cuda")
    thc.thc_aggregate_decode(payloads, scale, n, l, 1, bits, sums, out)
    total = np.zeros((count, 8 // bits), np.int64)
    for r in raw:
        for k in range(8 // bits):
            total[:, k] += (r >> (bits * k)) & ((1 << bits) - 1)
    got = sums.cpu().numpy().view(np.uint8 if one else np.uint16)
    assert (got == total.reshape(-1)[: P << l]).all()


@pytest.mark.parametrize("chunks", [224, 225])   # 64 workers: the last size read by ordinary loads, the first by streaming ones
def test_8_bit_payloads_around_the_size_of_the_last_level_cache(chunks):
    W, l, bits, seed = 64, 14, 8, 11
    n = (chunks << l) - 5
    gen = torch.Generator(device="cuda").manual_seed(chunks)
    payloads = [torch.randint(0, 256, (chunks << l,), dtype=torch.uint8, device="cuda", generator=gen) for _ in range(W)]
    scale = torch.rand(chunks, device="cuda", generator=gen) + 0.5
    sums = torch.zeros(chunks << l, dtype=torch.int16, device="cuda")
    thc.thc_aggregate(payloads, n, l, bits, sums)
    total = sum(p.to(torch.int32) for p in payloads)
    assert torch.equal(total.to(torch.int16), sums)
    want = torch.empty(n, device="cuda")
    thc.thc_decode(sums, scale, W, n, l, seed, bits, want)
    one = torch.full((n,), 7.0, device="cuda")
    mine = torch.zeros_like(sums)
    thc.thc_aggregate_decode(payloads, scale, n, l, seed, bits, mine, one)
    assert torch.equal(one, want) and torch.equal(mine, sums)
    many = torch.full((n,), 7.0, device="cuda")
    ws = torch.empty(thc.thc_batch_workspace_bytes([n], W, l), dtype=torch.uint8, device="cuda")
    thc.thc_aggregate_decode_batch([dict(n=n, seed=seed, payloads=payloads, scale=scale, out=many)], l, bits, ws)
    assert torch.equal(many, want)
