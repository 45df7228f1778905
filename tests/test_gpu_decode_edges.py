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
    n = 3 * (1 << 14) + 77   # (with more chunks than a device holds at once: the next test)
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


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("W", [1, 3, 4, 5, 9, 12, 17, 18, 33, 47, 64])
def test_sums_of_every_number_of_workers_while_the_previous_chunk_rotates(W, bits):
    """More chunks than a device holds workgroups (two per CU), so that a workgroup's later chunks are loaded and
    summed piece by piece inside the rotation of the one before: a single group, parts of groups, odd numbers of
    groups, sums of 16 bits of 4-bit payloads.  One call with and without the integer sums, and the batched call
    over two buckets, against thc_aggregate + thc_decode; the sums against torch."""
    l, seed = 14, 3
    resident = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    n = ((2 * resident + 9) << l) - 1111   # (a third item for some workgroups, a ragged last one)
    print(f"decoder W={W} bits={bits} n={n}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(W * 10 + bits)
    P, nb = thc.thc_num_chunks(n, l), thc.thc_payload_bytes(n, l, bits)
    payloads = [torch.randint(0, 256, (nb,), dtype=torch.uint8, device="cuda", generator=gen) for _ in range(W)]
    for p in payloads:
        p[nb // 2: nb // 2 + nb // 8] = 255   # the largest sums
    scale = torch.rand(P, device="cuda", generator=gen) + 0.5
    one = thc.thc_sum_bytes(W, bits) == 1
    sums = torch.zeros(P << l, dtype=torch.uint8 if one else torch.int16, device="cuda")
    thc.thc_aggregate(payloads, n, l, bits, sums)
    fields = torch.zeros((nb, 8 // bits), dtype=torch.int32, device="cuda")
    for p in payloads:
        for k in range(8 // bits):
            fields[:, k] += ((p >> (bits * k)) & ((1 << bits) - 1)).to(torch.int32)
    assert torch.equal(fields.view(-1).to(sums.dtype), sums)
    want = torch.empty(n, device="cuda")
    thc.thc_decode(sums, scale, W, n, l, seed, bits, want)
    fused = thc.thc_aggregate_decode_is_fused(W, l, bits)   # (one worker of 8 bits takes the two steps)
    for keep in (True, False) if fused else (True,):
        mine, out = torch.zeros_like(sums), torch.full((n,), float("nan"), device="cuda")
        thc.thc_aggregate_decode(payloads, scale, n, l, seed, bits, mine if keep else None, out)
        assert torch.equal(out, want), keep
        assert not keep or torch.equal(mine, sums)
    if not fused:
        return
    # two buckets: chunks 0 .. cut - 1 and the rest, each numbered from zero (their signs follow the bucket's seed)
    cut = resident - 3
    parts = [(0, cut << l), (cut << l, n)]
    outs = [torch.full((b - a,), float("nan"), device="cuda") for a, b in parts]
    buckets = [dict(n=b - a, seed=seed + k, payloads=[p[a * bits // 8:] for p in payloads], scale=scale[a >> l:].clone(),
                    out=outs[k]) for k, (a, b) in enumerate(parts)]
    ws = torch.empty(thc.thc_batch_workspace_bytes([b - a for a, b in parts], W, l), dtype=torch.uint8, device="cuda")
    thc.thc_aggregate_decode_batch(buckets, l, bits, ws)
    for k, (a, b) in enumerate(parts):
        ref = torch.empty(b - a, device="cuda")
        thc.thc_decode(sums[a:], buckets[k]["scale"], W, b - a, l, seed + k, bits, ref)
        assert torch.equal(outs[k], ref), k


@pytest.mark.parametrize("count", [False, True])
@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("W", [1, 3, 4, 5, 9, 18, 33, 64])
def test_saturating_decoder_of_every_number_of_workers_over_several_rounds(W, bits, count):
    """The same for the saturating decoder, whose workgroups load the first two groups of the next chunk one item
    ahead: aggregate, output and number of clipped coordinates against thc_sat_aggregate + thc_sat_decode."""
    l, seed = 14, 3
    resident = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    n = ((resident + 9) << l) - 1111
    print(f"saturating decoder W={W} bits={bits} n={n}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(W * 10 + bits)
    P, nb = thc.thc_num_chunks(n, l), thc.thc_payload_bytes(n, l, bits)
    # (the largest index on the grid of 2 M + 1 points is 2 M = 2^bits - 2, never all ones)
    low = torch.tensor(sum(1 << (bits * k) for k in range(8 // bits)), dtype=torch.uint8, device="cuda")
    payloads = []
    for _ in range(W):
        p = torch.randint(0, 256, (nb,), dtype=torch.uint8, device="cuda", generator=gen)
        ones = p.clone()
        for k in range(1, bits):
            ones &= p >> k
        payloads.append(p - (ones & low))   # fields of all ones lose their lowest bit
    scale = torch.rand(P, device="cuda", generator=gen) + 0.5
    aggregate, clipped = torch.zeros(nb, dtype=torch.uint8, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")
    thc.thc_sat_aggregate(payloads, n, l, bits, aggregate, clipped)
    want = torch.empty(n, device="cuda")
    thc.thc_sat_decode(aggregate, scale, W, n, l, seed, bits, want)
    for keep in (True, False):
        mine, mine_clipped = torch.zeros_like(aggregate), torch.zeros_like(clipped)
        out = torch.full((n,), float("nan"), device="cuda")
        thc.thc_sat_aggregate_decode(payloads, scale, n, l, seed, bits, mine if keep else None,
                                     mine_clipped if count else None, out)
        assert torch.equal(out, want), keep
        assert not keep or torch.equal(mine, aggregate)
        assert not count or torch.equal(mine_clipped, clipped)


@pytest.mark.parametrize("chunks", [224, 225])   # 64 workers, 224 MiB and a little more: ordinary loads on both sides (less than 8 M coordinates)
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


@pytest.mark.parametrize("form,l,chunks", [   # 16 workers: both sides of 20, 52 and 224 MiB, of 176 for small chunks
    ("exact", 14, 80), ("exact", 14, 81), ("exact", 14, 208), ("exact", 14, 209), ("sat", 14, 81), ("sat", 14, 209),
    ("sat counted", 14, 208),
    ("exact", 14, 896), ("exact", 14, 897), ("sat", 14, 896), ("sat", 14, 897), ("sat counted", 14, 897),
    ("exact", 12, 2816), ("exact", 12, 2817), ("exact", 5, 360449),
])
def test_8_bit_payloads_on_both_sides_of_the_line_of_streaming_loads(form, l, chunks):
    W, bits, seed = 16, 8, 11
    n = (chunks << l) - 5
    gen = torch.Generator(device="cuda").manual_seed(chunks)
    payloads = [torch.randint(0, 255, (chunks << l,), dtype=torch.uint8, device="cuda", generator=gen) for _ in range(W)]
    scale = torch.rand(chunks, device="cuda", generator=gen) + 0.5
    want, out = torch.empty(n, device="cuda"), torch.full((n,), 7.0, device="cuda")
    if form == "exact":
        sums = torch.zeros(chunks << l, dtype=torch.int16, device="cuda")
        mine = torch.zeros_like(sums)
        thc.thc_aggregate(payloads, n, l, bits, sums)
        thc.thc_decode(sums, scale, W, n, l, seed, bits, want)
        thc.thc_aggregate_decode(payloads, scale, n, l, seed, bits, mine, out)
        assert torch.equal(sum(p.to(torch.int32) for p in payloads).to(torch.int16), sums)
    else:
        sums = torch.zeros(chunks << l, dtype=torch.uint8, device="cuda")
        mine = torch.zeros_like(sums)
        clipped = torch.zeros(2, dtype=torch.int64, device="cuda")
        thc.thc_sat_aggregate(payloads, n, l, bits, sums, clipped[:1])
        thc.thc_sat_decode(sums, scale, W, n, l, seed, bits, want)
        thc.thc_sat_aggregate_decode(payloads, scale, n, l, seed, bits, mine, clipped[1:] if form != "sat" else None, out)
        assert form == "sat" or int(clipped[0]) == int(clipped[1])
    assert torch.equal(out, want) and torch.equal(mine, sums)


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("l", [5, 10, 11, 12, 13])
@pytest.mark.parametrize("W", [1, 3, 4, 5, 8, 9, 18])
def test_small_chunk_decoder_in_workgroups_of_every_width(W, l, bits):
    """Workgroups of four, two and one wave, on both sides of each length where the width changes (2, 4, a quarter, half, once
    and twice the number of CUs, in workgroups of four waves).  The sums of a call and of thc_aggregate, the output of it and of thc_decode,
    which deals the chunks out in its own widths; and two lengths of one gradient agree where both have whole chunks."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    seed, before = 5, None
    gen = torch.Generator(device="cuda").manual_seed(W * 10 + bits)
    most = (2 * cus) << 13
    flat = [torch.randint(0, 256, (most * bits // 8,), dtype=torch.uint8, device="cuda", generator=gen) for _ in range(W)]
    scales = torch.rand(most >> l, device="cuda", generator=gen) + 0.5
    for groups in (1, 2, 3, 4, 5, cus // 4, cus // 4 + 1, cus // 2, cus // 2 + 1, cus, cus + 1, 2 * cus - 1, 2 * cus):
        n = (groups << 13) - (1 << 13) + 33 if groups == 1 else (groups << 13) - 31
        P, nb = thc.thc_num_chunks(n, l), thc.thc_payload_bytes(n, l, bits)
        payloads, scale = [f[:nb] for f in flat], scales[:P]
        sums = torch.zeros(P << l, dtype=torch.uint8 if thc.thc_sum_bytes(W, bits) == 1 else torch.int16, device="cuda")
        thc.thc_aggregate(payloads, n, l, bits, sums)
        want, out, mine = torch.empty(n, device="cuda"), torch.full((n,), float("nan"), device="cuda"), torch.zeros_like(sums)
        thc.thc_decode(sums, scale, W, n, l, seed, bits, want)
        thc.thc_aggregate_decode(payloads, scale, n, l, seed, bits, mine, out)
        assert torch.equal(mine, sums) and torch.equal(out, want), groups
        whole = 0 if before is None else before.numel() >> l << l
        assert whole == 0 or torch.equal(out[:whole], before[:whole]), groups
        before = out


@pytest.mark.parametrize("bits,W", [(4, 8), (4, 13), (2, 9), (8, 5), (4, 18), (4, 24), (4, 25), (4, 64), (8, 64)])
@pytest.mark.parametrize("per_cu,more", [(1, 0), (1, 1), (2, 0), (2, 1)])
def test_one_chunk_per_workgroup_and_more(W, bits, per_cu, more):
    """One and two workgroups per CU and one more (two are resident): up to there every chunk has its own; the last chunk
    ragged, with and without the sums: against thc_aggregate + thc_decode."""
    l, seed = 14, 9
    chunks = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + more
    n = (chunks << l) - 12345
    gen = torch.Generator(device="cuda").manual_seed(W)
    flat = torch.randint(0, 256, (W, thc.thc_payload_bytes(n, l, bits)), dtype=torch.uint8, generator=gen, device="cuda")
    payloads = list(flat.unbind(0))
    scale = torch.rand(chunks, generator=gen, device="cuda") + 0.5
    dtype = torch.uint8 if thc.thc_sum_bytes(W, bits) == 1 else torch.int16
    want_sums, sums = (torch.empty(chunks << l, dtype=dtype, device="cuda") for _ in range(2))
    want, out, plain = (torch.empty(n, device="cuda") for _ in range(3))
    thc.thc_aggregate(payloads, n, l, bits, want_sums)
    thc.thc_decode(want_sums, scale, W, n, l, seed, bits, want)
    thc.thc_aggregate_decode(payloads, scale, n, l, seed, bits, sums, out)
    thc.thc_aggregate_decode(payloads, scale, n, l, seed, bits, None, plain)
    assert torch.equal(sums, want_sums) and torch.equal(out, want) and torch.equal(plain, want)
