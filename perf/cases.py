"""The work a user of this library has it do, as cases that can be timed and compared.

A case is one pass through the public entry points for one gradient (or one DDP-style bucket of
it) of W workers simulated on one GPU.  What a case does is named by "path":

  step    one-pass encode of all workers, then aggregate + decode: the timed path of bench.py
  batch   the same two calls over all buckets of a gradient at once
  calls   one call per step of the method and worker, as a deployment with one worker per process
          issues them: range, shared scale, encode, aggregate, decode
  sat     one-pass encode and decode with the saturating b-bit aggregate
  minmax  one-pass encode and decode on the min/max grid, with or without the rotation
  full    one rotation over the whole zero-padded gradient (2^l coordinates)
  topkc   a TopK Chunked round: norms, their sum, selection, chunk sums, dense estimate

Other fields: W workers, n coordinates per worker, dtype of the gradients, bits of a payload,
chunk_log2 of the rotation (14 where absent), values (how the gradients are distributed).
"""
import math

import torch

import paper_2407_01378_amd as thc

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_BUCKET = 25 * (1 << 20)   # coordinates of a DDP-style bucket


def listed():
    return [
        # the last, short bucket of a training step (one vocabulary-sized vector): launch latency
        dict(name="vector_bucket", path="step", W=8, n=50257, dtype="bf16", bits=4, chunk_log2=14, values="student3"),
        # the Tiny configuration: four workers, a million coordinates, small chunks
        dict(name="tiny", path="step", W=4, n=1 << 20, dtype="f32", bits=4, chunk_log2=10, values="layers"),
        # a 25 MB DDP bucket (framework default), chunks that also fit a smaller scratchpad, 8-bit payloads
        dict(name="bucket25mb_chunk12", path="step", W=8, n=6553593, dtype="bf16", bits=8, chunk_log2=12,
             values="student3"),
        # the ResNet-50 configuration: the whole fp32 gradient as one bucket, ragged end
        dict(name="resnet50", path="step", W=8, n=25557032, dtype="f32", bits=4, chunk_log2=14, values="layers"),
        # one bucket of the 1.3 B headline configuration
        dict(name="gpt_1p3b_bucket", path="step", W=8, n=_BUCKET, dtype="bf16", bits=4, chunk_log2=14,
             values="student3"),
        # many data-parallel workers on a smaller piece: sums wider than a byte
        dict(name="workers64", path="step", W=64, n=1 << 21, dtype="bf16", bits=4, chunk_log2=14, values="student3"),
        # the GPT 345M configuration at two bits, every bucket handed over in one call
        dict(name="gpt_345m_batch", path="batch", W=8, n=353551360, dtype="bf16", bits=2, values="student3"),
        # one BERT-base layer through the calls a one-worker-per-process deployment makes
        dict(name="bert_layer_calls", path="calls", W=8, n=7080960, dtype="bf16", bits=8, chunk_log2=14,
             values="student3"),
        # saturation-based aggregation, last bucket of the headline configuration
        dict(name="gpt_1p3b_tail_sat", path="sat", W=8, n=15494400, dtype="bf16", bits=4, values="student3"),
        # min/max range without rotation (the "no rotation" column of the throughput table)
        dict(name="minmax_no_rotation", path="minmax", W=8, n=_BUCKET, dtype="bf16", bits=4, rotate=False,
             values="student3"),
        # full rotation (the baseline of the partial one) of the ResNet-50 gradient
        dict(name="resnet50_full_rotation", path="full", W=8, n=25557032, dtype="f32", bits=4, values="layers"),
        # TopKC round on the BERT-base gradient (sparse embedding rows) at two bits per coordinate
        dict(name="bert_base_topkc", path="topkc", W=8, n=108412416, dtype="bf16", C=64, target_bits=2.0,
             values="sparse_rows"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["step", "step", "step", "step", "batch", "calls", "sat", "minmax", "full", "topkc"])
    W = rng.choice([2, 4, 8, 8, 8])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    values = rng.choice(["student3", "student3", "layers", "sparse_rows"])
    bits = rng.choice([2, 4, 4, 8])
    if path == "step":
        W = rng.choice([2, 4, 8, 8, 8, 16, 32, 64])
        return dict(path=path, W=W, n=_log_int(rng, 1 << 14, min(1 << 25, (1 << 28) // W)), dtype=dtype, bits=bits,
                    chunk_log2=rng.choice([8, 10, 11, 12, 13, 14, 14, 14, 14, 14]), values=values)
    if path == "batch":
        return dict(path=path, W=W, n=_log_int(rng, _BUCKET // 2, 5 * _BUCKET), dtype=dtype, bits=bits, values=values)
    if path == "calls":
        return dict(path=path, W=W, n=_log_int(rng, 1 << 15, 1 << 24), dtype=dtype, bits=bits,
                    chunk_log2=rng.choice([10, 12, 14, 14, 14]), values=values)
    if path == "sat":
        return dict(path=path, W=W, n=_log_int(rng, 1 << 16, 1 << 25), dtype=dtype, bits=bits, values=values)
    if path == "minmax":
        return dict(path=path, W=W, n=_log_int(rng, 1 << 16, 1 << 25), dtype=dtype, bits=bits,
                    rotate=rng.random() < 0.5, values=values)
    if path == "full":
        return dict(path=path, W=W, n=_log_int(rng, 1 << 17, 1 << 25), dtype=dtype, bits=bits, values=values)
    return dict(path=path, W=W, n=_log_int(rng, 1 << 17, 1 << 27), dtype=dtype, C=rng.choice([32, 64, 64, 128]),
                target_bits=rng.choice([1.0, 2.0, 2.0, 4.0]), values=values)


# ------------------------------------------------------------------------------ inputs
def _student3(m, gen):
    z = torch.randn(4, m, generator=gen, device="cuda")
    return z[0] / torch.sqrt((z[1] * z[1] + z[2] * z[2] + z[3] * z[3]) / 3.0)


def _gradient(case, gen, scales):
    """One worker's flattened gradient: layers of 2^20 coordinates, each with its own magnitude."""
    n = case["n"]
    v = torch.randn(n, generator=gen, device="cuda") if case["values"] == "layers" else _student3(n, gen)
    if case["values"] == "sparse_rows":   # the first fifth is an embedding: whole rows of 768 are zero
        rows = n // 5 // 768
        keep = torch.rand(rows, generator=gen, device="cuda") >= 0.99
        v[:rows * 768].view(rows, 768).mul_(keep.view(rows, 1))
        v *= 1e-3
    else:
        v *= scales.repeat_interleave(1 << 20)[:n]
    return v.to(_DTYPES[case["dtype"]])


def _gradients(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    layers = (case["n"] + (1 << 20) - 1) >> 20
    lo, hi = math.log(1e-5), math.log(1e-2)   # layer magnitudes, the same for every worker
    scales = torch.exp(torch.rand(layers, generator=gen, device="cuda") * (hi - lo) + lo)
    return [_gradient(case, gen, scales) for _ in range(case["W"])]


def _u8(count):
    return torch.empty(count, dtype=torch.uint8, device="cuda")


def _f32(count):
    return torch.empty(count, dtype=torch.float32, device="cuda")


def _payloads(W, count):
    """One flat buffer for all workers (a send buffer), and every worker's part of it."""
    flat = _u8(W * count)
    return dict(payload_buffer=flat, payloads=[flat[w * count:(w + 1) * count] for w in range(W)])


def _sums(case, count):
    return torch.empty(count, dtype=torch.uint8 if thc.thc_sum_bytes(case["W"], case["bits"]) == 1 else torch.int16,
                       device="cuda")


def _topkc_count(case):
    return max(1, int((case["target_bits"] / 16.0 - 1.0 / case["C"]) * case["n"] / case["C"]))


def prepare(case, seed):
    """Gradients, buffers and workspaces, as a training loop keeps them from step to step."""
    W, n, path = case["W"], case["n"], case["path"]
    l = case.get("chunk_log2", 14)
    s = dict(case=case, seed=seed & 0xFFFFF, grads=_gradients(case, seed), out=_f32(n))
    if path == "topkc":
        P, J = thc.topkc_num_chunks(n, case["C"]), _topkc_count(case)
        s.update(P=P, J=J, norms=torch.empty(W * P, dtype=torch.float16, device="cuda"),
                 total=torch.empty(P, dtype=torch.float16, device="cuda"),
                 indices=torch.empty(J, dtype=torch.int32, device="cuda"),
                 ws=_u8(thc.topkc_select_workspace_bytes(P)),
                 picked=torch.empty(J * case["C"], dtype=torch.float16, device="cuda"))
        return s
    bits = case["bits"]
    if path == "full":
        l = thc.thc_full_log2(n)
        s.update(l=l, ys=[_f32(1 << l) for _ in range(W)], absmax=_f32(W), scale=_f32(1),
                 sums=_sums(case, 1 << l), **_payloads(W, (bits << l) // 8))
        return s
    P = thc.thc_num_chunks(n, l)
    s.update(P=P, l=l, scale=_f32(P), **_payloads(W, thc.thc_payload_bytes(n, l, bits)))
    if path == "batch":
        # flat buffers, one record per bucket (whole chunks except at the end)
        s["buckets"] = []
        for k, at in enumerate(range(0, n, _BUCKET)):
            m = min(_BUCKET, n - at)
            p0, b0 = at >> 14, at * bits // 8
            pb = thc.thc_payload_bytes(m, 14, bits)
            s["buckets"].append(dict(grads=[g[at:at + m] for g in s["grads"]], n=m, seed=s["seed"] + k,
                                     payloads=[p[b0:b0 + pb] for p in s["payloads"]],
                                     scale=s["scale"][p0:p0 + thc.thc_num_chunks(m, 14)], out=s["out"][at:at + m]))
        s["ws"] = _u8(thc.thc_batch_workspace_bytes([b["n"] for b in s["buckets"]], W, 14))
    elif path == "minmax":
        s["scale"] = _f32(2 * P)
        s["ws"] = _u8(thc.thc_encode_all_minmax_workspace_bytes(W, n, 14))
    elif path == "calls":
        s.update(absmax=_f32(W * P), sums=_sums(case, P << l))
    else:
        # one workspace per bucket, cleared once: the calls leave it clear
        s["ws"] = _u8(thc.thc_encode_all_workspace_bytes(W, n, l))
        thc.thc_workspace_clear(s["ws"])
        s["sums"] = _sums(case, P << l) if path == "step" and l != 14 else None
    return s


# -------------------------------------------------------------------------------- a pass
def _step(s, n, l, bits):
    thc.thc_encode_all_cleared(s["grads"], l, s["seed"], bits, s["payloads"], s["scale"], s["ws"])
    thc.thc_aggregate_decode(s["payloads"], s["scale"], n, l, s["seed"], bits, s["sums"], s["out"])
    return [s["payload_buffer"], s["scale"], s["sums"], s["out"]]


def _batch(s, bits):
    thc.thc_encode_all_batch(s["buckets"], 14, bits, s["ws"])
    thc.thc_aggregate_decode_batch(s["buckets"], 14, bits, s["ws"])
    return [s["payload_buffer"], s["scale"], s["out"]]


def _calls(s, W, n, l, bits):
    P = s["P"]
    for w in range(W):
        thc.thc_chunk_absmax(s["grads"][w], l, s["seed"], s["absmax"][w * P:(w + 1) * P])
    thc.thc_scale_reduce(s["absmax"], W, P, s["scale"])
    for w in range(W):
        thc.thc_encode(s["grads"][w], l, s["seed"], w, bits, s["scale"], s["payloads"][w])
    thc.thc_aggregate(s["payloads"], n, l, bits, s["sums"])
    thc.thc_decode(s["sums"], s["scale"], W, n, l, s["seed"], bits, s["out"])
    return [s["absmax"], s["scale"], s["payload_buffer"], s["sums"], s["out"]]


def _sat(s, n, bits):
    thc.thc_sat_encode_all_cleared(s["grads"], 14, s["seed"], bits, s["payloads"], s["scale"], s["ws"])
    thc.thc_sat_aggregate_decode(s["payloads"], s["scale"], n, 14, s["seed"], bits, None, None, s["out"])
    return [s["payload_buffer"], s["scale"], s["out"]]


def _minmax(s, n, bits, rotate):
    thc.thc_encode_all_minmax(s["grads"], 14, s["seed"], bits, rotate, s["payloads"], s["scale"], s["ws"])
    thc.thc_aggregate_decode_minmax(s["payloads"], s["scale"], n, 14, s["seed"], bits, rotate, s["out"])
    return [s["payload_buffer"], s["scale"], s["out"]]


def _full(s, W, n, bits):
    l = s["l"]
    for w in range(W):
        thc.rht_forward_full_deferred(s["grads"][w], l, s["seed"], s["ys"][w], s["absmax"][w:w + 1])
    thc.thc_scale_reduce(s["absmax"], W, 1, s["scale"])
    for w in range(W):
        thc.thc_full_encode_deferred(s["ys"][w], n, l, s["seed"], w, bits, s["scale"], s["payloads"][w])
    thc.thc_aggregate(s["payloads"], 1 << l, 14, bits, s["sums"])
    thc.thc_full_decode_inverse(s["sums"], s["scale"], W, n, l, s["seed"], bits, s["ys"][0], s["out"])
    return [s["absmax"], s["scale"], s["payload_buffer"], s["sums"], s["out"]]


def _topkc(s, W, C):
    P, J = s["P"], s["J"]
    for w in range(W):
        thc.topkc_chunk_norms(s["grads"][w], C, s["norms"][w * P:(w + 1) * P])
    thc.topkc_sum_norms(s["norms"], W, P, s["total"])
    thc.topkc_select(s["total"], J, s["indices"], s["ws"])
    thc.topkc_gather_sum(s["grads"], C, s["indices"], J, s["picked"])
    thc.topkc_scatter_mean(s["picked"], s["indices"], J, C, W, s["out"])
    return [s["norms"], s["total"], s["indices"], s["picked"], s["out"]]


def run(s):
    case = s["case"]
    path, W, n = case["path"], case["W"], case["n"]
    if path == "step":
        return _step(s, n, case["chunk_log2"], case["bits"])
    if path == "batch":
        return _batch(s, case["bits"])
    if path == "calls":
        return _calls(s, W, n, case["chunk_log2"], case["bits"])
    if path == "sat":
        return _sat(s, n, case["bits"])
    if path == "minmax":
        return _minmax(s, n, case["bits"], case["rotate"])
    if path == "full":
        return _full(s, W, n, case["bits"])
    return _topkc(s, W, case["C"])


# -------------------------------------------------------------------- what a pass must do
def work(case):
    """Every gradient read once, every payload written once and read once, the estimate (and the
    sums, where the caller asks for them) written once; flops: the butterflies, range and
    quantizer of every worker, the decoder's butterflies."""
    W, n, path = case["W"], case["n"], case["path"]
    grads = W * n * (2 if case["dtype"] == "bf16" else 4)
    if path == "topkc":
        C, J = case["C"], _topkc_count(case)
        P = (n + C - 1) // C
        share = J * C / n
        return {"bytes": grads * (1 + share) + (2 * W + 3) * 2.0 * P + 8.0 * J + 4.0 * J * C + 4.0 * n,
                "flops": 2.0 * W * n + W * J * C}
    bits = case["bits"]
    rotate = case.get("rotate", True)
    if path == "full":
        l = max(15, (n - 1).bit_length())
        size, ranges = 1 << l, 1
    else:
        l = case.get("chunk_log2", 14)
        ranges = (n + (1 << l) - 1) >> l
        size = ranges << l
    payload = size * bits / 8.0
    sum_bytes = 1 if W * ((1 << bits) - 1) <= 255 else 2
    total = grads + 2.0 * W * payload + 8.0 * ranges * (2 if path == "minmax" else 1) + 4.0 * n
    if path in ("calls", "full"):
        total += 2.0 * sum_bytes * size + 8.0 * W * ranges
    elif path == "step" and l != 14:
        total += float(sum_bytes) * size
    stages = l if rotate else 0
    return {"bytes": total, "flops": float(size) * (W * (stages + 5.0) + stages + 3.0)}


def tolerance(case):
    """Payloads, sums, indices and half-precision values are whole numbers or rounded once: the
    same in every correct implementation.  The estimate is a chain of l fp32 additions."""
    return {"rel": 1e-5}
