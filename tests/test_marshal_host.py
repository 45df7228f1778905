"""The native marshalling of the binding, without a GPU: arguments of the plain form reach the
library (whose own argument checks answer before any HIP call), every other form is handed
back to the binding's checks, which raise."""
from types import SimpleNamespace

import pytest
import torch

import paper_2407_01378_amd as thc
from paper_2407_01378_amd import binding

NO_STREAM = SimpleNamespace(cuda_stream=0)
N = 40


def _f(n=N, dtype=torch.float32):
    return torch.zeros(n, dtype=dtype)


def _native():
    thc.lib()
    return binding._native


def _pieces(dtype=torch.bfloat16, W=3):
    return [_f(N, dtype) for _ in range(W)], [_f(1 << 14, torch.uint8) for _ in range(W)], _f(1), _f(4096, torch.uint8)


def test_plain_arguments_reach_the_library():
    g, p, scale, ws = _pieces()
    for fn in (thc.thc_encode_all, thc.thc_encode_all_cleared, thc.thc_sat_encode_all, thc.thc_sat_encode_all_cleared):
        with pytest.raises(thc.ThcError) as e:
            fn(g, 14, 0, 3, p, scale, ws, stream=NO_STREAM)
        assert e.value.status == -2
    for status, call in [
        (-3, lambda: thc.thc_chunk_absmax(_f(), 15, 0, _f(1), NO_STREAM)),
        (-2, lambda: thc.thc_encode(_f(), 14, 0, 0, 5, None, p[0], None, NO_STREAM)),
        (-2, lambda: thc.thc_aggregate(tuple(p), N, 14, 7, _f(1 << 14), NO_STREAM)),
        (-4, lambda: thc.thc_scale_reduce(_f(), 0, 1, scale, NO_STREAM)),
        (-2, lambda: thc.thc_decode(_f(), scale, 2, N, 14, 0, 1, _f(), NO_STREAM)),
        (-2, lambda: thc.thc_aggregate_decode(p, scale, N, 14, 0, 1, None, _f(), NO_STREAM)),
        (-2, lambda: thc.thc_sat_aggregate_decode(p, scale, N, 14, 0, 1, None, None, _f(), NO_STREAM)),
        (-3, lambda: thc.thc_encode_all_minmax(g, 13, 0, 4, True, p, _f(2), ws, NO_STREAM)),
        (-3, lambda: thc.thc_aggregate_decode_minmax(p, _f(2), N, 13, 0, 4, False, _f(), NO_STREAM)),
        (-3, lambda: thc.rht_forward_full_deferred(_f(), 14, 0, _f(1 << 14), _f(1), NO_STREAM)),
        (-3, lambda: thc.topkc_chunk_norms(_f(), 9, _f(8, torch.float16), NO_STREAM)),
        (-6, lambda: thc.topkc_select(_f(8, torch.float16), 9, _f(9, torch.int32), ws, NO_STREAM)),
        (-3, lambda: thc.thc_encode_all_batch([dict(n=N, grads=g, payloads=p, scale=scale)], 13, 4, ws, NO_STREAM)),
        (-3, lambda: thc.thc_aggregate_decode_batch([dict(n=N, payloads=p, scale=scale, out=_f())], 13, 4, ws, NO_STREAM)),
    ]:
        with pytest.raises(thc.ThcError) as e:
            call()
        assert e.value.status == status, e.value


def test_other_forms_are_handed_back():
    g, p, scale, ws = _pieces()
    m = _native()
    bad = [
        (g[:2] + [_f(N + 1, torch.bfloat16)], p), (g[:2] + [_f(N)], p),         # size, type of one worker
        ([x.double() for x in g], p), ([_f(2 * N)[::2]] * 3, p),                # dtype, stride
        (iter(g), p), (g, p[:2]), ([], []), (g + [None], p + p[:1]),            # not a list, lengths, not a tensor
        ([_f(N, torch.bfloat16)] * 65, [p[0]] * 65),
    ]
    for grads, payloads in bad:
        assert m.thc_encode_all(grads, 14, 0, 4, payloads, scale, ws, NO_STREAM) is None
    assert m.thc_encode_all(g, 14.0, 0, 4, p, scale, ws, NO_STREAM) is None
    assert m.thc_encode_all(g, 14, 0, 4, p, scale, ws, object()) is None
    assert m.thc_encode_all(g, 14, 0, 4, p, scale, ws) is None                  # argument count
    assert m.thc_encode_all_batch([dict(n=N, grads=g, payloads=p[:2])], 14, 4, ws, NO_STREAM) is None
    assert m.thc_encode_all_batch([dict(grads=g, payloads=p)], 14, 4, ws, NO_STREAM) is None
    with pytest.raises(ValueError):
        thc.thc_encode_all(g[:2] + [_f(N + 1, torch.bfloat16)], 14, 0, 4, p, scale, ws, NO_STREAM)
    with pytest.raises(TypeError):
        thc.thc_encode_all([x.double() for x in g], 14, 0, 4, p, scale, ws, NO_STREAM)
    with pytest.raises(ValueError):
        thc.rht_forward(_f(2 * N)[::2], 10, 0, _f(1024), NO_STREAM)
    with pytest.raises(TypeError):
        thc.topkc_chunk_norms(_f(), 8, _f(8), NO_STREAM)


class _AnswersInPython(torch.Tensor):
    """A tensor whose sizes are asked for in Python, where the answer is an error."""

    @staticmethod
    def __new__(cls, n):
        return torch.Tensor._make_wrapper_subclass(cls, (n,), dtype=torch.float32,
                                                   dispatch_sizes_strides_policy="sizes")

    @classmethod
    def __torch_dispatch__(cls, func, types, args=(), kwargs=None):
        raise KeyError("no answer")


def test_errors_of_the_arguments_reach_the_caller():
    """An argument that raises when it is looked at: its error, before anything is launched."""
    g, p = [_f(0), _f(0)], [_f(16, torch.uint8) for _ in range(2)]   # (no coordinates: a call would do nothing)
    ws = _f(4096, torch.uint8)
    with pytest.raises(RuntimeError, match="ambiguous"):
        thc.thc_encode_all_minmax(g, 14, 0, 4, torch.ones(2), p, _f(2), ws, NO_STREAM)
    with pytest.raises(RuntimeError, match="ambiguous"):
        thc.thc_aggregate_decode_minmax(p, _f(2), 0, 14, 0, 4, torch.ones(2), _f(0), NO_STREAM)
    with pytest.raises(KeyError, match="no answer"):
        thc.rht_forward(_AnswersInPython(8), 10, 0, _f(1024), NO_STREAM)
    m = _native()
    assert m.thc_encode_all_minmax(g, 14, 0, 4, torch.ones(2), p, _f(2), ws, NO_STREAM) is None
    assert m.rht_forward(_AnswersInPython(8), 10, 0, _f(1024), NO_STREAM) is None
    assert m.thc_encode_all_minmax(g, 14, 0, 4, torch.ones(1), p, _f(2), ws, NO_STREAM) == 0


def test_buckets_are_checked_as_the_binding_checks_them():
    g, p, ws = [_f(0), _f(0)], [_f(16, torch.uint8) for _ in range(2)], _f(4096, torch.uint8)

    def bucket(**other):
        return [dict(dict(n=0, seed=0, grads=g, payloads=p, scale=_f(1), out=_f(0)), **other)]

    thc.thc_encode_all_batch(bucket(), 14, 4, ws, NO_STREAM)
    thc.thc_aggregate_decode_batch(bucket(grads=None), 14, 4, ws, NO_STREAM)
    for fn in (thc.thc_encode_all_batch, thc.thc_aggregate_decode_batch):
        with pytest.raises(TypeError):
            fn(bucket(seed=None), 14, 4, ws, NO_STREAM)
        with pytest.raises(TypeError):
            fn(bucket(n=None), 14, 4, ws, NO_STREAM)
        with pytest.raises(AttributeError):
            fn(bucket(grads=[1, 2]), 14, 4, ws, NO_STREAM)
        with pytest.raises(AttributeError):
            fn(bucket(scale=1), 14, 4, ws, NO_STREAM)


def test_lists_shorter_than_the_workers_are_refused():
    """The library reads as many pointers as there are workers: a shorter list may not reach it.  (bits
    = 3, so that a call that does get through ends at the library's argument checks.)"""
    g, p, scale, ws = _pieces()
    for fn in (thc.thc_encode_all, thc.thc_encode_all_cleared, thc.thc_sat_encode_all, thc.thc_sat_encode_all_cleared):
        with pytest.raises(ValueError, match="3 workers"):
            fn(g, 14, 0, 3, p[:2], scale, ws, stream=NO_STREAM)
    with pytest.raises(ValueError, match="3 workers"):
        thc.thc_encode_all_static(g, 14, 0, 3, p[:2], scale, None, NO_STREAM)
    with pytest.raises(ValueError, match="3 workers"):
        thc.thc_encode_all_minmax(g, 14, 0, 3, True, [], _f(2), ws, NO_STREAM)
    whole = dict(n=N, grads=g, payloads=p, scale=scale, out=_f())
    for short in (dict(whole, payloads=p[:2]), dict(whole, grads=g[:2])):
        with pytest.raises(ValueError, match="3 workers"):
            thc.thc_encode_all_batch([whole, short], 14, 3, ws, NO_STREAM)
    with pytest.raises(ValueError, match="3 workers"):
        thc.thc_aggregate_decode_batch([whole, dict(whole, payloads=p[:2])], 14, 3, ws, NO_STREAM)
    # longer lists, lists that are not read and buckets without coordinates pass on
    for call in (lambda: thc.thc_encode_all(g[:2], 14, 0, 3, p, scale, ws, NO_STREAM),
                 lambda: thc.thc_encode_all_batch([whole, dict(whole, n=0, grads=[], payloads=[])], 14, 3, ws, NO_STREAM),
                 lambda: thc.thc_aggregate_decode_batch([whole, dict(whole, grads=g[:1])], 14, 3, ws, NO_STREAM)):
        with pytest.raises(thc.ThcError) as e:
            call()
        assert e.value.status == -2
