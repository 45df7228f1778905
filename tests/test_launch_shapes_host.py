"""Launches without a GPU, through a stand-in for the HIP calls of a launch (tests/fake_hip.cpp).  Grids
of the small-chunk encoder: what one call asks for depends neither on the calls before it nor on the
other devices of the process.  Full rotation: every plan finds its passes.  Each sequence of calls runs
in a process of its own, without PyTorch."""
import json
import os
import subprocess
import sys

import pytest

import paper_2407_01378_amd as thc
from paper_2407_01378_amd import binding

TESTS = os.path.dirname(os.path.abspath(__file__))

CHILD = """
import ctypes, json, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
lib.thc_encode_all_workspace_bytes.restype = ctypes.c_uint64
u64, vp = ctypes.c_uint64, ctypes.c_void_p
seen = []
for device, l, W, dtype, bits, n, *off in json.loads(sys.argv[3]):
    fake.fake_use(device)
    at = (vp * W)(*[0x10000 * (w + 1) for w in range(W)])   # (addresses that only a launch would use)
    need = lib.thc_encode_all_workspace_bytes(W, u64(n), l)
    before = fake.fake_queries()
    grads = (vp * W)(*[a + (off[0] if off else 0) for a in at])
    launches = fake.fake_launches()
    rc = lib.thc_encode_all(grads, dtype, W, u64(n), l, u64(1), bits, at, vp(0x1000), vp(0x2000), u64(need), None)
    seen.append([rc, fake.fake_grid(), fake.fake_block(), fake.fake_lds(), fake.fake_queries() - before,
                 fake.fake_launches() - launches])
print(json.dumps(seen))
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    thc.lib()
    fake = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    res = subprocess.run(["hipcc", "-O1", "-std=c++17", "-fPIC", "-shared", "-o", fake, os.path.join(TESTS, "fake_hip.cpp")],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-3000:]

    def calls(*sequence):
        res = subprocess.run([sys.executable, "-c", CHILD, fake, binding.LIB_PATH, json.dumps(sequence)],
                             stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
        assert res.returncode == 0, res.stderr[-3000:]
        return json.loads(res.stdout.splitlines()[-1])
    calls.fake = fake
    return calls


F32, BF16 = 0, 1
WIDE = (5, 1, F32, 4, 1 << 24)      # 8 waves and 84 KB: one workgroup per CU
NARROW = (9, 8, F32, 4, 1 << 24)    # 8 waves of the same kernel and 66 KB: two


def test_a_grid_does_not_depend_on_earlier_calls(run):
    first, second = run((0, *WIDE), (0, *NARROW))
    assert first == run((0, *WIDE))[0] and first[0] == 0 and first[1] == 256 and first[3] > 81920
    assert second[:4] == run((0, *NARROW))[0][:4] and second[1] == 512 and 65536 < second[3] < 81920
    back = run((0, *NARROW), (0, *WIDE))
    assert [b[:4] for b in back] == [second[:4], first[:4]]


def test_every_device_is_told_of_the_workgroups_beyond_64_kb(run):
    seen = run((0, *WIDE), (1, *WIDE), (0, *WIDE), (7, 13, 4, F32, 8, 1 << 22), (1, 13, 4, F32, 8, 1 << 22))
    assert [s[0] for s in seen] == [0] * 5
    assert seen[0][:4] == seen[1][:4] == seen[2][:4]


def test_answers_are_kept_per_shape_and_beyond_the_table(run):
    # more shapes of one kernel than the table has room for (devices count too), then the first ones again
    shapes = [(d, *s) for d in range(12) for s in (WIDE, NARROW, (6, 2, F32, 4, 1 << 24))]
    seen = run(*shapes, *shapes[:9])
    assert all(s[0] == 0 for s in seen)
    for k, s in enumerate(seen):
        assert s[:4] == seen[k % 3][:4]
    assert [s[4] for s in seen[:9]] == [1] * 9
    assert sum(s[4] for s in seen[-9:]) <= 4      # (what the overflow displaced is asked for again, no more)


def _spread_over(W, l, n, dtype, cus=256):
    """Workgroups that the workers of a chunk are spread over: 1 where one workgroup holds them or takes them in rounds."""
    waves = W << max(0, l - 11)
    if waves <= 16:
        return 1
    parts = -(-waves // 8)
    items = -(-(-(-n // (1 << l)) << l) // (1 << max(l, 11)))
    if parts == 3 and l <= 12 and 7 * cus < 8 * items <= 8 * cus:
        return 1
    rounds, spread = -(-items // cus), -(-items // (2 * cus // parts))
    return 1 if rounds * parts * (l + 4 * (dtype == F32)) < 14 * spread else parts


def test_workers_beyond_16_waves_are_spread_over_resident_workgroups_or_taken_in_rounds(run):
    calls = [(0, l, W, dtype, 4, n) for l in range(5, 14) for W in (1, 4, 5, 8, 9, 16, 17, 33, 64)
             for dtype in (F32, BF16) for n in (1, 350_000, 500_000, 5_000_000)]
    forms = set()
    for (_, l, W, dtype, _, n), (rc, grid, block, lds, _, launches) in zip(calls, run(*calls)):
        wpw = 1 << max(0, l - 11)
        parts = _spread_over(W, l, n, dtype)
        assert rc == 0 and launches == (2 if parts > 1 else 1), (l, W, dtype, n)    # (with the clearing of the words)
        items = -(-n // (1 << max(l, 11)))
        resident = 256 * min(2048 // block, 163840 // lds)   # as the stand-in has it
        if parts > 1:
            assert grid % parts == 0 and block == 64 * wpw * -(-W // parts) <= 512
            assert grid == min(items, resident // parts) * parts
            forms.add(("spread", l <= 9))
        elif W * wpw > 16:
            rounds = -(-W // (16 // wpw))
            assert block == 64 * wpw * -(-W // rounds) <= 1024 and grid == min(items, resident)
            forms.add(("rounds", l <= 9))
    assert {("spread", True), ("spread", False), ("rounds", True)} <= forms


@pytest.mark.parametrize("dtype,off", [(F32, 4), (BF16, 2)])
def test_gradients_off_the_16_byte_grid_take_the_generic_kernels(run, dtype, off):
    W, n = 3, 100_003
    for l in range(5, 14):
        on, generic = run((0, l, W, dtype, 4, n), (0, l, W, dtype, 4, n, off))
        assert on[0] == generic[0] == 0
        assert on[5] == 1
        # clear + W ranges + their maximum + W encoders, tiles of 2^14 coordinates
        assert generic[5] == 2 * W + 2 and generic[1:4] == [(n + (1 << 14) - 1) >> 14, 1024, 0]


AGREEING_CHILD = """
import ctypes, json, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
fake.fake_scarce(int(sys.argv[3]))
u64, vp = ctypes.c_uint64, ctypes.c_void_p
lib.thc_encode_all_workspace_bytes.restype = lib.thc_encode_all_minmax_workspace_bytes.restype = u64
seen = []
for W in (1, 2, 8, 16, 17, 32, 33, 48, 64):
    at = (vp * W)(*[0x10000 * (w + 1) for w in range(W)])   # (addresses that only a launch would use)
    for chunks in (1, 255 // W + 1, 512 // W, 512 // W + 1, 1024 // W, 1024 // W + 1, 6 * (1024 // W), 700):
        for n in ((chunks << 14), (chunks << 14) - 3):
            for dtype in (0, 1):
                for bits in (2, 4, 8):
                    need = lib.thc_encode_all_workspace_bytes(W, u64(n), 14)
                    rc = lib.thc_encode_all(at, dtype, W, u64(n), 14, u64(1), bits, at, vp(0x1000), vp(0x2000), u64(need), None)
                    seen.append(["one-pass", W, n, dtype, bits, rc, fake.fake_grid(), fake.fake_resident()])
                    need = lib.thc_encode_all_minmax_workspace_bytes(W, u64(n), 14)
                    for rotate in (0, 1):
                        rc = lib.thc_encode_all_minmax(at, dtype, W, u64(n), 14, u64(1), bits, rotate, at, vp(0x1000),
                                                       vp(0x2000), u64(need), None)
                        seen.append([f"min/max {rotate}", W, n, dtype, bits, rc, fake.fake_grid(), fake.fake_resident()])
print(json.dumps(seen))
"""


@pytest.mark.parametrize("scarce", [0, 2, 3])
def test_workgroups_that_wait_for_one_another_are_resident_in_the_kernel_launched(run, scarce):
    """A grid of them is at most what the device keeps of that very kernel, also where it keeps fewer of some
    instantiations than of others, and whole chunks per round."""
    res = subprocess.run([sys.executable, "-c", AGREEING_CHILD, run.fake, binding.LIB_PATH, str(scarce)],
                         stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert res.returncode == 0, res.stderr[-3000:]
    seen = json.loads(res.stdout.splitlines()[-1])
    for call in seen:
        what, W, n, dtype, bits, rc, grid, resident = call
        assert rc == 0, call
        assert 0 < grid <= resident and grid % W == 0, call


FULL_CHILD = """
import ctypes, json, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
u32, u64, vp = ctypes.c_uint32, ctypes.c_uint64, ctypes.c_void_p
x, y, m, p = vp(0x10000), vp(0x20000), vp(0x30000), vp(0x40000)
seen = []
def count(call):
    before = fake.fake_launches()
    rc = call()
    return [rc, fake.fake_launches() - before]
for l in range(15, 34):
    for n in (1, (1 << l) - 1):
        seen.append([l] + [count(c) for c in (
            lambda: lib.rht_forward_full(x, 0, u64(n), u32(l), u64(1), y, None),
            lambda: lib.rht_forward_full_deferred(x, 1, u64(n), u32(l), u64(1), y, m, None),
            lambda: lib.rht_inverse_full(y, u64(n), u32(l), u64(1), x, None),
            *[lambda b=b: lib.thc_full_encode_deferred(y, u64(n), u32(l), u64(1), u32(0), u32(b), m, p, None)
              for b in (2, 4, 8)])])
print(json.dumps(seen))
"""


def test_every_full_rotation_has_its_passes(run):
    res = subprocess.run([sys.executable, "-c", FULL_CHILD, run.fake, binding.LIB_PATH],
                         stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert res.returncode == 0, res.stderr[-3000:]
    seen = json.loads(res.stdout.splitlines()[-1])
    assert len(seen) == 38
    for l, forward, deferred, inverse, *encodes in seen:
        passes = 1 if l <= 25 else 2       # up to 11 stages each behind the 14 of the chunk kernels
        assert forward == deferred == inverse == [0, 1 + passes], l
        assert encodes == [[0, 1]] * 3, l
