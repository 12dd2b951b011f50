"""The claim of summarize's hash table under every order of its memory
operations (CPU).

Key spaces past 16,384 keys take their slots from an LDS hash table. When the
slots run out, a thread may drop its event only if its key gets no slot in
this pass: a key with a slot is written out and not looked at again. The probe
runs the kernel's own function on host memory, several threads as coroutines,
and counts the schedules after which an event would be lost.
"""
import ctypes
import os

import pytest

PROBE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "probe", "libhashclaimprobe.so")
SLOTS = 4


def _bucket(key):
    return (key * 0x9E3779B1 & 0xFFFFFFFF) >> 21


def _play(keys, used, random=0, seed=0):
    if not os.path.exists(PROBE):
        import tests.probe.build
        tests.probe.build.build()
    L = ctypes.CDLL(PROBE)
    L.probe_hash_claim.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_int64, ctypes.c_uint32,
                                   ctypes.c_void_p]
    out = (ctypes.c_int64 * 2)()
    assert L.probe_hash_claim((ctypes.c_int32 * len(keys))(*keys), len(keys), used, random, seed, out) == 0
    return out[0], out[1]


K = 100
SAME_BUCKET = next(k for k in range(K + 1, 65536) if _bucket(k) == _bucket(K))


@pytest.mark.parametrize("used", range(SLOTS + 1))
@pytest.mark.parametrize("keys", [(K, K), (K, SAME_BUCKET), (K, K + 1)], ids=["one key", "one bucket", "two keys"])
def test_two_threads_in_every_order(keys, used):
    played, lost = _play(keys, used)
    assert played > 100 and lost == 0, (played, lost)


@pytest.mark.parametrize("used", range(SLOTS + 1))
@pytest.mark.parametrize("keys", [(K, K, K), (K, K, SAME_BUCKET), (K, K, K + 1, K + 1), (K, K, SAME_BUCKET, K + 1)])
def test_more_threads_in_random_orders(keys, used):
    played, lost = _play(keys, used, random=100_000, seed=7)
    assert played > 10_000 and lost == 0, (played, lost)
