"""GPU parity of argus_summarize_keyed and argus_compact through the C ABI
against the CPU oracle: every keyed summary field and every byte of the
record stream must match exactly, with identical segment offsets.

Cases: random events whose kernels run on several streams (with invalid
records), key spaces in the dense and the mapped (two passes) layout, the
tiny trace with re-drawn streams, the record stream of both keyings,
truncation at a short capacity and sizing at capacity 0, cell counts and
record sizes at the kernel's limits, and full-size
production and cluster summaries compacted in the launch configuration the
benchmark times.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2606_20374_amd as pa
import tracegen
from tests import parity as P

pytestmark = pytest.mark.gpu
DEV = "cuda"
SUM_FIELDS = ["count", "sum_ns", "min_ns", "max_ns", "hist", "n_valid", "n_invalid", "t_first", "t_last", "step_ns",
              "busy_ns", "stream_busy_ns", "wire_bytes"]


def _announce(name):
    print(f"\n[gpu-case] {name}", flush=True)


def _dev(ev):
    return {k: torch.from_numpy(np.ascontiguousarray(v)).to(DEV) for k, v in ev.items()}


def _random_events(rng, G, K, NS, n_per, p_bad=0.02):
    lens = rng.integers(0, n_per, size=G)
    off = np.zeros(G + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    n = int(off[-1])
    kid = rng.integers(0, K, size=n).astype(np.int32)
    st = rng.integers(0, NS, size=n).astype(np.int32)
    bad = rng.random(n) < p_bad
    kid[bad] = -3
    t0 = rng.integers(0, 10**13, size=n).astype(np.int64)
    t1 = t0 + (2.0 ** rng.uniform(0, 36, size=n)).astype(np.int64)
    return {"kernel_id": kid, "stream": st, "start_ns": t0, "end_ns": t1, "seg_off": off}


def _keyed_both(ev, R, S, K, NS, what):
    s = pa.summarize(_dev(ev), R, S, K, NS, keyed=True)
    torch.cuda.synchronize()
    o = oracle.summarize(ev, K, NS, keyed=True)
    P.assert_int_equal(s, o, SUM_FIELDS, what)
    assert int(s["dev_status"].item()) == 0
    return s, o


def _compact_both(s, o, G, C, NS, what, cap=None):
    g = pa.compact(s, G, 1, C, NS, capacity=cap)
    torch.cuda.synchronize()
    ob, ooff = oracle.compact(o, G, C, NS, cap=cap)
    assert np.array_equal(g["seg_byte_off"].cpu().numpy(), ooff), what
    total = int(ooff[-1])
    gb = g["bytes"].cpu().numpy()
    n = len(ob)
    if cap is None or cap >= total:
        assert n == total and np.array_equal(gb[:total], ob), what
        assert int(g["dev_status"].item()) == 0
    else:
        # both write the records that fit entirely: compare the written prefix
        last = int(ooff[np.searchsorted(ooff, cap, side="right") - 1])
        assert np.array_equal(gb[:last], ob[:last]), what
        assert int(g["dev_status"].item()) == pa.argus.DEV_COMPACT_CAPACITY
    return g


@pytest.mark.parametrize("G,K,NS,seed", [(6, 7, 3, 0), (5, 64, 32, 1), (3, 1000, 16, 2), (2, 2048, 16, 3)])
def test_keyed_random(G, K, NS, seed):
    _announce(f"keyed summarize random G={G} K={K} NS={NS}")
    rng = np.random.default_rng(seed)
    ev = _random_events(rng, G, K, NS, 30_000)
    s, o = _keyed_both(ev, G, 1, K, NS, f"keyed {G}x{K}x{NS}")
    _compact_both(s, o, G, K * NS, NS, "compact keyed")


def test_keyed_tiny_with_redrawn_streams():
    _announce("keyed summarize: tiny trace, streams redrawn per event")
    t = tracegen.make("tiny")
    c = t.cfg
    ev = t.fill_host()
    rng = np.random.default_rng(9)
    ev["stream"] = ((ev["kernel_id"] + rng.integers(0, 3, size=len(ev["stream"]))) % c.n_streams).astype(np.int32)
    s, o = _keyed_both(ev, c.n_ranks, c.n_steps, c.n_kernels, c.n_streams, "tiny keyed")
    _compact_both(s, o, c.n_segments, c.n_kernels * c.n_streams, c.n_streams, "tiny keyed compact")


def test_compact_kernel_keys_capacity_and_sizing():
    _announce("compact: kernel-id keys, capacity cut, sizing only")
    t = tracegen.make("tiny")
    c = t.cfg
    G, K, NS = c.n_segments, c.n_kernels, c.n_streams
    ev = t.fill_host()
    s = pa.summarize(_dev(ev), c.n_ranks, c.n_steps, K, NS)
    o = oracle.summarize(ev, K, NS)
    g = _compact_both(s, o, G, K, 0, "tiny compact")
    total = int(g["seg_byte_off"][-1].item())
    assert np.array_equal(np.diff(g["seg_byte_off"].cpu().numpy()), o["wire_bytes"])
    for cap in (1, 100, total // 3 + 5, total - 1):
        _compact_both(s, o, G, K, 0, f"cap {cap}", cap=cap)
    # capacity 0 sizes the stream and writes nothing
    off = torch.empty(G + 1, dtype=torch.int64, device=DEV)
    st = torch.empty(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(8 * G, dtype=torch.uint8, device=DEV)
    sm = pa.argus.Summary(*[s[f].data_ptr() if f in ("count", "sum_ns", "min_ns", "max_ns", "hist") else None
                            for f in pa.argus.SUMMARY_FIELDS])
    rc = pa.lib().argus_compact(ctypes.byref(sm), G, 1, K, 0, None, 0, off.data_ptr(), st.data_ptr(), ws.data_ptr(),
                                ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and int(off[-1].item()) == total
    assert int(st.item()) == (pa.argus.DEV_COMPACT_CAPACITY if total > 0 else 0)


@pytest.mark.parametrize("G,C,fill", [(1, 1, 0.9), (9, 63, 0.5), (70, 64, 1.0), (300, 65, 0.02), (17, 256, 0.7),
                                      (5, 511, 1.0), (8, 512, 0.3), (9, 513, 0.9), (3, 1024, 1.0), (70, 1025, 0.05),
                                      (4, 2048, 1.0), (3, 5000, 0.6), (130, 3, 0.0)])
@pytest.mark.parametrize("bins", [2, 32])
def test_compact_cell_counts_and_full_records(G, C, fill, bins):
    """Cell counts around a wavefront's window and the sizes at which segments
    change from a wavefront to a workgroup each, segment counts past one
    look-back window, empty segments, records of every octave bin (more bytes
    than a wavefront stages, so the rest is read again), every alignment of
    the caller's buffer, and capacities that cut inside a record."""
    _announce(f"compact G={G} C={C} fill={fill} bins={bins}")
    rng = np.random.default_rng(G * 10_007 + C * 31 + bins)
    n = G * C
    cnt = np.where(rng.random(n) < fill, rng.integers(1, 2**32, n), 0).astype(np.uint32)
    cnt[rng.integers(0, n)] = 0
    hist = rng.integers(1, 2**32, size=(n, 32)).astype(np.uint32)
    hist[rng.random((n, 32)) >= (1.0 if bins == 32 else bins / 32)] = 0
    f = lambda: rng.integers(-2**62, 2**62, n)  # noqa: E731
    o = {"count": cnt, "sum_ns": f(), "min_ns": f(), "max_ns": f(), "hist": hist.reshape(-1)}
    s = {k: torch.from_numpy(v.view(np.int32) if v.dtype == np.uint32 else v).to(DEV) for k, v in o.items()}
    _compact_both(s, o, G, C, 0, "sized")
    ob, ooff = oracle.compact(o, G, C, 0)
    total = int(ooff[-1])
    for skew, cap in ((1, total), (2, total + 3), (3, max(total - 1, 0)), (7, total // 2), (0, min(total, 20))):
        buf = torch.full((total + 64,), 0xA5, dtype=torch.uint8, device=DEV)
        g = pa.compact(s, G, 1, C, 0, capacity=cap, out=buf[skew:])
        torch.cuda.synchronize()
        assert np.array_equal(g["seg_byte_off"].cpu().numpy(), ooff)
        want, end = np.full(total + 64, 0xA5, np.uint8), 0
        while end < total and end + 33 + 5 * int(ob[end + 32]) <= cap:
            end += 33 + 5 * int(ob[end + 32])
        want[skew:skew + end] = ob[:end]
        assert np.array_equal(buf.cpu().numpy(), want), (skew, cap)
        assert int(g["dev_status"].item()) == (pa.argus.DEV_COMPACT_CAPACITY if cap < total else 0)


@pytest.mark.parametrize("name", ["production", "cluster"])
def test_compact_full_size(name):
    _announce(f"compact full size {name}")
    t = tracegen.make(name)
    c = t.cfg
    R, S, K, NS = c.n_ranks, c.n_steps, c.n_kernels, c.n_streams
    G = c.n_segments
    s = pa.summarize(t.fill_device(device=DEV), R, S, K, NS)
    g = pa.compact(s, R, S, K, 0)
    torch.cuda.synchronize()
    assert int(g["dev_status"].item()) == 0
    goff = g["seg_byte_off"].cpu().numpy()
    gbytes = g["bytes"]
    del s
    torch.cuda.empty_cache()
    # sampled segments: each regenerated and summarized by the oracle, its
    # records compared byte for byte at the GPU's offset
    rng = np.random.default_rng(1)
    segs = sorted(rng.choice(G, size=min(G, 48), replace=False).tolist()) + [G - 1]
    for seg in segs:
        ev = t.fill_host(seg, seg + 1)
        o = oracle.summarize(ev, K, NS)
        ob, ooff = oracle.compact(o, 1, K, 0)
        assert goff[seg + 1] - goff[seg] == ooff[1], (name, seg)
        got = gbytes[goff[seg]:goff[seg + 1]].cpu().numpy()
        assert np.array_equal(got, ob), (name, seg)
    raw = 24 * c.events_per_seg
    print(f"[gpu-case] {name}: {goff[-1] / G:.0f} B per rank-step vs {raw} B raw ({raw * G / goff[-1]:.0f}x)",
          flush=True)


@pytest.mark.parametrize("G,C,fill", [(1030, 100, 0.8), (2050, 130, 0.6), (1100, 129, 0.9), (2100, 300, 0.5),
                                      (600, 400, 0.9), (1030, 513, 0.3), (4100, 70, 0.7), (33, 129, 1.0)])
def test_compact_segments_shared_by_wavefronts(G, C, fill):
    """Segment counts at which one, two, four and eight wavefronts share a
    segment, with shares that don't divide the cells and a last workgroup that
    is not full."""
    test_compact_cell_counts_and_full_records(G, C, fill, 6)
