"""GPU parity of argus_l2 (section 6.1 routing; Appendix B, Eq. 5) through
the C ABI against the CPU oracle.

Group sizes, CV classes, straggler flags and counts must match exactly (both
sides decide them with exact integer comparisons); mean, std and CV (double)
and z (float) within 1e-5 relative. Cases: closed-form outlier groups, CV
boundaries, identical and all-zero groups, routing / membership / domain
rules with malformed and duplicate listings, random groups over ragged event
counts up to 65,536 ranks, the medium trace through the GPU chain
summarize -> l2, group sizes and means at the kernels' limits, sparse
listings, small and large groups of one dimension, and few ranks. The full-size workloads are checked in test_gpu_full.py.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_20374_amd as pa
import tracegen
from tests import parity as P

pytestmark = pytest.mark.gpu
DEV = "cuda"
STATUS_BITS = {1: pa.argus.DEV_GROUPS_MALFORMED, 2: pa.argus.DEV_GROUPS_DUPLICATE, 4: pa.argus.DEV_L2_DOMAIN}


def _announce(name):
    print(f"\n[gpu-case] {name}", flush=True)


def _t(x, dt):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(x, dtype=dt))).to(DEV)


def assert_l2_equal(g: dict, o: dict, what: str):
    P.assert_int_equal(g, o, P.L2_INT_FIELDS, what)
    P.assert_float_close(g, o, P.L2_FLOAT_FIELDS, what)


def _both(cnt, sm, R, S, E, route, off, mem, what, **params):
    g = pa.l2(_t(np.asarray(cnt, np.uint32).view(np.int32), np.int32), _t(sm, np.int64), R, S, E, _t(route, np.uint8),
              _t(off, np.int32), _t(mem, np.int32), **params)
    torch.cuda.synchronize()
    o = oracle.l2(cnt, sm, R, S, E, route, off, mem, **params)
    assert_l2_equal(g, o, what)
    expect = sum(v for k, v in STATUS_BITS.items() if o["status"] & k)
    assert int(g["dev_status"].item()) == expect, (what, int(g["dev_status"].item()), o["status"])
    return g, o


def _one_group(xs, what, **params):
    R = len(xs)
    return _both(np.ones(R, np.uint32), np.asarray(xs, np.int64), R, 1, 1, np.zeros(1, np.uint8),
                 np.array([[0, R]], np.int32), np.arange(R, dtype=np.int32).reshape(1, R), what, **params)


def test_l2_hand_built_groups():
    _announce("l2 hand-built groups")
    for n in (3, 10, 11, 40):
        xs = [10_000] * n
        xs[n // 3] = 13_000
        g, _ = _one_group(xs, f"outlier n={n}")
        assert bool(P.to_np(g["flags"])[n // 3] & 2) == (n >= 11)
    for d in (99, 100, 249, 250):
        _one_group([5000 - d, 5000, 5000 + d], f"cv boundary d={d}")
    _one_group([7000] * 6, "identical")
    _one_group([0] * 4, "zeros")
    _one_group([2**40 - 1, 2**40 - 2, 3, 2**39], "near the domain edge")
    _one_group([5, 2**41, 6, 7], "out of the domain")


def test_l2_routing_membership_and_domain():
    _announce("l2 routing, membership, domain")
    R, S, E = 6, 2, 3
    cnt = np.ones(R * S * E, np.uint32)
    sm = np.full(R * S * E, 5000, np.int64)
    sm[((1 * S + 0) * E + 1)] = 9000
    cnt[((2 * S + 1) * E + 1)] = 0
    sm[((3 * S + 1) * E + 1)] = 1 << 41
    route = np.array([0xFF, 0, 1], np.uint8)
    off = np.array([[0, 3, 6], [0, 6, 6]], np.int32)
    mem = np.array([[0, 1, 2, 3, 4, 5], [0, 1, 2, 3, 2, 5]], np.int32)
    _both(cnt, sm, R, S, E, route, off, mem, "duplicate + domain", min_group=2)
    off2 = np.array([[0, 4, 2], [0, 6, 6]], np.int32)
    mem2 = np.array([[0, 1, 9, 3, 4, 5], [0, 1, 2, 3, 4, 5]], np.int32)
    _both(cnt, sm, R, S, E, route, off2, mem2, "malformed", min_group=2)
    off3 = np.array([[-1, 3, 7], [0, 6, 6]], np.int32)
    _both(cnt, sm, R, S, E, np.array([7, 0, 2], np.uint8), off3, mem2, "bad ranges and routes", min_group=2)


@pytest.mark.parametrize("R,S,E,seed", [(5, 2, 7, 0), (64, 3, 65, 1), (300, 1, 130, 2), (4099, 2, 33, 3),
                                        (65536, 1, 3, 4)])
def test_l2_random_groups(R, S, E, seed):
    _announce(f"l2 random groups R={R} S={S} E={E}")
    rng = np.random.default_rng(seed)
    cnt = rng.integers(0, 5, size=R * S * E).astype(np.uint32)
    base = rng.integers(1000, 10**8, size=E)
    slow = np.where(rng.random(R) < 0.02, rng.uniform(1.1, 1.6, size=R), 1.0)
    r_of = np.arange(R * S * E) // (S * E)
    xs = (base[np.arange(R * S * E) % E] * slow[r_of] * rng.uniform(0.97, 1.03, size=R * S * E)).astype(np.int64)
    sm = xs * cnt.astype(np.int64)
    n_dims, G = 3, max(2, R // 16)
    off = np.zeros((n_dims, G + 1), np.int32)
    mem = np.zeros((n_dims, R), np.int32)
    for d in range(n_dims):
        mem[d] = rng.permutation(R)
        off[d, 1:G] = np.sort(rng.integers(0, R + 1, size=G - 1))
        off[d, G] = R
    mem[2, :3] = mem[2, R - 3:]  # duplicate listings
    route = rng.integers(0, n_dims + 1, size=E).astype(np.uint8)
    route[route == n_dims] = 0xFF
    _both(cnt, sm, R, S, E, route, off, mem, f"random {R}x{S}x{E}", min_group=int(rng.integers(2, 5)),
          cv_mild_pm=int(rng.integers(5, 40)), cv_severe_pm=int(rng.integers(40, 120)),
          z_pm=int(rng.integers(1500, 3500)))


def test_l2_medium_chain():
    _announce("l2 medium trace: GPU summarize -> l2")
    t = tracegen.make("medium")
    c = t.cfg
    R, S, K, NS = c.n_ranks, c.n_steps, c.n_kernels, c.n_streams
    route, off, mem = tracegen.workload_groups("medium", R, K)
    s = pa.summarize(t.fill_device(device=DEV), R, S, K, NS)
    g = pa.l2(s["count"], s["sum_ns"], R, S, K, _t(route, np.uint8), _t(off, np.int32), _t(mem, np.int32))
    torch.cuda.synchronize()
    assert int(g["dev_status"].item()) == 0
    so = P.oracle_summary_sharded(t)
    o = oracle.l2(so["count"], so["sum_ns"], R, S, K, route, off, mem)
    assert_l2_equal(g, o, "medium chain")


@pytest.mark.parametrize("size,E,scale", [(7, 2049, 1), (8, 2047, 1), (9, 65, 1), (24, 130, 1), (25, 64, 1),
                                          (32, 513, 1), (33, 300, 1), (191, 70, 1), (193, 1, 1), (512, 3, 1),
                                          (8, 65, 2**13), (40, 65, 2**13), (200, 9, 2**13)])
def test_l2_group_size_edges(size, E, scale):
    """Groups of one size, every listing valid: sizes around the batch (8), the
    means kept between the passes (24 to a wavefront), the small / large
    boundary (32) and eight wavefronts' keep (192); event counts around the
    64-lane and 2,048-id tiles; scale 2^13 puts the means of some members
    beyond 2^32 ns and some sums beyond 2^53 (the wide arithmetic) next to
    narrow ones. Sparse listings and mixed sizes have tests of their own below."""
    _announce(f"l2 group size {size}, {E} events, scale {scale}")
    rng = np.random.default_rng(size * 7919 + E)
    G = 11  # more groups than one workgroup's wavefronts
    R, S = size * G, 2
    cnt = rng.integers(0, 4, size=R * S * E).astype(np.uint32)
    xs = rng.integers(10**5, 10**6, size=R * S * E) * rng.integers(1, 1 + scale, size=R * S * E)
    cnt[xs > 2**32] *= np.uint32(2**21)
    sm = xs * cnt.astype(np.int64) + rng.integers(0, 3, size=R * S * E) * (cnt > 3)
    route = rng.integers(0, 3, size=E).astype(np.uint8)
    off = np.tile(np.arange(G + 1, dtype=np.int32) * size, (2, 1))
    mem = np.stack([rng.permutation(R), np.arange(R)]).astype(np.int32)
    _both(cnt, sm, R, S, E, route, off, mem, f"size {size} E {E} scale {scale}", z_pm=1500)


@pytest.mark.parametrize("size", [3, 12, 40])
@pytest.mark.parametrize("mean", [2**32 - 2, 2**32 - 1, 2**32])
def test_l2_means_around_32_bits(size, mean):
    """A member's mean at the largest 32-bit values and one past them, in small
    and large groups, as the one outlier (a straggler from 12 members on) and
    as every member's."""
    _announce(f"l2 mean {mean} in a group of {size}")
    xs = 1000 + np.arange(size, dtype=np.int64)
    xs[size // 2] = mean
    g, _ = _one_group(xs, f"one member at {mean}")
    assert int(P.to_np(g["flags"])[size // 2]) == (3 if size > 11 else 1)
    _one_group(np.full(size, mean, np.int64), f"all members at {mean}")


@pytest.mark.parametrize("filler", ["invalid", "duplicate"])
@pytest.mark.parametrize("listings,valid", [(600, 1), (600, 10), (1024, 5), (1024, 20), (2100, 13), (4096, 9)])
def test_l2_sparse_listings(listings, valid, filler):
    """A group of many listings of which few count: the rest are ids that are
    skipped or second listings. A wavefront's share (an eighth) spans several
    of its 64-listing chunks, each with a few members that count, which fit
    what it keeps between its two passes."""
    _announce(f"l2 {listings} listings, {valid} valid per share, filler {filler}")
    rng = np.random.default_rng(listings * 31 + valid)
    R, S, E = listings, 1, 70
    mem = np.full(R, -1, np.int32)
    ids = rng.permutation(R)
    n = 0
    for w in range(8):
        lo, hi = R * w // 8, R * (w + 1) // 8
        for i in np.sort(rng.choice(np.arange(lo, hi), size=valid, replace=False)):
            mem[i] = ids[n]
            n += 1
    if filler == "duplicate":
        mem[mem < 0] = mem[mem >= 0][0]
    cnt = rng.integers(0, 4, size=R * S * E).astype(np.uint32)
    sm = rng.integers(10**5, 10**6, size=R * S * E) * cnt.astype(np.int64)
    _both(cnt, sm, R, S, E, np.zeros(E, np.uint8), np.array([[0, R]], np.int32), mem.reshape(1, R),
          f"{listings} listings, {valid} valid, {filler}", z_pm=1500)


@pytest.mark.parametrize("n,x", [(12, 2**40 - 3), (21831, 949394193386), (54702, 1073001553514)])
def test_l2_equal_members_have_positive_zero(n, x):
    """Equal members have std 0 and z = +0, also where the sum passes 2^53 and
    the double mean rounds to one side of them."""
    _announce(f"l2 {n} equal members of {x}")
    g, _ = _one_group(np.full(n, x, np.int64), f"{n} x {x}")
    z = P.to_np(g["z"])
    assert not z.any() and not np.signbit(z).any()


@pytest.mark.parametrize("E", [1100, 2048, 4100])
def test_l2_mixed_sizes_one_dimension(E):
    """Small and large groups side by side in a span of eight, and so many
    events of one dimension among 2,048 ids that a workgroup takes several
    shares of 64 of them one after another."""
    _announce(f"l2 mixed group sizes, {E} events of one dimension")
    rng = np.random.default_rng(E)
    sizes = [8, 40, 200, 3, 33, 1, 64, 5, 32, 100, 2, 48, 6, 7, 90, 12, 34]
    R, S = sum(sizes), 1
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32).reshape(1, -1)
    cnt = rng.integers(0, 4, size=R * S * E).astype(np.uint32)
    sm = rng.integers(10**5, 10**6, size=R * S * E) * cnt.astype(np.int64)
    _both(cnt, sm, R, S, E, np.zeros(E, np.uint8), off, rng.permutation(R).astype(np.int32).reshape(1, R),
          f"mixed sizes, E {E}", z_pm=1500)


@pytest.mark.parametrize("R,S,E", [(8, 3, 64), (31, 2, 65), (32, 5, 130), (32, 1, 2049), (33, 5, 130), (40, 2, 1),
                                   (70, 200, 700), (150, 130, 100)])
def test_l2_few_ranks_and_many_steps(R, S, E):
    """Rank counts around the one (32) up to which every group has wavefronts
    of its own, and steps and events at which a workgroup takes several
    shares of a tile in turn; mixed group sizes with second and invalid
    listings, absent cells, unrouted events and means out of the domain."""
    _announce(f"l2 R={R} S={S} E={E}")
    rng = np.random.default_rng(R * 1009 + S * 31 + E)
    cnt = rng.integers(0, 4, size=R * S * E).astype(np.uint32)
    xs = rng.integers(10**5, 10**6, size=R * S * E)
    xs[rng.integers(0, R * S * E, size=3)] = 2**40 + 5
    D, G = 3, max(2, R // 5)
    off, mem = np.zeros((D, G + 1), np.int32), np.zeros((D, R), np.int32)
    for d in range(D):
        off[d, 1:G] = np.sort(rng.integers(0, R + 1, size=G - 1)) if d else np.minimum(np.arange(1, G), R)
        off[d, G] = R
        mem[d] = rng.permutation(R)
    mem[1, R // 2] = mem[1, 0]
    mem[2, 0] = -1
    route = rng.choice([0, 1, 1, 2, 0xFF], size=E).astype(np.uint8)
    _both(cnt, xs * cnt.astype(np.int64), R, S, E, route, off, mem, f"few ranks {R}x{S}x{E}", z_pm=1500)
