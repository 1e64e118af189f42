"""Parity of the trace-preparation steps with the oracle where their launches change: one
workgroup's sort against passes of tiles, two, three or four digits of the pairing's hash (many
distinct addresses, so that unequal ones share it), offsets checked by one workgroup or several,
traces past the range of the packed key, tile counts added up or scanned."""
import numpy as np
import pytest

import oracle
from gpu_util import log
from test_gpu_prep import _gpu, check_attribute, check_lifecycles, check_orchestrate, random_blocks  # noqa: F401

pytestmark = pytest.mark.gpu


def raw_of(n, n_addr, seed, stride=512):
    rng = np.random.default_rng(seed)
    raw = np.zeros(n, oracle.RAW_DTYPE)
    raw["ts"] = np.cumsum(rng.integers(0, 4, n))
    raw["addr"] = (rng.integers(0, n_addr, n) * stride + 0x7F0000000000).astype(np.uint64)
    raw["bytes"] = rng.choice([1, -1, 0], n, p=[0.5, 0.46, 0.04]) * rng.integers(1, 1 << 30, n)
    return raw


@pytest.mark.parametrize("n", [1, 63, 4095, 4096, 4097, 8191, 8192, 8193, (1 << 20) - 1, (1 << 20) + 1])
def test_lifecycles_sizes(n):
    cut = n // 3
    check_lifecycles(raw_of(n, max(n // 3, 1), n), np.array([0, cut, cut, n]), what=f"{n} events, many addresses")


def test_lifecycles_many_tiles():
    n = (4096 << 10) + 5  # one tile more than its counts are added up for
    check_lifecycles(raw_of(n, n // 4, 5), np.array([0, n]), what="over 1,024 tiles")


@pytest.mark.parametrize("n_traces", [16384, 16385, 40000])
def test_many_short_traces(n_traces):
    """Offsets checked by one workgroup and by several; traces from 2^15 on have mixed keys."""
    rng = np.random.default_rng(n_traces)
    lens = rng.integers(0, 6, n_traces)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    check_lifecycles(raw_of(int(off[-1]), 3, n_traces), off, what=f"{n_traces} traces")
    check_orchestrate(*random_blocks(n_traces, n_traces, 4), what=f"{n_traces} traces")


@pytest.mark.parametrize("blocks", [1, 2047, 2048, 2049, 4095, 4096, 4097])
@pytest.mark.parametrize("scale_bits", [0, 34, 41])
def test_orchestrate_sizes(blocks, scale_bits):
    """Around one workgroup's sort (8,192 records), by the joint key and by rank, time and trace apart."""
    b, boff, st, soff, zg, zoff = random_blocks(blocks + scale_bits, 1, 2)
    rng = np.random.default_rng(blocks)
    b = np.zeros(blocks, oracle.BLOCK_DTYPE)
    s = np.int64(1) << np.int64(scale_bits)
    b["size"], b["category"] = rng.integers(1, 1 << 30, blocks), rng.integers(0, 5, blocks)
    b["t_alloc"] = np.sort(rng.integers(-1000, 1 << 20, blocks)) * s
    b["t_free"] = np.where(rng.random(blocks) < 0.1, oracle.PERSISTENT, b["t_alloc"] + rng.integers(0, 300, blocks) * s)
    cut = blocks // 2
    check_orchestrate(b, np.array([0, cut, blocks]), np.arange(0, 50) * 20000 * s, np.array([0, 25, 50]),
                      np.arange(0, 60) * 17000 * s, np.array([0, 30, 60]), what=f"{blocks} blocks x 2^{scale_bits}")


# The pairing's key of a record and its 36-bit hash (life_key and run_of in csrc/xmem_prep.hip), to
# choose addresses that meet: at most 2^20 records are sorted by the hash's upper 18 bits.
def life_hash(addr, trace, bits=18):
    u, m = np.uint64, np.uint64(0xD6E8FEB86659FD93)
    with np.errstate(over="ignore"):
        x = (addr ^ (u(trace) * m)) * m
        x = (x ^ (x >> u(32))) * m
        wide = u(1 << 63) | (((x ^ (x >> u(32))) & u((1 << 61) - 1)) << u(1))
        key = np.where((addr < u(1 << 47)) & (trace < 1 << 15), (u(trace) << u(48)) | (addr << u(1)), wide)
        return ((key | u(1)) * u(0x9E3779B97F4A7C15)) >> u(64 - bits)


def hot_raw(n, base, trace, meet, seed):
    """n events, half of them at one address, taken and freed in turn; 30 rare addresses, 8 random
    events each (so pairs, allocations never freed, frees of nothing, before, in and after the hot
    ones), that share its 18 hash bits (meet) or don't; the rest pairs at other addresses."""
    rng = np.random.default_rng(seed)
    hot = np.uint64(base + (5 << 21))
    cand = (base + (rng.permutation(1 << 24) << 9)).astype(np.uint64)
    same = life_hash(cand, trace) == life_hash(np.array([hot]), trace)[0]
    rare = cand[same & (cand != hot) if meet else ~same][:30]
    assert len(rare) == 30
    raw = np.zeros(n, oracle.RAW_DTYPE)
    raw["ts"] = np.arange(n)
    place = np.sort(rng.permutation(n - 2000)[: n // 2] + 1000)  # none among the first and last 1,000
    rest = np.setdiff1d(np.arange(n), place)
    raw["addr"][place] = hot
    raw["bytes"][place] = np.where(np.arange(len(place)) % 2 == 0, 4096, -4096)
    raw["addr"][rest] = cand[~same][: len(rest)][np.arange(len(rest)) // 2]
    raw["bytes"][rest] = np.where(np.arange(len(rest)) % 2 == 0, 512, -512)
    at = rng.choice(rest, (30, 8), replace=False)
    at[:3, 0], at[:3, 1] = np.arange(3), n - 1 - np.arange(3)
    raw["addr"][at] = rare[:, None]
    raw["bytes"][at] = rng.choice([1024, -1024], (30, 8))
    raw["bytes"][at[0, :2]] = 1024, -1024
    return raw


@pytest.mark.parametrize("n", [8192, 40000, 1 << 20])
@pytest.mark.parametrize("base,trace", [(0x7F0000000000, 0), (1 << 52, 0), (0x7F0000000000, 40000)],
                         ids=["packed", "wide-address", "wide-trace"])
def test_lifecycles_hot_address(n, base, trace):
    """A hot address's records lie between those of the addresses that share its hash."""
    if n == 8192 and trace:
        pytest.skip("the one-workgroup sort is tested with one trace")
    raw = hot_raw(n, base, trace, True, n)
    off = np.concatenate([np.zeros(trace + 1, np.int64), [n]])  # (empty traces before it)
    check_lifecycles(raw, off, what=f"{n} events, half at one address")


@pytest.mark.parametrize("base", [0x7F0000000000, 1 << 52], ids=["packed", "wide"])
def test_lifecycles_partner_distance(base):
    """A partner, or the end of the run, at the edges of what a thread (16 records), its wavefront (64
    more) and its workgroup (2,048 a step) look at: rare addresses between the records of a hot one."""
    hot = np.uint64(base + (5 << 21))
    cand = (base + (np.arange(1 << 24) << 9)).astype(np.uint64)
    rare = cand[(life_hash(cand, 0) == life_hash(np.array([hot]), 0)[0]) & (cand != hot)]
    edges = [1, 2, 15, 16, 17, 18, 79, 80, 81, 82, 16 + 64 + 2048, 16 + 64 + 2049, 5000]
    assert len(rare) > len(edges)
    for end in edges:
        rows, h = [(rare[0], -64)], 0  # a free of nothing
        def hots(n):
            nonlocal h
            for _ in range(n):
                rows.append((hot, 4096 if h % 2 == 0 else -4096))
                h += 1
        for d, a in zip(edges, rare[1:]):
            rows.append((a, 512))
            hots(d - 1)
            rows.append((a, -512))
        rows.append((rare[0], 64))  # never freed, the run's end `end` records on
        hots(end - 1)
        raw = np.zeros(len(rows), oracle.RAW_DTYPE)
        raw["ts"] = np.arange(len(rows))
        raw["addr"] = np.array([a for a, _ in rows], np.uint64)
        raw["bytes"] = [b for _, b in rows]
        check_lifecycles(raw, np.array([0, len(rows)]), what=f"distances to {edges[-1]}, the run's end after {end}")


def test_lifecycles_hot_address_time():
    """The records between are stepped over by a workgroup: the call takes at most 4 times as long as
    where no address shares the hot one's hash (2.4 measured; over 500 by single threads)."""
    import torch
    import paper_2510_21048_amd as xm
    n, times = 1 << 20, []
    off = torch.tensor([0, n], device="cuda")
    for meet in (False, True):
        raw = torch.from_numpy(hot_raw(n, 0x7F0000000000, 0, meet, 3).view(np.uint8)).cuda()
        ms = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            xm.lifecycles(raw, off)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        times.append(sorted(ms)[1])
    log(f"[gpu-prep] {n} events, half at one address, whose hash none and 30 share: {times} ms")
    assert times[1] <= 4 * times[0], times


def sparse_offsets(rng, n_traces, filled, longest):
    """Offsets of traces of 0 records but for a share `filled` of them."""
    lens = np.where(rng.random(n_traces) < filled, rng.integers(1, longest + 1, n_traces), 0)
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)


@pytest.mark.parametrize("n_traces,filled,longest", [(70000, 0.03, 3), (30000, 0.5, 2), (20000, 0.9, 12), (5000, 0.01, 400),
                                                     (40000, 0.0001, 5000)])
def test_empty_traces_between(n_traces, filled, longest):
    """Runs of empty traces of every length between the records of one tile, at its edges, before the
    first record and after the last."""
    rng = np.random.default_rng(n_traces)
    off = sparse_offsets(rng, n_traces, filled, longest)
    wb, wboff = check_lifecycles(raw_of(int(off[-1]), 3, 1), off, what=f"{n_traces} traces, {filled} of them filled")
    woff = sparse_offsets(rng, n_traces, filled, longest)
    win = np.zeros(int(woff[-1]), oracle.WINDOW_DTYPE)
    win["start"] = np.arange(len(win)) * 2
    win["end"], win["parent"], win["kind"] = win["start"] + 1000, -1, 1
    check_attribute(wb, wboff, win, woff, what=f"{n_traces} traces, {filled} of them filled")
    none = np.zeros(n_traces + 1, np.int64)
    check_orchestrate(wb, wboff, none[:0], none, none[:0], none, what=f"{n_traces} traces, {filled} of them filled")


def test_empty_traces_time():
    """The trace of a record is found in steps that double: 40,000 traces of one record among
    2,000,000 take at most 10 times as long as alone (2.6 measured; with a step a trace, 100)."""
    import torch
    import paper_2510_21048_amd as xm
    n, times = 40000, []
    raw = raw_of(n, 3, 2)
    raw["bytes"] = 512
    d = torch.from_numpy(raw.view(np.uint8)).cuda()
    win = torch.zeros((n, 32), dtype=torch.uint8, device="cuda")
    for n_traces in (n, 2000000):
        off = np.zeros(n_traces + 1, np.int64)
        off[1 + np.sort(np.random.default_rng(4).choice(n_traces, n, replace=False))] = 1
        off = torch.from_numpy(np.cumsum(off)).cuda()
        no, none = torch.zeros(n_traces + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")
        ms = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            blocks, boff, _u, _s = xm.lifecycles(d, off)
            xm.attribute(blocks, boff, win, off)
            xm.orchestrate(blocks, boff, none, no, none, no)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        times.append(sorted(ms)[1])
    log(f"[gpu-prep] {n} traces alone and among 2,000,000: {times} ms")
    assert times[1] <= 10 * times[0], times
