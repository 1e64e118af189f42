"""Parity of the row tables (a pool's free blocks sorted in registers, on 1 to 8, 10 or 12 rows of
64, one slot always empty but in 12) with the CPU oracle, bit-exact: free counts that cross and
settle on every row boundary, full tables, runs of allocations freed at once (skipped when a cached
block fits them), and reclamation from tables of several rows."""
import numpy as np
import pytest

import oracle
from evw import A, F, KiB, MiB
from gpu_util import check
from spill_traces import batch

pytestmark = pytest.mark.gpu

P = oracle.paper_params()
PT = oracle.pytorch_like_params()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_21048_amd as xm
    xm.load()
    yield


def around(seed: int, holes: int, large: bool, churn: int = 400, pairs: bool = True) -> np.ndarray:
    """`holes` free blocks that cannot coalesce, then random allocations and frees that keep the
    free count around it (some allocations freed by the very next event, of sizes up to past every
    free block), then everything freed but a few blocks."""
    rng = np.random.default_rng(seed)
    unit, top = (MiB + 512, 6 * MiB) if large else (512, 24 * KiB)
    size = lambda: int(rng.integers(unit, top))
    ev = [A(size()) for _ in range(2 * holes + 1)]
    live = list(range(0, 2 * holes + 1, 2))
    gone = list(range(1, 2 * holes + 1, 2))
    rng.shuffle(gone)
    ev += [F(h) for h in gone]
    for _ in range(churn):
        r = rng.random()
        if pairs and r < 0.4:  # freed at once: usually fits, sometimes needs a new segment
            big = rng.random() < 0.1
            ev.append(A(top * 4 if big and large else MiB if big else size()))
            ev.append(F(len(ev) - 1))
        elif r < 0.7 or not live:
            live.append(len(ev))
            ev.append(A(size()))
        else:
            k = int(rng.integers(len(live)))
            live[k], live[-1] = live[-1], live[k]
            ev.append(F(live.pop()))
    rng.shuffle(live)
    ev += [F(h) for h in live[3:]]
    return np.array(ev, dtype=np.uint64)


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("params", [P, PT], ids=["paper", "pytorch_like"])
@pytest.mark.parametrize("chunks", [0, 1])
def test_every_row_boundary(params, large, chunks):
    holes = [0, 1, 62, 63, 64, 104, 127, 128, 191, 192, 255, 256, 319, 320, 383, 384, 447, 448, 511, 512, 639, 640, 766, 767, 768]
    ev, off = batch([around(100 + h, h, large) for h in holes])
    check(ev, off, params, chunks=chunks, what=f"row boundaries large={large}")


@pytest.mark.parametrize("gap", [0, 1, 61, 62, 63, 64, 65])
def test_pairs_across_a_tile(gap):
    """Allocation/free pairs at every place of the 64-event tiles, split by a tile boundary, with
    the other pool's pairs inside them, and runs that stop at one that needs a new segment."""
    ev = [A(1 * KiB)] * gap
    for i in range(200):
        ev += [A(2 * KiB + 512 * (i % 7)), F(len(ev))]
        if i % 3 == 0:
            n = len(ev)
            ev += [A(600), A(3 * MiB), F(n + 1), F(n)]
        if i % 50 == 49:
            ev += [A(MiB), A(MiB), F(len(ev))]
    ev, off = batch([np.array(ev, dtype=np.uint64)])
    check(ev, off, P, what=f"pairs, {gap} events before")
    check(ev, off, dict(P, device_capacity_bytes=64 * MiB), what=f"pairs under a capacity, {gap} events before")


@pytest.mark.parametrize("holes", [3, 64, 130, 300, 600])
def test_reclaim_from_rows(holes):
    """Idle segments released from tables of one to twelve rows in both pools, among fragments that
    stay; then the pools grow again, up to OOM."""
    n = holes + 1
    ev = [A(MiB)] * (2 * n)                                       # two to a segment
    ev += [F(i) for i in range(0, 2 * n, 2)]                      # fragments: no segment idle
    ev += [F(i) for i in range(1, n, 2)]                          # half of the segments idle
    s = len(ev)
    ev += [A(15 * MiB)] * 8
    ev += [F(s + i) for i in (1, 2, 5)]
    ev += [A((11 + i) * MiB) for i in range(40)]                  # past the capacity: reclaim, reuse, OOM at last
    ev, off = batch([np.array(ev, dtype=np.uint64)])
    cap = (2 * n + 8 * 16 + 100) * MiB
    g, _ = check(ev, off, dict(P, device_capacity_bytes=cap), what=f"reclaim, {holes} fragments")
    assert int(g["segments_released"][0]) > 0 and int(g["status"][0]) == 1


# every request of two units or more is served by a segment of its own size: free blocks never touch
EXACT = oracle.paper_params(small_max_bytes=512, small_segment_bytes=512, mid_segment_bytes=1024,
                            min_large_alloc_bytes=1024, large_round_bytes=512)


def full_table(n: int, seed: int) -> np.ndarray:
    """n free blocks of as many sizes, then requests that split or take one, are freed at once, or fit
    none and are kept: the free count is n at most, again and again."""
    rng = np.random.default_rng(seed)
    ev = [A(512 * (2 + i)) for i in range(n)]
    ev += [F(int(i)) for i in rng.permutation(n)]
    live = []
    for i in range(600):
        r = rng.random()
        if r < 0.1:
            ev.append(A(512 * (n + 10 + i)))  # fits none, kept
        elif r < 0.4:
            ev += [A(512 * int(rng.integers(1, n + 2))), F(len(ev))]
        elif r < 0.7 or not live:
            live.append(len(ev))
            ev.append(A(512 * int(rng.integers(2, n + 2))))
        else:
            ev.append(F(live.pop(int(rng.integers(len(live))))))
    return np.array(ev + [F(i) for i in live], dtype=np.uint64)


@pytest.mark.parametrize("chunks", [0, 1, 9])
def test_full_table(chunks):
    """Twelve rows may be full, where a search can end at no key and no empty slot."""
    ev, off = batch([full_table(n, s) for n in (766, 767, 768, 769) for s in (1, 2, 3)])
    for cap in (None, 1 << 40):
        p = EXACT if cap is None else dict(EXACT, device_capacity_bytes=cap)
        g, _ = check(ev, off, p, chunks=chunks, what=f"full table, capacity {cap}")
        assert g["max_free_blocks_large"].tolist() == [n for n in (766, 767, 768, 769) for _ in range(3)]
    ev, off = batch([full_table(768, s) for s in (1, 2, 3)])
    held = 512 * sum(range(2, 770))
    g, _ = check(ev, off, dict(EXACT, device_capacity_bytes=held + 512 * 2000), what="reclaim from a full table")
    assert (g["segments_released"] > 0).all()


def test_full_table_time():
    """Pools that fill the table stay on it: 400 traces whose pools peak at 768 free blocks take at most
    3 times as long as at 754 (1.03 measured; 32 where the paged kernel has to replay them)."""
    import torch
    import paper_2510_21048_amd as xm
    from paper_2510_21048_amd import binding
    us = {}
    for peak, seed in ((754, 101), (768, 7)):
        trace = around(seed, 400, True, churn=3000, pairs=False)
        _rc, r, _ = oracle.replay(*batch([trace]), P, series=False)
        assert int(r["max_free_blocks_large"][0]) == peak
        ev, off = batch([trace] * 400)
        e, o, p = torch.from_numpy(ev.view(np.int64)).cuda(), torch.from_numpy(off).cuda(), xm.params(0)
        ws = torch.empty(binding.xmem_workspace_bytes(400, len(ev), p), dtype=torch.uint8, device="cuda")
        times = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            binding.replay(e, o, p, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3)
        us[peak] = min(times)
    print(us, flush=True)
    assert us[768] <= 3 * us[754], us


def test_serial_batch_time_by_pool():
    """20,000 traces, too many for chunks, of 1,000 events: all in one pool they take about as long as
    half in each (1.0 measured; 1.5 where every second shader engine gets the idle pools)."""
    import torch
    import paper_2510_21048_amd as xm
    from paper_2510_21048_amd import binding
    T, n, us = 20000, 1000, {}
    for kind in ("both", "small", "large"):
        rng = np.random.default_rng(1)
        ev, live = [], ([], [])
        for i in range(n):
            pool = {"small": 0, "large": 1, "both": i & 1}[kind]
            if len(live[pool]) < 20 or rng.random() < 0.5:
                live[pool].append(len(ev))
                ev.append(A(int(rng.integers(MiB + 1, 8 * MiB) if pool else rng.integers(1, 24 * KiB))))
            else:
                ev.append(F(live[pool].pop(int(rng.integers(len(live[pool]))))))
        e = torch.from_numpy(np.tile(np.array(ev, dtype=np.uint64), T).view(np.int64)).cuda()
        o, p = torch.arange(T + 1, device="cuda") * n, xm.params(0)
        ws = torch.empty(binding.xmem_workspace_bytes(T, T * n, p), dtype=torch.uint8, device="cuda")
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            binding.replay(e, o, p, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3)
        us[kind] = min(times)
    print(us, flush=True)
    assert max(us["small"], us["large"]) <= 1.25 * us["both"], us
