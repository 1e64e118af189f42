"""The work that a user of this library has it do, as cases that can be timed and compared.

Every case goes through the package's public calls: a replay of recorded allocator traces (one
trace, a sweep, a Monte Carlo batch, under a device capacity or not, with the per-event reserved
series or not), the preparation of raw profiler streams, and the whole estimate from raw events
to the out-of-memory prediction.  Inputs come from the seeded generators of ``tracegen``; they
are resident on the GPU and the workspaces are held by the caller, as in a serving program.

All results are integers: two correct implementations give the same bits.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2510_21048_amd as xm
import tracegen
from paper_2510_21048_amd import binding
from tracegen import prep as profiles

GIB = 1 << 30
MIX = 0x9E3779B97F4A7C15  # spreads consecutive seeds over the generators' 64-bit seed space


def listed():
    return [
        # The smallest call: the first events of one training script, from a loop that may not
        # allocate (the library's own scratch): latency and launches only.
        {"name": "short_noalloc", "kind": "noalloc", "config": 3, "traces": 1, "events": 1001},
        # One small model estimated alone: a 12-layer MLP, three iterations.
        {"name": "mlp_one", "kind": "replay", "config": 1, "traces": 1, "events": 4096, "preset": 0, "series": False},
        # One Transformer estimated alone, with the memory curve that a user plots.
        {"name": "gpt_one_series", "kind": "replay", "config": 3, "traces": 1, "events": 262144, "preset": 0,
         "series": True},
        # A batch-size sweep of one CNN: which batch still fits.
        {"name": "resnet_sweep", "kind": "replay", "config": 2, "traces": 256, "events": 65536, "preset": 0,
         "series": False},
        # The largest batch: every Transformer shape, long traces.
        {"name": "gpt_batch", "kind": "replay", "config": 3, "traces": 1024, "events": 262144, "preset": 0,
         "series": False},
        # Monte Carlo perturbations of the Transformer shapes: very many traces.
        {"name": "monte_carlo", "kind": "replay", "config": 4, "traces": 4096, "events": 65536, "preset": 0,
         "series": False},
        # One very long training run with a fragmented heap.
        {"name": "long_fragmented", "kind": "replay", "config": 5, "traces": 1, "events": 16777216, "preset": 0,
         "series": False},
        # Jobs of a mixed queue: CNNs and Transformers of odd lengths, the PyTorch-like split
        # rule, with the per-event series.
        {"name": "mixed_ragged_series", "kind": "ragged", "traces": 48, "shortest": 501, "longest": 40001},
        # The same sweep under a device's capacity (40 GiB): reclamation, simulated OOM and the
        # prediction flags.
        {"name": "resnet_capped", "kind": "capped", "config": 2, "traces": 64, "events": 65536, "capacity_gib": 40},
        # One short profile prepared: lifecycles, attribution, orchestration.
        {"name": "prep_one", "kind": "prep", "traces": 1, "events": 4001, "layers": 24, "capacity_gib": 0},
        # A batch of long profiles prepared.
        {"name": "prep_batch", "kind": "prep", "traces": 128, "events": 65536, "layers": 24, "capacity_gib": 0},
        # The whole estimate of a few jobs: raw events, replay, out-of-memory prediction at 12 GiB.
        {"name": "estimate", "kind": "estimate", "traces": 16, "events": 20011, "layers": 24, "capacity_gib": 12},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["replay", "replay", "replay", "long", "noalloc", "ragged", "capped", "prep", "prep", "estimate"])
    if kind == "replay":
        config = rng.choice([1, 2, 3, 4])
        events = 2 * _log_int(rng, 2100, 8000) if config == 1 else _log_int(rng, 1000, 262144)
        traces = _log_int(rng, 1, max(1, min(1024, (1 << 25) // events)))
        return {"kind": "replay", "config": config, "traces": traces, "events": events,
                "preset": rng.choice([0, 1]), "series": rng.random() < 0.5}
    if kind == "long":
        return {"kind": "replay", "config": 5, "traces": 1, "events": _log_int(rng, 1 << 20, 1 << 24), "preset": 0,
                "series": rng.random() < 0.5}
    if kind == "noalloc":
        return {"kind": "noalloc", "config": rng.choice([2, 3, 4]), "traces": rng.randint(1, 4),
                "events": _log_int(rng, 300, 6000)}
    if kind == "ragged":
        return {"kind": "ragged", "traces": _log_int(rng, 3, 200), "shortest": _log_int(rng, 50, 2000),
                "longest": _log_int(rng, 4000, 60000)}
    if kind == "capped":
        return {"kind": "capped", "config": rng.choice([2, 3]), "traces": _log_int(rng, 4, 256),
                "events": _log_int(rng, 2000, 65536), "capacity_gib": rng.choice([12, 24, 40, 80])}
    if kind == "prep":
        return {"kind": "prep", "traces": _log_int(rng, 1, 100), "events": _log_int(rng, 500, 50000),
                "layers": rng.randint(4, 40), "capacity_gib": 0}
    return {"kind": "estimate", "traces": _log_int(rng, 1, 40), "events": _log_int(rng, 500, 30000),
            "layers": rng.randint(4, 40), "capacity_gib": rng.choice([12, 24, 40])}


# ---------------------------------------------------------------- inputs
def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _traces(case, seed):
    """Event words and offsets of a replay case (numpy)."""
    s = (int(seed) * MIX) % (1 << 63)
    if case["kind"] != "ragged":
        return tracegen.generate(case["config"], case["traces"], case["events"], seed=s)
    rng = np.random.default_rng(case["traces"] + case["longest"])  # the queue's job list: the case's own
    lo, hi = math.log(case["shortest"]), math.log(case["longest"])
    jobs = [(int(rng.choice([2, 3, 4])), int(math.exp(rng.uniform(lo, hi))) | 1, int(rng.integers(0, 256)))
            for _ in range(case["traces"])]
    parts = [tracegen.generate(config, 1, n, seed=s, first_trace=first, threads=1)[0] for config, n, first in jobs]
    return np.concatenate(parts), np.concatenate([[0], np.cumsum([n for _c, n, _f in jobs])]).astype(np.int64)


@functools.lru_cache(maxsize=4)
def _generated(count, events, layers):
    return profiles.batch_profiles(count, events, seed=layers, layers=layers, windows=True)


def _profiles(case, seed):
    """A batch of profiler streams: up to 8 generated ones, repeated.  Each stream is a job of its
    own: another clock (start and tick), another heap base, another batch size (all its tensors'
    bytes), all from the seed; how many blocks it holds is the case's own."""
    T = case["traces"]
    base = min(T, 8)
    raw, _cat, roff, st, soff, zg, zoff, win, woff = _generated(base, case["events"], case["layers"])
    rng = np.random.default_rng(int(seed))
    start, tick, heap, size = (torch.from_numpy(v).cuda() for v in (
        rng.integers(0, 1 << 20, T), rng.integers(1, 5, T), rng.integers(0, 1 << 12, T) << 24, rng.integers(1, 17, T)))

    def tile(a, off, words):
        """Trace t takes generated profile t % base; `words` int64 words a record."""
        a = torch.from_numpy(np.ascontiguousarray(a).view(np.int64).reshape(-1, words)).cuda()
        lens = np.array([int(off[t % base + 1] - off[t % base]) for t in range(T)], np.int64)
        o = np.zeros(T + 1, np.int64)
        o[1:] = np.cumsum(lens)
        of = torch.repeat_interleave(torch.arange(T, device="cuda"), torch.from_numpy(lens).cuda())
        a = torch.cat([a[int(off[t % base]): int(off[t % base + 1])] for t in range(T)])
        return a, torch.from_numpy(o).cuda(), of

    r, r_off, of = tile(raw, roff, 3)
    r[:, 0] = r[:, 0] * tick[of] + start[of]
    r[:, 1] += heap[of]
    r[:, 2] *= size[of]
    w, w_off, of = tile(win, woff, 4)
    w[:, :2] = w[:, :2] * tick[of, None] + start[of, None]
    s, s_off, of = tile(st, soff, 1)
    s = s[:, 0] * tick[of] + start[of]
    z, z_off, of = tile(zg, zoff, 1)
    z = z[:, 0] * tick[of] + start[of]
    return {"raw": r.view(torch.uint8), "raw_off": r_off, "win": w.view(torch.uint8), "win_off": w_off,
            "steps": s, "steps_off": s_off, "zg": z, "zg_off": z_off}


def prepare(case, seed):
    s = {"case": case}
    if case["kind"] in ("prep", "estimate"):
        s.update(_profiles(case, seed))
        T, N = case["traces"], s["raw"].shape[0]
        # one workspace for the three steps, the largest that any of them takes
        records = max(2 * N, s["win"].shape[0])
        s["workspace"] = torch.empty(binding.xmem_prep_workspace_bytes(T, records), dtype=torch.uint8, device="cuda")
        if case["kind"] == "estimate":
            s["params"] = xm.params()
            need = binding.xmem_workspace_bytes(T, 2 * N, s["params"])
            s["replay_workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        return s
    ev, off = _traces(case, seed)
    s["events"], s["offsets"] = _gpu(ev.view(np.int64)), _gpu(off)
    preset = {"ragged": 1, "replay": case.get("preset", 0)}.get(case["kind"], 0)
    s["params"] = xm.params(preset)
    if case["kind"] == "capped":
        s["params"] = xm.params(preset, device_capacity_bytes=case["capacity_gib"] * GIB)
    if case["kind"] == "noalloc":
        s["out"] = torch.empty((case["traces"], 96), dtype=torch.uint8, device="cuda")
    else:
        need = binding.xmem_workspace_bytes(len(off) - 1, len(ev), s["params"])
        s["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    return s


# ---------------------------------------------------------------- one pass
def _words(t):
    """Records as rows of int64 words."""
    return t.view(torch.int64)


def _prep(s):
    ws = s["workspace"]
    blocks, boff, unmatched, st1 = binding.lifecycles(s["raw"], s["raw_off"], workspace=ws)
    kept, koff, window, st2 = binding.attribute(blocks, boff, s["win"], s["win_off"], workspace=ws)
    words, eoff, st3 = binding.orchestrate(kept, koff, s["steps"], s["steps_off"], s["zg"], s["zg_off"], workspace=ws)
    n_words = int(eoff[-1])  # the caller sizes the replay (or the file it writes) by it
    nb = window.shape[0]
    out = {"blocks": _words(blocks[:nb]), "block_offsets": boff, "unmatched": unmatched, "window": window,
           "kept_offsets": koff, "event_offsets": eoff, "status": [st1, st2, st3]}
    return words[:n_words], eoff, kept, koff, out


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "prep":
        words, _eoff, kept, koff, out = _prep(s)
        out["kept"] = _words(kept[: int(koff[-1])])
        out["words"] = words
        return out
    if kind == "estimate":
        words, eoff, _kept, _koff, _out = _prep(s)
        res, _ = binding.replay(words, eoff, s["params"], workspace=s["replay_workspace"])
        flags = binding.oom_predicted(res, case["capacity_gib"] * GIB)
        return {"words": words, "event_offsets": eoff, "results": _words(res), "oom": flags}
    if kind == "noalloc":
        rc = binding.xmem_replay_batch_noalloc(s["events"], s["offsets"], case["traces"], s["events"].numel(), s["params"],
                                               s["out"], None, torch.cuda.current_stream().cuda_stream)
        if rc != binding.XMEM_OK:
            raise RuntimeError(binding.xmem_strerror(rc))
        return _words(s["out"])
    series = kind == "ragged" or bool(case.get("series"))
    res, ser = binding.replay(s["events"], s["offsets"], s["params"], series=series, workspace=s["workspace"])
    if kind == "capped":
        return {"results": _words(res), "oom": binding.oom_predicted(res, case["capacity_gib"] * GIB)}
    return {"results": _words(res), "series": ser} if series else _words(res)


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    T = case["traces"]
    if case["kind"] in ("prep", "estimate"):
        # per raw event of these streams: about 0.51 windows, 0.507 blocks, 0.495 attributed
        # blocks and 0.986 event words
        n = float(T * case["events"])
        read = 24 * n + 32 * 0.51 * n
        if case["kind"] == "prep":
            return {"bytes": read + (32 + 4) * 0.507 * n + 32 * 0.495 * n + 8 * 0.986 * n, "flops": 0}
        return {"bytes": read + 8 * 0.986 * n + 100 * T, "flops": 0}
    if case["kind"] == "ragged":
        ratio = case["longest"] / case["shortest"]
        n = T * (case["longest"] - case["shortest"]) / math.log(ratio)  # the mean of a log-uniform length
    else:
        n = float(T * case["events"])
    series = case["kind"] == "ragged" or bool(case.get("series"))
    return {"bytes": 8 * n + (8 * n if series else 0) + 104 * T, "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """Whole numbers and bytes throughout: any difference counts, so there is no 64-bit value to
    be nearer to or further from."""
    return None
