"""Parity of the trace-preparation steps with the oracle where their launches change: one
workgroup's sort against passes of tiles, two, three or four digits of the pairing's hash (many
distinct addresses, so that unequal ones share it), offsets checked by one workgroup or several,
traces past the range of the packed key, tile counts added up or scanned."""
import numpy as np
import pytest

import oracle
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
