"""The one-workgroup selection with 2, 4, 8, 16, 24 and 32 positions a thread: histories that fill a form's round, and one position more or less, against the
selection by blocks, bit for bit, and against the oracle; few and nearly all positions kept, piles of equal scores, every pooling radius with a form of its own."""

import numpy as np
import pytest

import parity
from paper_2508_15806_amd import binding as B
from paper_2508_15806_amd import workloads as wl

pytestmark = pytest.mark.gpu

EDGES = [2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193, 16383, 16384, 16385, 24575, 24576, 24577, 32768]


@pytest.mark.parametrize("m", EDGES)
@pytest.mark.parametrize("pool,pool_kernel", [("avg", 5), ("max", 3), ("avg", 13), ("none", 1), ("max", 7)])
def test_edges(monkeypatch, m, pool, pool_kernel):
    w = 16
    mode = {"max": B.SLKV_POOL_MAX, "avg": B.SLKV_POOL_AVG, "none": B.SLKV_POOL_NONE}[pool]
    lay = wl.make_layer((701, m), [m + w, 500], 4, 4, 64, w, dtype="bf16", bias_frac=0.02)
    lay.k[3, :m] = lay.k[3, :3][np.arange(m) % 3]                # three different keys
    budgets = np.array([w + 1, 900, m + w - 1, m // 2], dtype=np.int32)
    got = []
    for path in ("resident", "blocks"):
        monkeypatch.setenv("SLKV_SELECT", path)
        gpu = parity.run_gpu(lay, budgets, pool_kernel, mode)
        got.append(gpu)
    for name in ("kept", "pooled", "importance"):
        np.testing.assert_array_equal(got[0][name], got[1][name])
    if m in (2049, 8193, 16385):
        rep = parity.compare_layer(lay, budgets, got[0], pool_kernel, mode)
        assert rep["ranked"] == 5 and rep["tolerant"] == 0
