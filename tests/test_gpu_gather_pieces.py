"""GPU parity where a call keeps so many rows that every gather thread copies four 16-byte pieces (more than 524288
pieces of K, one a thread up to there): all segment tables, both selections (which copies segments of up to 256 kept rows
itself, or leaves all of them to the gather), carried positions, empty segments, padded strides."""

import numpy as np
import pytest

import parity
from paper_2508_15806_amd import workloads as wl

pytestmark = pytest.mark.gpu

ONE_PIECE_MOST = 256 * 2048
BUDGETS = np.array([300, 40, 100000, 2], dtype=np.int32)   # ranked and gathered; ranked and copied by the selection; all kept; the window only
W = 8


def kept(n, cap):
    return n if n <= W or n <= cap else max(cap, W)


def ragged_lengths(rng, nseg, rows):
    """Lengths of the segments of 4 heads of which `rows` rows are kept in all: runs of empty segments, a few rows, lengths
    around the window, the capacities and the 256 rows that the selection copies itself; the third head's make up the sum."""
    lens = rng.choice([0, 0, 0, 1, 3, W, W + 1, 39, 41, 255, 256, 257, 301, 500], size=nseg)
    for s in range(5, nseg, 23):
        lens[s:s + 6] = 0                                    # more empty segments in a row than are fetched at once
    big = np.arange(2, nseg, 4)[1::2]
    lens[big] = 0
    left = rows - sum(kept(int(n), int(BUDGETS[s % 4])) for s, n in enumerate(lens))
    assert left > len(big)
    cuts = np.sort(rng.choice(np.arange(1, left), size=len(big) - 1, replace=False))
    lens[big] = np.diff(np.concatenate([[0], cuts, [left]]))
    return lens.tolist()


@pytest.mark.parametrize("select", ["resident", "blocks"])
@pytest.mark.parametrize("extra", [0, 1, 45])
@pytest.mark.parametrize("nseg,d,dtype", [(64, 128, "bf16"), (64, 64, "bf16_kv8"), (200, 128, "f32"), (400, 64, "f32")])
def test_ragged_cache(monkeypatch, nseg, d, dtype, extra, select):
    # 64 segments (everything per segment in the argument), 200 (per sequence and head), 400 (in the workspace); exactly as many
    # rows as one piece a thread takes, one row and some rows more
    monkeypatch.setenv("SLKV_SELECT", select)
    per_row = d * {"bf16": 2, "bf16_kv8": 1, "f32": 4}[dtype] // 16
    rows = ONE_PIECE_MOST // per_row + extra
    lens = ragged_lengths(np.random.default_rng(nseg + extra), nseg, rows)
    rc = wl.make_ragged_cache((305, nseg, extra), lens, nseg // 4, 4, 4, d, W, dtype=dtype, bias_frac=0.04)
    gpu = parity.run_gpu_ragged(rc, BUDGETS, positions=extra != 45)
    assert gpu["call"].total_kept == rows
    rep = parity.compare_ragged(rc, BUDGETS, gpu)
    assert rep["ranked"] >= 2 and rep["tolerant"] == 0


@pytest.mark.parametrize("select", ["resident", "blocks"])
@pytest.mark.parametrize("lens", [[5000, 3, 7001, 90, 4300], [1000, 1, 1300, 999, 256, 257, 2100, 40, 1500, 1201, 700, 1800, 7, 2300, 650, 1417, 1111]])
def test_layer(monkeypatch, lens, select):
    # 20 segments and 68, a token-major cache with padded V rows
    monkeypatch.setenv("SLKV_SELECT", select)
    lay = wl.make_layer((306, len(lens)), lens, 4, 4, 128, W, dtype="f32", bias_frac=0.04)
    gpu = parity.run_gpu(lay, BUDGETS, token_major=True)
    assert gpu["call"].total_kept * 32 > ONE_PIECE_MOST
    rep = parity.compare_layer(lay, BUDGETS, gpu)
    assert rep["ranked"] >= 6 and rep["tolerant"] == 0
