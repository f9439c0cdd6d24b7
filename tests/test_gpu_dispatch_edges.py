"""GPU parity where the scoring passes and the segment tables change their form: key groups, waves that share a group's
query tiles, segments of one chunk, tables in the kernel argument or in the workspace."""

import numpy as np
import pytest

import parity
from paper_2508_15806_amd import workloads as wl

pytestmark = pytest.mark.gpu


def check(lay, budgets):
    parity.compare_layer(lay, budgets, parity.run_gpu(lay, budgets))


@pytest.mark.parametrize("dtype", ["f32", "bf16_kv8"])
@pytest.mark.parametrize("Hq,Hkv,w,d", [(2, 2, 16, 64), (4, 2, 17, 128), (8, 2, 32, 128), (8, 2, 32, 64), (8, 1, 33, 128), (14, 2, 40, 64)])
def test_key_groups_and_query_tiles(dtype, Hq, Hkv, w, d):
    # histories of one key, around one and two groups (32 or 64 keys) and of some; 16 to 280 query rows: one tile, a part of the
    # second, four tiles, more rows than a block holds
    lay = wl.make_layer((301, Hq, w, d), [w + n for n in (1, 31, 32, 33, 64, 65, 129, 515)], Hq, Hkv, d, w, dtype=dtype, bias_frac=0.05)
    check(lay, np.array([w + 5 + 9 * h for h in range(Hkv)], dtype=np.int32))


@pytest.mark.parametrize("dtype,lens", [("f32", [3000]), ("f32", [9000, 40]), ("bf16_kv8", [5000]), ("bf16_kv8", [20000, 300])])
def test_many_chunks_per_segment(dtype, lens):
    lay = wl.make_layer((302, len(lens)), lens, 8, 2, 128, 32, dtype=dtype, bias_frac=0.03)
    check(lay, np.array([300, 90], dtype=np.int32))


@pytest.mark.parametrize("Hq,Hkv,w,lens", [(4, 2, 32, [32 + 127, 32 + 128, 32 + 129, 2000]), (16, 2, 64, [500, 64 + 256]), (14, 2, 64, [3000, 90]),
                                          (8, 8, 48, [4500])])
def test_16_bit_chunks_of_two_tiles_and_more(Hq, Hkv, w, lens):
    # 64, 512, 448 and 48 query rows; chunks of 128 keys, around whose ends the short histories lie
    lay = wl.make_layer((304, Hq, w), lens, Hq, Hkv, 128, w, dtype="bf16", bias_frac=0.04)
    check(lay, np.array([w + 30 + 11 * h for h in range(Hkv)], dtype=np.int32))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,Hkv", [(8, 8), (13, 5), (32, 8), (57, 8)])
def test_segment_tables(dtype, B, Hkv):
    # 64 segments (everything per segment in the argument), 65 and 256 (per sequence and head), 456 (in the workspace)
    rng = np.random.default_rng(B)
    lay = wl.make_layer((303, B, Hkv), rng.integers(1, 260, size=B).tolist(), Hkv, Hkv, 64, 8, dtype=dtype, bias_frac=0.05)
    check(lay, np.array([10 + 13 * h for h in range(Hkv)], dtype=np.int32))
