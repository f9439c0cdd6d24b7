"""Selection from the largest scores of groups of 8 positions: the call that uses them (no pooled scores asked for) keeps the same positions,
bit for bit, as the call that ranks every position, which other tests compare with the oracle."""

import numpy as np
import pytest

from paper_2508_15806_amd import binding as B
from test_gpu_one_scan import both

pytestmark = pytest.mark.gpu

# one history of more than 8192 positions makes a call use them: others of 1, 7, 8, 9 positions, around the ends of groups and chunks, and of the
# most positions a thread block ranks
LENS = [33, 39, 40, 41, 32 + 127, 32 + 129, 2048 + 32, 8225, 32768 + 32]


@pytest.mark.parametrize("kernel,pool", [(1, B.SLKV_POOL_NONE), (3, B.SLKV_POOL_MAX), (5, B.SLKV_POOL_MAX), (7, B.SLKV_POOL_MAX), (15, B.SLKV_POOL_MAX),
                                         (63, B.SLKV_POOL_MAX)])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64)])
def test_lengths_and_windows(kernel, pool, dtype, d):
    caps = np.array([33, 35, 40, 60, 130, 300, 1200, 4000], dtype=np.int32)     # from one kept position to more groups than a list holds
    for lens in (LENS[:8], [8192 + 39], [12345, 20000], LENS[8:]):
        both(dtype, 32, 8, d, 32, lens, caps, kernel, pool)


@pytest.mark.parametrize("shape", ["equal keys", "zero queries", "few heavy keys", "one overwhelming key"])
@pytest.mark.parametrize("kernel", [1, 7, 31])
def test_ties_and_ranges(shape, kernel):
    # all scores alike (no bound below them but that of all), all but a few alike, one score that leaves the others far below
    caps = np.array([70, 100, 2000, 65], dtype=np.int32)
    pool = B.SLKV_POOL_MAX if kernel > 1 else B.SLKV_POOL_NONE
    for lens in ([300, 1000, 9000], [20000, 700]):
        both("bf16", 16, 4, 128, 64, lens, caps, kernel, pool, shape=shape)


@pytest.mark.parametrize("dtype", ["f32", "bf16_kv8"])
@pytest.mark.parametrize("Hq,Hkv,d,w,lens", [(4, 4, 64, 32, [9024, 100, 40]), (8, 1, 128, 64, [8800, 700]), (8, 2, 128, 32, [20001])])
def test_keys_of_32_and_8_bits(dtype, Hq, Hkv, d, w, lens):
    # one and several row blocks (512 rows), chunks shared by waves, segments that the first pass completes
    both(dtype, Hq, Hkv, d, w, lens, np.array([w + 20 + 60 * h for h in range(Hkv)], dtype=np.int32))


def test_decode_cache():
    both("bf16", 32, 8, 128, 32, [122, 929, 124, 134, 128, 10000, 140, 132] * 9, np.array([58, 865, 60, 70, 64, 60, 76, 68], dtype=np.int32), ragged=True)


def test_more_empty_segments_than_scores():
    # the groups of the last segment would lie behind the end of their array: such a call ranks every position
    both("bf16", 2, 1, 64, 16, [0] * 9999 + [9000, 0], np.array([100], dtype=np.int32))
    both("bf16", 2, 1, 64, 16, [0] * 6000 + [9000, 0], np.array([100], dtype=np.int32))     # (these fit)
