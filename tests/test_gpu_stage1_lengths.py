"""Stage 1 over rows of any length: the lengths at which the row kernel changes its workgroup, rows that begin at
every float of a 16-byte group, rows whose last group reaches past the tensor."""

import numpy as np
import pytest

import oracle
from paper_2508_15806_amd import api
from paper_2508_15806_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,topk", [(3, 2), (4, 3), (5, 3), (7, 7), (66, 64), (1021, 16), (1022, 64), (1025, 1), (2045, 32), (2046, 64),
                                    (4093, 64), (4094, 5), (8189, 64), (8190, 32), (13867, 27), (16381, 64), (16382, 33),
                                    (32765, 64), (32766, 20), (65533, 64), (65534, 32)])
def test_lengths_around_the_workgroup_sizes(n, topk):
    import torch
    nr = wl.config4(L=1, H=3, T=5, n=n, needle_len=max(1, min(27, n // 3)), seed_extra=1000 + n)
    acc, sc = api.score_heads(torch.from_numpy(nr.rows).cuda(), nr.needle_start, nr.needle_len, topk)
    racc, rsc = oracle.score_heads(nr.rows, nr.needle_start, nr.needle_len, topk)
    np.testing.assert_allclose(acc.cpu().numpy(), racc, rtol=1e-12, atol=1e-15)
    np.testing.assert_allclose(sc.cpu().numpy(), rsc, rtol=1e-11, atol=1e-15)


@pytest.mark.parametrize("n", [1023, 5001, 16383, 40001])
def test_ties_at_the_cut_in_rows_of_odd_length(n):
    # quantised weights: thousands of equal values at the K-th place overflow the candidate lists
    import torch
    rng = np.random.default_rng(n)
    q = rng.integers(0, 4, size=(1, 2, 3, n)).astype(np.float32)
    q /= q.sum(-1, keepdims=True)
    for start, topk in ((0, 50), (n - 40, 40)):
        acc, _ = api.score_heads(torch.from_numpy(q).cuda(), start, 40, topk)
        racc, _ = oracle.score_heads(q, start, 40, topk)
        np.testing.assert_allclose(acc.cpu().numpy(), racc, rtol=1e-12, atol=1e-15)
