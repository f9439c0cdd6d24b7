"""Stage 1 over rows whose length is the most that a form of the row kernel holds, or one form further: rows of whole 16-byte groups, and others."""

import numpy as np
import pytest

import oracle
from paper_2508_15806_amd import api
from paper_2508_15806_amd import workloads as wl

pytestmark = pytest.mark.gpu

GROUPS = [384, 512, 640, 768, 1280, 1536, 1792, 2560, 3072, 3584, 4608, 5120, 6144, 7168, 9216, 10240, 11264]


@pytest.mark.parametrize("n", [4 * g + d for g in GROUPS for d in (0, -3, -2, 4)])
def test_most_groups_of_a_form(n):
    import torch
    topk = 64 if n % 8 else 17
    nr = wl.config4(L=1, H=2, T=5, n=n, needle_len=27, seed_extra=2000 + n)
    acc, sc = api.score_heads(torch.from_numpy(nr.rows).cuda(), nr.needle_start, nr.needle_len, topk)
    racc, rsc = oracle.score_heads(nr.rows, nr.needle_start, nr.needle_len, topk)
    np.testing.assert_allclose(acc.cpu().numpy(), racc, rtol=1e-12, atol=1e-15)      # the order of double sums
    np.testing.assert_allclose(sc.cpu().numpy(), rsc, rtol=1e-11, atol=1e-15)


@pytest.mark.parametrize("n", [2400, 5002, 17001, 20480, 28671, 33001, 45056])
def test_ties_at_the_cut(n):
    # quantised weights: the candidate lists overflow and the general path takes the row
    import torch
    rng = np.random.default_rng(n)
    q = rng.integers(0, 4, size=(1, 2, 3, n)).astype(np.float32)
    q /= q.sum(-1, keepdims=True)
    acc, _ = api.score_heads(torch.from_numpy(q).cuda(), n - 40, 40, 40)
    racc, _ = oracle.score_heads(q, n - 40, 40, 40)
    np.testing.assert_allclose(acc.cpu().numpy(), racc, rtol=1e-12, atol=1e-15)


@pytest.mark.parametrize("n", [4096, 8192, 12288, 16384, 20480, 32768])
def test_multiples_of_16_kib_at_any_place(n):
    # weights of many magnitudes, whose double sums are rounded: a head scored alone and at each of 40 places of a call gives the same bits
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n)
    one = torch.softmax(12 * torch.randn(1, 1, 3, n, generator=gen, device="cuda"), -1)
    start, topk = n // 3, 21
    alone, sc_alone = api.score_heads(one, start, 27, topk)
    acc, sc = api.score_heads(one.expand(2, 20, 3, n).contiguous(), start, 27, topk)
    assert torch.equal(acc, alone.expand(2, 20, 5)) and torch.equal(sc, sc_alone.expand(2, 20, 3))
    racc, rsc = oracle.score_heads(one.cpu().numpy(), start, 27, topk)
    np.testing.assert_allclose(alone.cpu().numpy(), racc, rtol=1e-12, atol=1e-15)
    np.testing.assert_allclose(sc_alone.cpu().numpy(), rsc, rtol=1e-11, atol=1e-15)


@pytest.mark.parametrize("n", [777, 1800, 3000, 5002, 8192, 12000, 16384, 28000, 40001, 60000])
@pytest.mark.parametrize("topk,above,equal", [(64, 61, 2), (64, 63, 2), (64, 60, 9), (62, 0, 66), (40, 39, 7), (33, 20, 30)])
def test_few_equal_weights_at_the_cut(n, topk, above, equal):
    # `equal` equal weights behind the `above` largest ones, all of them in lists of at most 256: no value is reached by exactly K of them, each is ranked, and the lower positions
    # count.  (Above 64 candidates four to a lane, which K = 62 and 64 make sure of.)
    import torch
    rng = np.random.default_rng(n + topk + equal)
    rows = rng.random((1, 2, 8, n)).astype(np.float32)
    for row in rows.reshape(-1, n):
        order = np.argsort(-row)
        row[order[above:above + equal]] = row[order[above]]
    rows /= n
    start = n // 4
    acc, sc = api.score_heads(torch.from_numpy(rows).cuda(), start, n // 2, topk)
    racc, rsc = oracle.score_heads(rows, start, n // 2, topk)
    np.testing.assert_allclose(acc.cpu().numpy(), racc, rtol=1e-12, atol=1e-15)
    np.testing.assert_allclose(sc.cpu().numpy(), rsc, rtol=1e-11, atol=1e-15)
