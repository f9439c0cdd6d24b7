"""GPU parity of slkv_score_heads_qk (Stage 1 straight from decode queries and context keys, the
attention rows never in memory) against the float64 oracle, through the C ABI.

The GPU computes logits as fp32 sums of exact bf16 products and weights as fp32 exponentials, the
oracle everything in float64: weights agree to about 1e-5 relative, so do the cells (sums of at
most K weights per row).  Two logits closer than fp32 rounding could rank differently on the two
sides; the seeded inputs here hold no such pair at the K-th place (a flip would move a whole
weight between cells and fail the comparison)."""

import numpy as np
import pytest

import oracle
from paper_2508_15806_amd import api
from paper_2508_15806_amd import workloads as wl

pytestmark = pytest.mark.gpu

RTOL, ATOL = 2e-4, 2e-7


def run_gpu(x, acc=None):
    import torch
    q = api.to_device(x.q, "bf16")
    k = api.to_device(x.k, "bf16")
    acc_d, sc_d = api.score_heads_qk(q, k, x.needle_start, x.needle_len, x.topk, acc)
    torch.cuda.synchronize()
    return acc_d, sc_d


def check(x):
    acc_d, sc_d = run_gpu(x)
    racc, rsc = oracle.score_heads_from_qk(x.q, x.k, x.needle_start, x.needle_len, x.topk)
    np.testing.assert_allclose(acc_d.cpu().numpy(), racc, rtol=RTOL, atol=ATOL)
    np.testing.assert_allclose(sc_d.cpu().numpy(), rsc, rtol=5 * RTOL, atol=1e-6)
    return acc_d, racc


def test_one_row_group_ragged_context():
    # 64 rows per KV head (4 query heads x 16 steps); n is no multiple of the 32-key sub-tile or of a stripe of them
    check(wl.config4_qk(L=2, Hq=8, Hkv=2, T=16, n=4096 + 37, d=128))


def test_partial_row_group_head_dim_64_small_k():
    x = wl.config4_qk(L=1, Hq=8, Hkv=2, T=5, n=700, d=64, needle_len=5, seed_extra=1)
    x.topk = 8
    check(x)


@pytest.mark.parametrize("n,topk,d", [(40, 8, 128), (257, 16, 64), (1024, 64, 128), (1025, 1, 128), (5000, 64, 128)])
def test_short_contexts_and_the_largest_k(n, topk, d):
    # fewer keys than one stripe of sub-tiles, exactly the first chunk, one key more, K = 1 and the largest K
    x = wl.config4_qk(L=1, Hq=4, Hkv=2, T=7, n=n, d=d, needle_len=min(16, n // 2), seed_extra=10 + n)
    x.topk = topk
    check(x)


@pytest.mark.parametrize("n,topk,d", [(31, 7, 64), (288, 64, 128), (511, 64, 64), (512, 1, 128), (513, 64, 128), (1152, 33, 64),
                                      (1153, 64, 128)])
def test_equal_logits_at_the_kth_place_and_the_ends_of_chunks(n, topk, d):
    # every key twice: an odd K cuts a pair of equal logits, of which the lower position counts.  Around the first chunk
    # (512 keys, two sub-tiles per wave) and the rest that the second one takes along (up to 1152).
    # (K = n is left out: WS and Wide are then 1 minus a sum of fp32 weights, rounding of up to T * 2**-23 = 8e-7 where
    # the exact value is 0, which is above the 2e-7 that check() allows a small cell.)
    x = wl.config4_qk(L=1, Hq=4, Hkv=2, T=7, n=n, d=d, needle_len=min(16, n // 2), seed_extra=30 + n)
    x.k[:, :, 1::2] = x.k[:, :, 0:n - 1:2]
    x.topk = topk
    check(x)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("subtiles", [1, 2, 3, 4, 5, 6, 7, 8])
def test_last_chunks_in_which_some_waves_have_no_keys(subtiles, d):
    # the chunk after the first 512 keys has one to eight sub-tiles of 32, so that waves without one meet the others at
    # once: the queries that those still read and the statistics that these leave share one area of LDS.  With 1280
    # keys before the last sub-tiles, d = 128 cuts a head into ranges of 768 keys and 512 + 32 * subtiles - 5.
    for before, topk in ((512, 32), (1280, 33)):
        x = wl.config4_qk(L=1, Hq=16, Hkv=4, T=16, n=before + 32 * subtiles - 5, d=d, needle_len=16, seed_extra=100 + subtiles)
        x.topk = topk
        check(x)


@pytest.mark.parametrize("L,Hkv,T,n,topk,d", [(1, 1, 3, 16385, 33, 64), (1, 2, 16, 8000, 64, 128), (3, 2, 5, 2049, 1, 128), (2, 3, 40, 4100, 9, 64)])
def test_few_heads_cut_their_keys_into_ranges(L, Hkv, T, n, topk, d):
    # most keys twice, half the context apart, so that pairs of equal logits meet when the ranges are put together (K is
    # odd or large); the last range is short, the needle lies across two ranges where n allows it
    x = wl.config4_qk(L=L, Hq=2 * Hkv, Hkv=Hkv, T=T, n=n, d=d, needle_len=32, seed_extra=60 + n)
    x.k[:, :, n // 2:2 * (n // 2)] = x.k[:, :, :n // 2]
    x.needle_start, x.topk = 1024 - 16, topk
    check(x)


def test_several_row_groups_and_accumulation():
    import torch
    x = wl.config4_qk(L=1, Hq=8, Hkv=1, T=12, n=3000, d=128, seed_extra=2)      # 96 rows per KV head: 64 + 32
    acc_d, racc = check(x)
    acc_d, _ = run_gpu(x, acc_d)                                                 # a second call adds to the accumulators
    np.testing.assert_allclose(acc_d.cpu().numpy(), 2 * racc, rtol=RTOL, atol=ATOL)


def test_rows_of_equal_logits_go_through_the_fallback():
    # identical keys under the first KV head: every logit of its rows ties, T_k is the K lowest positions
    x = wl.config4_qk(L=1, Hq=4, Hkv=2, T=3, n=1500, d=128, needle_len=16, seed_extra=3, tie_rows=1)
    x.needle_start, x.topk = 8, 16                                                # needle [8, 24) against T_k = [0, 16)
    acc_d, racc = check(x)
    got = acc_d.cpu().numpy()
    np.testing.assert_allclose(got[0, 0, :3], [3 * 8 / 1500, 3 * 8 / 1500, 3 * 8 / 1500], rtol=1e-6)


def test_logits_rising_along_the_context_overflow_into_the_fallback():
    # keys of the first KV head = (j / n) * v: rows with q.v > 0 see logits that rise with the position, so every
    # chunk of keys beats the bound taken from the chunks before it and the candidate lists overflow; rows with
    # q.v < 0 have their top-K at the very beginning
    x = wl.config4_qk(L=1, Hq=8, Hkv=2, T=8, n=6000 + 13, d=128, needle_len=16, seed_extra=4)
    n = x.k.shape[2]
    v = np.random.default_rng(9).standard_normal(128).astype(np.float32)
    ramp = (np.arange(n, dtype=np.float32) / n * 6.0)[:, None] * v[None, :]
    x.k[0, 0] = wl.to_bf16_bits(ramp)
    x.needle_start = n - 40
    check(x)


def test_needle_run_shape_sampled_heads():
    # the shape bench.py times (32 layers x 32 query / 8 KV heads, 16 steps, 16384 keys); the oracle takes sampled heads
    x = wl.config4_qk()
    acc_d, sc_d = run_gpu(x)
    got_acc, got_sc = acc_d.cpu().numpy(), sc_d.cpu().numpy()
    rng = np.random.default_rng(0)
    for l, kv in zip(rng.integers(0, 32, size=6).tolist(), rng.integers(0, 8, size=6).tolist()):
        racc, rsc = oracle.score_heads_from_qk(x.q[l:l + 1, kv * 4:kv * 4 + 4], x.k[l:l + 1, kv:kv + 1], x.needle_start,
                                               x.needle_len, x.topk)
        np.testing.assert_allclose(got_acc[l, kv * 4:kv * 4 + 4], racc[0], rtol=RTOL, atol=ATOL)
        np.testing.assert_allclose(got_sc[l, kv * 4:kv * 4 + 4], rsc[0], rtol=5 * RTOL, atol=1e-6)
    # every row's cells sum to one row of mass
    np.testing.assert_allclose(got_acc[..., :4].sum(axis=-1), 16.0, rtol=1e-6)


@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("n", [2559, 2560, 2561, 3455, 3456, 3457, 4609, 5001, 6911, 6913, 10123])
def test_chunk_ends_of_both_schedules(n, equal):
    # d = 128, 256 heads that are not cut into ranges: from 2560 keys on half of the workgroups have their chunk ends half an octave earlier than the others (768, 1536, 3072,
    # 6144; an eighth more keys join the chunk before them: 3456, 6912).  The same two heads of queries and keys at every place give the same bits, those of the oracle;
    # `equal`: every key twice, and an odd K cuts a pair
    import torch
    x = wl.config4_qk(L=1, Hq=2, Hkv=2, T=9, n=n, d=128, needle_len=16, seed_extra=200 + n)
    if equal:
        x.k[:, :, 1::2] = x.k[:, :, 0:n - 1:2]
    x.topk = 33
    q, k = api.to_device(x.q, "bf16"), api.to_device(x.k, "bf16")
    racc, rsc = oracle.score_heads_from_qk(x.q, x.k, x.needle_start, x.needle_len, x.topk)
    acc, sc = api.score_heads_qk(q.repeat(32, 4, 1, 1), k.repeat(32, 4, 1, 1), x.needle_start, x.needle_len, x.topk)
    acc, sc = acc.view(128, 2, 5), sc.view(128, 2, 3)
    np.testing.assert_allclose(acc[0].cpu().numpy(), racc[0], rtol=RTOL, atol=ATOL)
    np.testing.assert_allclose(sc[0].cpu().numpy(), rsc[0], rtol=5 * RTOL, atol=1e-6)
    assert torch.equal(acc, acc[:1].expand_as(acc)) and torch.equal(sc, sc[:1].expand_as(sc))
