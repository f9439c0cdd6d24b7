"""Both scoring passes in one launch, whose workgroups meet in between: the same scores, bit for bit, as the two launches (which calls take
that are selected by blocks), whether the workgroups of a segment wait for each other or leave and the last one completes their chunks."""

import numpy as np
import pytest

from paper_2508_15806_amd import api
from paper_2508_15806_amd import binding as B
from paper_2508_15806_amd import workloads as wl

pytestmark = pytest.mark.gpu

HEADER = 65536


def results(call, run):
    import torch
    outs = [call.kept_idx, call.k_out, call.v_out, call.importance, call.pooled]
    for x in outs:
        x.zero_()
    run()
    torch.cuda.synchronize()
    assert not bool(call.workspace[:HEADER].any())          # the meeting places are left as they were found
    return [x.view(torch.uint8).clone() for x in outs]


def launches(run):
    import torch
    B.slkv_profile_begin(16)
    run()
    torch.cuda.synchronize()
    return [k for k, _ in B.slkv_profile_end(16)]


def compare(monkeypatch, call, run, together=True):
    import torch
    monkeypatch.delenv("SLKV_MEET_US", raising=False)
    monkeypatch.setenv("SLKV_SELECT", "blocks")
    assert "score_stats" in launches(run)
    two = results(call, run)
    monkeypatch.delenv("SLKV_SELECT")
    assert ("score_stats" not in launches(run)) == together
    for limit in (None, "0", "0", "3", None):               # (0: nearly all leave; 3 us: some do)
        if limit is not None:
            monkeypatch.setenv("SLKV_MEET_US", limit)
        else:
            monkeypatch.delenv("SLKV_MEET_US", raising=False)
        for _ in range(3):
            for a, b in zip(results(call, run), two):
                assert torch.equal(a, b)


# 32 to 512 query rows, segments of one chunk, of one key more, of several; the ends of chunks and of tile pairs
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("Hq,Hkv,w,d,lens", [
    (2, 2, 32, 128, [32 + 1, 32 + 128, 32 + 129, 700]), (8, 2, 16, 64, [5000]), (8, 2, 32, 128, [32 + 255, 1300, 90]),
    (16, 4, 64, 64, [4000, 64 + 513]), (32, 8, 64, 128, [9000]), (14, 2, 64, 128, [3000, 200]), (16, 2, 64, 64, [2000])])
def test_layer(monkeypatch, dtype, Hq, Hkv, w, d, lens):
    lay = wl.make_layer((401, Hq, w, d), lens, Hq, Hkv, d, w, dtype=dtype, bias_frac=0.04)
    call = api.LayerCall(dtype, len(lens), Hq, Hkv, d, w, lay.cu_seqlens, np.array([w + 20 + 31 * h for h in range(Hkv)], dtype=np.int32), debug_scores=True)
    q, k, v = (api.to_device(x, dtype) for x in (lay.qwin, lay.k, lay.v))
    compare(monkeypatch, call, lambda: call.run(q, k, v))


# fp32 and E4M3 keys: one and several blocks of query rows, key groups that all stay in registers and more of them, waves that share a
# group, segments of one chunk among longer ones
@pytest.mark.parametrize("dtype,Hq,Hkv,w,d,lens,together", [
    ("f32", 4, 4, 32, 64, [1024], True), ("f32", 2, 2, 32, 128, [32 + 1, 32 + 33, 700], True), ("f32", 8, 2, 64, 128, [64 + 31, 1300], True),
    ("f32", 16, 2, 64, 64, [900, 300], True), ("f32", 8, 8, 64, 64, [3000], False), ("bf16_kv8", 8, 2, 16, 64, [2000], True),
    ("bf16_kv8", 32, 8, 64, 128, [20000], True), ("bf16_kv8", 14, 2, 64, 128, [3000, 200], True), ("bf16_kv8", 16, 2, 32, 128, [32 + 1, 32 + 64, 32 + 65, 1500], True),
    ("bf16_kv8", 32, 8, 32, 128, [20000, 31000, 9000], True), ("bf16_kv8", 32, 8, 32, 128, [8192], False)])
def test_keys_in_registers(monkeypatch, dtype, Hq, Hkv, w, d, lens, together):
    lay = wl.make_layer((404, Hq, w, d), lens, Hq, Hkv, d, w, dtype=dtype, bias_frac=0.04)
    call = api.LayerCall(dtype, len(lens), Hq, Hkv, d, w, lay.cu_seqlens, np.array([w + 20 + 31 * h for h in range(Hkv)], dtype=np.int32), debug_scores=True)
    q, k, v = (api.to_device(x, dtype) for x in (lay.qwin, lay.k, lay.v))
    compare(monkeypatch, call, lambda: call.run(q, k, v), together)


def test_most_chunks_of_a_segment(monkeypatch):
    # one KV head: as many chunks as a meeting place counts take one launch, more take two
    for n, together in ((48 * 128 + 32, True), (48 * 128 + 33, False)):
        lay = wl.make_layer((402, n), [n], 4, 1, 128, 32, dtype="bf16", bias_frac=0.02)
        call = api.LayerCall("bf16", 1, 4, 1, 128, 32, lay.cu_seqlens, np.array([100], dtype=np.int32), debug_scores=True)
        q, k, v = (api.to_device(x, "bf16") for x in (lay.qwin, lay.k, lay.v))
        compare(monkeypatch, call, lambda: call.run(q, k, v), together)


def test_cache_of_many_segments(monkeypatch):
    # 256 segments of one to eight chunks: the table by sequence and head
    import torch
    caps = np.array([107, 1834, 111, 132, 119, 110, 143, 127], dtype=np.int32)
    rng = np.random.default_rng(5)
    lens = [int(c + t) for t in rng.integers(1, 129, size=32) for c in caps]
    rc = wl.make_ragged_cache((403,), lens, 32, 32, 8, 128, 64, dtype="bf16", bias_frac=0.03)
    call = api.RaggedCall("bf16", 32, 32, 8, 128, 64, rc.in_offsets, caps, debug_scores=True)
    q, k, v = (api.to_device(x, "bf16") for x in (rc.qwin, rc.k_rows, rc.v_rows))
    pos = torch.from_numpy(rc.pos_in).cuda()
    compare(monkeypatch, call, lambda: call.run(q, k, v, pos))


# finish: the launch also selects and copies (more than 64 segments, histories of at most 2048, some that keep more than 256 rows)
@pytest.mark.parametrize("finish", [False, True])
def test_three_streams(monkeypatch, finish):
    # three calls of nearly as many workgroups as the chip holds, started together: none may wait for another
    import torch
    if finish:
        caps = np.array([107, 1834, 111, 132, 119, 110, 143, 127], dtype=np.int32)
        lens = [int(c + t) for t in np.random.default_rng(6).integers(1, 129, size=32) for c in caps]
        rc = wl.make_ragged_cache((406,), lens, 32, 32, 8, 128, 64, dtype="bf16", bias_frac=0.03)
        calls = [api.RaggedCall("bf16", 32, 32, 8, 128, 64, rc.in_offsets, caps) for _ in range(3)]
        args = [api.to_device(x, "bf16") for x in (rc.qwin, rc.k_rows, rc.v_rows)] + [torch.from_numpy(rc.pos_in).cuda()]
    else:
        lens, caps = [4000] * 16, np.array([60, 300, 90, 80, 70, 200, 100, 64], dtype=np.int32)
        lay = wl.make_layer((404,), lens, 32, 8, 128, 32, dtype="bf16", bias_frac=0.03)
        calls = [api.LayerCall("bf16", 16, 32, 8, 128, 32, lay.cu_seqlens, caps) for _ in range(3)]
        args = [api.to_device(x, "bf16") for x in (lay.qwin, lay.k, lay.v)]

    def outs(call):
        return [call.kept_idx, call.k_out, call.v_out, call.out_offsets] + ([call.pos_out] if finish else [])
    monkeypatch.setenv("SLKV_SELECT", "blocks")
    assert "score_stats" in launches(lambda: calls[0].run(*args))
    want = [x.view(torch.uint8).clone() for x in outs(calls[0])]
    monkeypatch.delenv("SLKV_SELECT")
    took = launches(lambda: calls[0].run(*args))
    assert "score_stats" not in took and ("select" in took) != finish
    streams = [torch.cuda.Stream() for _ in calls]
    for _ in range(5):
        for call in calls:
            for x in outs(call):
                x.zero_()
        torch.cuda.synchronize()
        for _ in range(4):
            for call, s in zip(calls, streams):
                call.run(*args, stream=s)
        torch.cuda.synchronize()
        for call in calls:
            assert not bool(call.workspace[:HEADER].any())
            for x, y in zip(outs(call), want):
                assert torch.equal(x.view(torch.uint8), y)


def test_streams_long_passes():
    # passes of 140 us, on more streams than the chip has room for: workgroups that left each other before a pass was over would leave nearly all
    # chunks to the few that come last (three times as long)
    import time
    import torch
    lens, caps = [32768] * 8, np.array([107, 1834, 111, 132, 119, 110, 143, 127], dtype=np.int32)
    gen = torch.Generator(device="cuda").manual_seed(7)
    q = torch.randn(8, 32, 64, 128, generator=gen, device="cuda").to(torch.bfloat16)
    kv = [torch.randn(2, 8, sum(lens), 128, generator=gen, device="cuda").to(torch.float8_e4m3fn).view(torch.uint8) for _ in range(4)]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    calls = [api.LayerCall("bf16_kv8", 8, 32, 8, 128, 64, cu, caps) for _ in range(4)]
    assert "score_stats" not in launches(lambda: calls[0].run(q, *kv[0]))

    def us_a_call(streams):
        took = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(15):
                for call, x, s in zip(calls, kv, streams):
                    call.run(q, *x, stream=s)
            torch.cuda.synchronize()
            took.append((time.perf_counter() - t0) / (15 * len(calls)) * 1e6)
        return float(np.median(took))
    streams = [torch.cuda.Stream() for _ in range(4)]
    us = [us_a_call([streams[i % n] for i in range(4)]) for n in (1, 2, 3, 4)]
    assert max(us) < 1.35 * us[0], us
