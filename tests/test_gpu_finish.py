"""Scoring, selection and copy in one launch (many segments, some of which keep more than 256 rows): the same outputs, bit for bit, as the scoring launch
followed by the selection and the gather.  Histories of 1 and 2048 positions and of one more (two launches), chunks with fewer kept rows than there are
of them, equal scores, empty segments, segments kept whole, windows alone; workgroups that wait for each other and such that leave."""

import numpy as np
import pytest

from paper_2508_15806_amd import api
from paper_2508_15806_amd import binding as B
from paper_2508_15806_amd import workloads as wl

pytestmark = pytest.mark.gpu

HEADER = 65536
POOLS = {"max": B.SLKV_POOL_MAX, "avg": B.SLKV_POOL_AVG, "none": B.SLKV_POOL_NONE}


def launches(run):
    import torch
    B.slkv_profile_begin(16)
    run()
    torch.cuda.synchronize()
    return [k for k, _ in B.slkv_profile_end(16)]


def outputs(call, run, scores):
    import torch
    outs = [call.kept_idx, call.k_out, call.v_out, call.out_offsets, call.pos_out] + ([call.importance, call.pooled] if scores else [])
    for x in outs:
        x.zero_()
    run()
    torch.cuda.synchronize()
    assert not bool(call.workspace[:HEADER].any())
    return [x.view(torch.uint8).clone() for x in outs]


# longest: rows of the longest segment
@pytest.mark.parametrize("dtype,G,d,w,pool,pool_kernel,longest,scores,equal", [
    ("bf16", 4, 128, 64, "max", 7, 2048 + 64, False, False), ("bf16", 4, 128, 64, "max", 7, 2049 + 64, False, False),
    ("f16", 4, 64, 8, "avg", 13, 2048 + 8, True, False), ("bf16", 2, 64, 16, "none", 1, 2000, True, False),
    ("bf16", 7, 128, 64, "max", 63, 1500, False, False), ("f16", 1, 128, 32, "max", 3, 1999, True, True), ("bf16", 4, 128, 32, "avg", 5, 1111, False, True)])
def test_many_segments(monkeypatch, dtype, G, d, w, pool, pool_kernel, longest, scores, equal):
    import torch
    nseq, Hkv = 66, 4
    caps = np.array([w + 1, 40 + w, 300, 2 * w], dtype=np.int32)
    rng = np.random.default_rng(longest + G)
    lens = [[0, w, w + 1, int(c)][i % 4] if rng.random() < 0.2 else int(c + t) for i, t in enumerate(rng.integers(1, 120, size=nseq)) for c in caps]
    lens[1], lens[8], lens[-2], lens[-4] = longest, min(1900, longest), longest - 1, longest   # one row kept beside the window, in the last one, of many chunks
    rc = wl.make_ragged_cache((601, longest, G), lens, nseq, G * Hkv, Hkv, d, w, dtype=dtype, bias_frac=0.04)
    if equal:
        rc.k_rows[::2] = rc.k_rows[0]
    call = api.RaggedCall(dtype, nseq, G * Hkv, Hkv, d, w, rc.in_offsets, caps, pool_kernel, POOLS[pool], debug_scores=scores)
    q, k, v = (api.to_device(x, dtype) for x in (rc.qwin, rc.k_rows, rc.v_rows))
    pos = torch.from_numpy(rc.pos_in).cuda()

    def run():
        call.run(q, k, v, pos)
    monkeypatch.setenv("SLKV_SELECT", "resident")
    assert "select" in launches(run)
    want = outputs(call, run, scores)
    assert (np.diff(call.out_offsets.cpu().numpy()) > 256).any()
    monkeypatch.delenv("SLKV_SELECT")
    assert ("select" not in launches(run)) == (longest <= 2048 + w)
    for limit in (None, "0", "3", None):
        if limit is None:
            monkeypatch.delenv("SLKV_MEET_US", raising=False)
        else:
            monkeypatch.setenv("SLKV_MEET_US", limit)
        for a, b in zip(outputs(call, run, scores), want):
            assert torch.equal(a, b)


def test_prompts(monkeypatch):
    # a layer call: token-major keys, an empty prompt, prompts below the window and below every capacity
    import torch
    lens, caps = [700, 0, 20, 310, 1000, 333] + [500] * 27, np.array([33, 400, 90, 120, 60, 50, 320, 64], dtype=np.int32)
    lay = wl.make_layer((602,), lens, 32, 8, 128, 32, dtype="bf16", bias_frac=0.03)
    T = int(lay.cu_seqlens[-1])
    call = api.LayerCall("bf16", len(lens), 32, 8, 128, 32, lay.cu_seqlens, caps, k_strides=(8 * 128, 128), v_strides=(8 * 128, 128))
    q, k, v = (api.to_device(x, "bf16") for x in (lay.qwin, lay.k, lay.v))
    k, v = (x.view(8, T, 128).transpose(0, 1).contiguous() for x in (k, v))
    got = {}
    for mode in ("resident", None):
        if mode:
            monkeypatch.setenv("SLKV_SELECT", mode)
        else:
            monkeypatch.delenv("SLKV_SELECT")
        assert ("gather" in launches(lambda: call.run(q, k, v))) == (mode is not None)
        for x in (call.kept_idx, call.k_out, call.v_out, call.out_offsets):
            x.zero_()
        call.run(q, k, v)
        torch.cuda.synchronize()
        got[mode] = [x.view(torch.uint8).clone() for x in (call.kept_idx, call.k_out, call.v_out, call.out_offsets)]
    for a, b in zip(got["resident"], got[None]):
        assert torch.equal(a, b)
