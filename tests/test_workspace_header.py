"""The header of a call's workspace is zero before every call: also after one that failed between its launches, and on another stream than the one that
filled it, once that has been waited for."""

import numpy as np
import pytest

from paper_2508_15806_amd import api
from paper_2508_15806_amd import binding as B
from paper_2508_15806_amd import workloads as wl


@pytest.mark.parametrize("kind", ["layer", "ragged"])
@pytest.mark.parametrize("status,cleared", [(B.SLKV_ERR_HIP, True), (6, False)])
def test_cleared_after_a_call_that_failed(monkeypatch, kind, status, cleared):
    if kind == "layer":
        call = api.LayerCall("bf16", 1, 4, 2, 64, 8, np.array([0, 300], dtype=np.int64), np.array([20, 30], dtype=np.int32), device="cpu")
    else:
        call = api.RaggedCall("bf16", 1, 4, 2, 64, 8, np.array([0, 300, 500], dtype=np.int64), np.array([20, 30], dtype=np.int32), device="cpu")

    def failing(*args):
        call.workspace[:128] = 1                                  # counters of a launch whose selection never came
        raise B.SlkvError(status, "launch failed")
    for name in ("slkv_compress_layer", "slkv_recompress_layer"):
        monkeypatch.setattr(B, name, failing)
    with pytest.raises(B.SlkvError) as ei:
        call.run(None, None, None)
    assert ei.value.status == status
    assert bool(call.workspace[:B.SLKV_WORKSPACE_HEADER_BYTES].any()) != cleared      # (what was refused has launched nothing)


@pytest.mark.gpu
def test_first_call_on_another_stream():
    # the fill stands behind 50 ms of another kernel on the constructing stream, in memory that held other values; the stream of the first call waits for it
    import torch
    lens, caps = [4000, 2500], np.array([60, 300, 90, 80], dtype=np.int32)
    lay = wl.make_layer((701,), lens, 16, 4, 128, 32, dtype="bf16", bias_frac=0.03)
    q, k, v = (api.to_device(x, "bf16") for x in (lay.qwin, lay.k, lay.v))

    def make():
        return api.LayerCall("bf16", 2, 16, 4, 128, 32, lay.cu_seqlens, caps, debug_scores=True)
    ref = make()
    ref.run(q, k, v)
    torch.cuda.synchronize()
    torch.full((ref.workspace.numel(),), 255, dtype=torch.uint8, device="cuda")      # (freed at once: the next workspace takes its place)
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda._sleep(100_000_000)
    call = make()
    other.wait_stream(torch.cuda.current_stream())
    call.run(q, k, v, stream=other)
    torch.cuda.synchronize()
    assert not bool(call.workspace[:B.SLKV_WORKSPACE_HEADER_BYTES].any())
    for a, b in ((call.kept_idx, ref.kept_idx), (call.k_out, ref.k_out), (call.v_out, ref.v_out), (call.importance, ref.importance), (call.pooled, ref.pooled)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
