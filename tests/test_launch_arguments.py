"""A kernel whose arguments exceed 4 KiB does not compile: launch.h adds up the arguments of the kernel that is launched, not those of one among them."""

import os
import subprocess

import pytest

from paper_2508_15806_amd import build as b


@pytest.mark.parametrize("words,compiles", [(1020, True), (1021, False)])      # 4 bytes each, and a pointer and a number behind them
def test_bound(tmp_path, words, compiles):
    src = tmp_path / "launch.hip"
    src.write_text('#include "launch.h"\n'
                   "struct Words { int w[%d]; };\n"
                   "__global__ void kernel(const Words a, const float* p, int n) {}\n"
                   "void launch(hipStream_t st) { SLKV_LAUNCH(kernel, dim3(1), dim3(64), 0, st, Words{}, (const float*)nullptr, 1); }\n" % words)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    run = subprocess.run([hipcc] + b.COMMON + b.DEVICE + ["--offload-host-only", "-fsyntax-only", str(src)], capture_output=True, text=True, timeout=300)
    assert (run.returncode == 0) == compiles, run.stderr[-2000:]
    assert compiles or "kernel arguments are at most 4 KiB" in run.stderr
