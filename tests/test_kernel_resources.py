"""The GEMM kernels keep their accumulators in registers: none spills.

A tile's accumulators and two sets of fragments leave the widest tiles few
registers to spare, and an epilogue that needs more goes to scratch memory
without a word from the compiler, at several per cent of the launch.  The
kernels are compiled for the GPU with the library's own flags, and the compiler's
resource report is read (CPU only)."""
import importlib.util
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _build_script():
    spec = importlib.util.spec_from_file_location("_sc_build", os.path.join(ROOT, "paper_2609_22283_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    return b


def test_gemm_kernels_do_not_spill(tmp_path):
    b = _build_script()
    if shutil.which(b.HIPCC) is None:
        pytest.skip("needs hipcc")
    cmd = [b.HIPCC] + b.COMMON + ["-x", "hip", "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                                  os.path.join(b.CSRC, "gemm.hip"), "-o", str(tmp_path / "gemm.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    reports = r.stderr.split("Function Name: ")[1:]
    gemms = [t for t in reports if "gemm_bf16_kernel" in t.split()[0]]
    assert len(gemms) >= 28  # seven or eight tiles of four epilogues
    for t in gemms:
        spills = [int(n) for n in re.findall(r"(?:SGPRs|VGPRs) Spill: (\d+)", t)]
        scratch = [int(n) for n in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", t)]
        assert len(spills) == 2 and len(scratch) == 1
        assert spills[1] == 0 and scratch[0] == 0, t.split()[0]
