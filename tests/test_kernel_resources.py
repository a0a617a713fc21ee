"""Register use of the backward's matrix-core kernels, from the compiler's own
report for the flags of the build (no GPU needed).

A register tuple that this compiler spills partly to accumulation registers and
partly to scratch memory can come back incomplete: a rotary key kernel that kept
gK and gV through its window loop (d = 128, three column tiles, all 512
registers and 116 bytes of scratch) put two of the four registers of one gV
operand into a254 and a255 and the other two into scratch, and reloaded all but
a255, so that dv was wrong. No kernel may therefore use scratch beside accumulation registers, and
the rotary key kernels, the widest ones, spill nothing."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _builder():
    spec = importlib.util.spec_from_file_location(
        "dar_build_flags", os.path.join(ROOT, "paper_2606_18587_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _resources(source):
    b = _builder()
    if not os.path.exists(b._hipcc()):
        pytest.skip("no hipcc")
    cmd = [b._hipcc(), *b.HIPCC_FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
           "-c", os.path.join(b.CSRC, source), "-o", os.devnull]
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-2000:]
    kernels = {}
    for key, value in re.findall(r"remark: [^\n]*?(Function Name|AGPRs|ScratchSize \[bytes/lane\]|VGPRs Spill): (\S+)",
                                 p.stdout):
        if key == "Function Name":
            cur = kernels[value] = {}
        else:
            cur[key.split()[0]] = int(value)
    return kernels


def test_no_spill_beside_accumulation_registers():
    kernels = _resources("backward_mfma.hip")
    keys = [n for n in kernels if "bwd_rope_keys_kernel" in n]
    assert len(kernels) > 20 and len(keys) == 5, sorted(kernels)
    for name, r in kernels.items():
        assert r["AGPRs"] == 0 or r["ScratchSize"] == 0, (name, r)
    for name in keys:
        assert kernels[name]["ScratchSize"] == 0 and kernels[name]["VGPRs"] == 0, (name, kernels[name])
