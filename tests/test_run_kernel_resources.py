"""Resource use of the run kernels, from the compiler's own report: no scratch, and
no vector registers spilled (their launch shapes were chosen by it)."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1202_2355_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
UNITS = ("m2m_run_f32.hip", "m2m_run_f32s.hip", "m2m_run_f64.hip", "m2m_run_f64s.hip")


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None,
                    reason="hipcc not available")
def test_no_run_kernel_spills_vector_registers():
    from paper_1202_2355_amd.build import HIPCC_FLAGS
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC", "-Wall")]
    procs = [subprocess.Popen([HIPCC, *flags, "--offload-device-only", "-Rpass-analysis=kernel-resource-usage",
                               "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", "-o", os.devnull,
                               os.path.join(CSRC, u)], stdout=subprocess.DEVNULL, stderr=subprocess.PIPE, text=True)
             for u in UNITS]
    kernels, spills, name = 0, [], None
    for p in procs:
        _, err = p.communicate()
        assert p.returncode == 0, err[-2000:]
        for line in err.splitlines():
            if m := re.search(r"Function Name: (\S+)", line):
                name = m.group(1)
                kernels += 1
            elif m := re.search(r"(ScratchSize \[bytes/lane\]|VGPRs Spill): (\d+)", line):
                if int(m.group(2)) > 0:
                    spills.append((name, m.group(1), int(m.group(2))))
    # (5 kinds of observables) x (FP32 512 and 1024 threads, FP64 512) x (start known or
    # not, batch, smoothed)
    assert kernels == 60, kernels
    assert not spills, spills[:10]
