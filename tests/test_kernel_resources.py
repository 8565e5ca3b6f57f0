"""No kernel of the library spills registers to scratch memory.

The step kernels are written to the register budget of their occupancy (128 registers per lane at
16 wavefronts per workgroup for the resident kernel, 256 or 512 for the streaming ones); a helper
that grows by a few registers tips them over without any error, and the spill traffic then costs
several per cent of throughput.  The compiler reports the figures; this test reads them.
"""
import os
import re
import shutil
import subprocess
import tempfile
from functools import lru_cache
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _resource_report(src, flags, hipcc, csrc):
    with tempfile.TemporaryDirectory() as tmp:
        cmd = [hipcc, *flags, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
               os.path.join(csrc, src), "-o", os.path.join(tmp, "dev.o")]
        out = subprocess.run(cmd, check=True, capture_output=True, text=True, timeout=600).stderr
    kernels, name = {}, None
    for line in out.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            kernels[name] = {}
            continue
        m = re.search(r"remark:\s+(VGPRs Spill|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]): (\d+)", line)
        if m and name:
            kernels[name][m.group(1)] = int(m.group(2))
    return kernels


@lru_cache(maxsize=1)
def _reports():
    from paper_1810_08313_amd import build
    hipcc = build.HIPCC if os.path.exists(build.HIPCC) else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not available")
    sources = [s for s in build.SOURCES if s != "lc_api.hip"]   # lc_api.hip holds host code only
    with ThreadPoolExecutor(max_workers=len(sources)) as ex:
        return sources, list(ex.map(lambda s: _resource_report(s, build.FLAGS, hipcc, build.CSRC), sources))


def test_no_kernel_spills_registers():
    sources, reports = _reports()
    seen = 0
    for src, kernels in zip(sources, reports):
        assert kernels, src
        for name, r in kernels.items():
            seen += 1
            assert r.get("VGPRs Spill", 0) == 0, (src, name, r)
            assert r.get("ScratchSize [bytes/lane]", 0) == 0, (src, name, r)
    assert seen >= 40   # forward, backward, head, resident, first-layer and streaming instances


# (source, part of the mangled name, how many instances, wavefronts per SIMD)
OCCUPANCY = [
    # bf16 (DF16b), 128 samples (8 tiles), whole rows (access modes 1 and 2), no dA: three workgroups per compute unit
    ("lc_mlp_kernels.hip", r"backward_kernelIDF16bLi8ELi[12]ELb0ELb1E", 4, 3),
    # ... with dA, any rows of 64 columns and more: two
    ("lc_mlp_kernels.hip", r"backward_kernelIDF16bLi8ELi[123]ELb0ELb0E", 3, 2),
    # either operand type, up to 64 samples, no dA: three
    ("lc_mlp_kernels.hip", r"backward_kernelI(f|DF16b)Li[24]ELi[123]ELb0ELb1E", 12, 3),
    # first-layer kernel up to 64 samples: two wavefronts per SIMD, of two workgroups or one of eight
    ("lc_first_layer_kernels.hip", r"first_layer_kernelI(f|DF16b)Li[24]E", 20, 2),
]


@pytest.mark.parametrize("src,name,count,waves", OCCUPANCY)
def test_workgroups_that_share_a_compute_unit(src, name, count, waves):
    """Rules that choose these instances were measured with so many wavefronts on a SIMD at once."""
    sources, reports = _reports()
    found = {k: r for k, r in reports[sources.index(src)].items() if re.search(name, k)}
    assert len(found) == count, sorted(found)
    for k, r in found.items():
        assert r["Occupancy [waves/SIMD]"] >= waves, (k, r)
