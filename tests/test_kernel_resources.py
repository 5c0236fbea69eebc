"""Register spills of the convolution kernels, as the compiler reports them (CPU only:
the source is compiled for gfx950, nothing runs). The kernels of a run-time image size
serve every size but 28 x 28; the compile-time instances serve that one."""
import os
import re
import subprocess

import pytest

from paper_1812_04352_amd import build as B


def scratch(src, tmp_path):
    """Scratch bytes per lane of each kernel, by demangled name."""
    r = subprocess.run([B.HIPCC, *B.FLAGS, "-Rpass-analysis=kernel-resource-usage", "--offload-device-only", "-x", "hip",
                        "-c", os.path.join(B.CSRC, src), "-o", str(tmp_path / "k.o")], capture_output=True, text=True,
                       timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    found = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", r.stderr, re.S)
    names = subprocess.run(["c++filt"], input="\n".join(n for n, _ in found), capture_output=True, text=True).stdout
    return {n: int(s) for n, (_, s) in zip(names.split("\n"), found)}


def test_convolution_kernels_hardly_spill(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no compiler")
    use = scratch("lp_conv.hip", tmp_path)
    sweeps = {n: s for n, s in use.items() if re.search(r"k_(fwd|adj)<", n)}
    run_time = {n: s for n, s in sweeps.items() if re.search(r"<\d, 0, 0,", n)}
    assert len(sweeps) == 80 and len(run_time) == 40
    # the fp32 instructions' kernels had 6972 (run-time sizes) and 1116 in all, at most 1284 in one
    assert sum(run_time.values()) <= 500 and max(run_time.values()) <= 150, run_time
    assert sum(sweeps.values()) - sum(run_time.values()) <= 400, sweeps
    assert all(s == 0 for n, s in use.items() if n not in sweeps), use
