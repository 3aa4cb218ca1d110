"""What the compiler reports for the kernels that keep small arrays in
registers: no scratch (an array indexed by a run-time value would go there)."""
import os
import re
import subprocess

from paper_2512_01251_amd import build_lib


def _scratch(src):
    """{kernel: scratch bytes per lane} of one source, compiled with the library's flags."""
    flags = [f for f in build_lib.FLAGS if f != "-shared"]
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-c",
           "-Rpass-analysis=kernel-resource-usage", os.path.join(build_lib.HERE, "csrc", src), "-o", os.devnull]
    r = subprocess.run(cmd, capture_output=True, text=True, check=True)
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    sizes = re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)
    assert names and len(names) == len(sizes)
    return dict(zip(names, map(int, sizes)))


def test_refinement_kernels_use_no_scratch():
    scratch = _scratch("geo_refine.hip")
    assert any("k_ref_nbr" in k for k in scratch)
    assert set(scratch.values()) == {0}, scratch
