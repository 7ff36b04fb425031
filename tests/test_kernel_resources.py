"""What the compiler reports of the kernels' registers: the mass pass of large batches is bound by its operations, and
scalar registers kept from the accept decision on are spilled to vector registers and back in its loops
(64 x 152064 bf16: 17.2 us with 30 of them, 16.35 without)."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _report(source, tmp_path):
    spec = importlib.util.spec_from_file_location("_sv_build", os.path.join(ROOT, "paper_2509_24328_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    cmd = [HIPCC] + [f for f in build.FLAGS if f != "-shared"] + build.OWN_FLAGS.get(source, []) + [
        "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(build.CSRC, source), "-o",
        str(tmp_path / "x.o")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    out, name = {}, None
    for line in res.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m[1]
            out[name] = {}
        m = re.search(r"remark:.*?(\w+) Spill: (\d+)", line)
        if m:
            out[name][m[1]] = int(m[2])
    return out


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no compiler")
def test_the_mass_pass_of_large_batches_spills_nothing(tmp_path):
    kernels = _report("verify_sample.hip", tmp_path)
    mass = {n: k for n, k in kernels.items() if "verify_mass_kernel" in n}
    assert len(mass) == 16
    for n, k in kernels.items():
        assert k["VGPRs"] == 0, n
    for n, k in mass.items():                            # <type, cutoffs, chained, a granule per workgroup>
        cut, chained, wide = (m == "1" for m in re.search(r"Lb(\d)ELb(\d)ELb(\d)E", n).groups())
        if not chained:
            assert k["SGPRs"] == 0, (n, k)
    # the other kernels of the sampling stage: what they spill, and no more.  The draw that weighs its runs one at a time leaves 78
    # scalar registers, two workgroups of 1024 lanes to a compute unit.
    for n, k in kernels.items():
        if "verify_mass_of_whole_kernel" in n:
            chained, wide = (m == "1" for m in re.search(r"Lb(\d)ELb(\d)E", n).groups())
            assert k["SGPRs"] <= (20 if chained and not wide else 0), (n, k)
        if "verify_draw_kernel" in n:
            assert k["SGPRs"] <= (28 if "Li1024ELi4ELi1E" in n else 0), (n, k)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no compiler")
def test_the_statistics_of_short_rows_spill_nothing(tmp_path):
    """Four registers spilled by the form of four bf16 places, two workgroups to a compute unit, were 8 % in the mean and up to 18 % of its time."""
    kernels = {n: k for n, k in _report("row_stats.hip", tmp_path).items() if "row_stats_terms_kernel" in n}
    assert len(kernels) == 19
    for n, k in kernels.items():
        assert k["VGPRs"] == 0 and k["SGPRs"] == 0, (n, k)
