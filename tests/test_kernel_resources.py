"""What the compiler gives the kernels whose speed hangs on it: registers, spills and the waves that fit a SIMD (no GPU
needed, the device code is compiled once more with remarks)."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _resources(unit):
    """{kernel: (vector registers, spilled ones, waves per SIMD)} of csrc/<unit>.hip"""
    spec = importlib.util.spec_from_file_location("ecgemm_hip_build", os.path.join(ROOT, "paper_2203_03341_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    res = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                          os.path.join(build.CSRC, unit + ".hip"), "-o", os.devnull], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    found, current = {}, None
    for line in res.stderr.splitlines():
        m = re.search(r"remark: .*?(Function Name|VGPRs|VGPRs Spill|Occupancy \[waves/SIMD\]): (\S+)", line)
        if m and m[1] == "Function Name":
            current = found.setdefault(m[2], {})
        elif m and current is not None:
            current[m[1]] = int(m[2])
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True).stdout.split("\n")
    return {re.sub(r"^void ecgemm::|\(.*", "", name): (r["VGPRs"], r["VGPRs Spill"], r["Occupancy [waves/SIMD]"])
            for name, r in zip(names, found.values())}


def test_the_split_of_four_tiles_keeps_every_wave_of_a_simd():
    """The kernels that live on loads in flight: at most 64 vector registers, so that eight waves fit a SIMD, no spills."""
    four_tiles = {name: r for name, r in _resources("kernels_split").items() if re.match(r"split_kernel<\d, 1, ", name)}
    assert len(four_tiles) == 7, four_tiles
    for name, (registers, spilled, waves) in four_tiles.items():
        assert registers <= 64 and spilled == 0 and waves == 8, (name, registers, spilled, waves)
