"""The register DFTs of the operator product's transforms, run on the host:
each radix against the definition of the DFT (a half-zero butterfly must not
read its zero half, which is NaN), and each length's sequence of radices
against the one that a run-time plan makes of the factors 16, 8, 4, 2, 3, 5.

Tolerances: a radix of up to 16 on values of size one sums 16 terms of one in
double, 16 x 16 x 1.1e-16 = 3e-14, doubled; a length's composite radices may
not lose against the plan's, 2% beyond (60 random vectors per length leave
about half a percent)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("radix") / "radix_driver")
    csrc = os.path.join(ROOT, "paper_1902_02196_amd", "csrc")
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O2", "-std=c++17", "-ffp-contract=fast",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w", "-I", csrc,
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "native", "radix_driver.hip"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=120).stdout
    return [line.split() for line in out.splitlines()]


def test_every_radix_is_a_dft(lines):
    rows = [r for r in lines if r[0] == "radix"]
    assert len(rows) == 11 * 2 + 7 * 2
    for r in rows:
        assert float(r[4]) < 6e-14, r   # false for NaN


def test_no_length_loses_accuracy_to_its_radices(lines):
    rows = [r for r in lines if r[0] == "length"]
    assert len(rows) == 38
    for _, n, mix, plan in rows:
        assert float(mix) <= 1.02 * float(plan), (n, mix, plan)
