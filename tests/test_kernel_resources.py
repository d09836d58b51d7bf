"""What the compiler gives the kernels (its own resource report, on the CPU): the wavefronts that fit a
SIMD, registers and scratch.  Results do not depend on any of it, but the times that the comments beside
the kernels state do."""
import re
import shutil
import subprocess

import pytest

from paper_2004_14020_amd import build

pytestmark = pytest.mark.skipif(shutil.which(build.hipcc()) is None, reason="hipcc not available")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel with its template arguments: {quantity: value}}"""
    obj = str(tmp_path_factory.mktemp("resources") / "kernels.o")
    res = subprocess.run([build.hipcc(), *build.flags(), "--cuda-device-only", "-c", f"{build.HERE}/csrc/kernels.hip",
                          "-o", obj, "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-2000:]
    reports = res.stderr.split("Function Name: ")[1:]
    names = subprocess.run(["c++filt"], input="\n".join(r.split()[0] for r in reports), capture_output=True, text=True,
                           check=True).stdout.splitlines()
    short = [re.search(r"(k_\w+(<.*?>)?)\(", n).group(1) for n in names]
    found = {s: {k.strip(): int(v) for k, v in re.findall(r"remark: [^\n]*?  +([A-Z][^:\n]*): (\d+)", r)}
             for s, r in zip(short, reports)}
    assert len(found) == len(reports) and any(s.startswith("k_walk<") for s in found)
    return found


def test_long_walks_run_one_workgroup_per_compute_unit(kernels):
    walks = {n: r for n, r in kernels.items() if n.startswith("k_tree_walk<") or re.match(r"k_walk<.*, [48]>", n)}
    assert len(walks) > 20
    # 1024 lanes are four wavefronts per SIMD
    assert {n: r["Occupancy [waves/SIMD]"] for n, r in walks.items() if r["Occupancy [waves/SIMD]"] != 4} == {}


def test_no_kernel_spills_vector_registers(kernels):
    quantities = ("VGPRs Spill", "ScratchSize [bytes/lane]")
    assert {n: r for n, r in kernels.items() if any(r[q] for q in quantities)} == {}


def test_copies_address_both_sides_with_one_offset(kernels):
    copies = {n: r["VGPRs"] for n, r in kernels.items() if n.startswith("k_copy<")}
    # a 128-bit value, a 64-bit offset, the counter and the lane
    assert len(copies) == 8 and max(copies.values()) <= 10, copies
