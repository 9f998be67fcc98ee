"""Compiler output check (no GPU): the reduction's exchanges that the language's memory model does not cover by itself have the form that they rely
on."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Name -> assembly of the kernels of tridiag_columns.hip."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    from paper_2503_10501_amd import build
    out = tmp_path_factory.mktemp("forms") / "x.s"
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "tridiag_columns.hip"), "-o", str(out)], check=True,
                   capture_output=True, timeout=600)
    return {m[1]: m[2] for m in re.finditer(r"^(_ZN2tc\S+):.*?\n(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S)}


def test_lanes_that_exchange_through_lds_are_kept_in_order(kernels):
    # one barrier for the wavefront where its lanes' results leave and one at the end of a column, in each of the eight classes of columns
    last = [code for name, code in kernels.items() if "tridiag_last_kernel" in name]
    assert len(last) == 1
    assert last[0].count("; wave barrier") >= 16
