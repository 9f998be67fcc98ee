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


def test_near_and_far_stores_have_the_forms_that_the_polls_find(kernels):
    columns = [code for name, code in kernels.items() if "tridiag_columns_kernel" in name]
    assert len(columns) == 9
    for code in columns:
        flags = [line.split(";")[0].split() for line in code.splitlines() if re.match(r"\s(global|flat)_(store|load)_dwordx2 ", line)]
        flags = [(f[0], {x for x in f if x in ("sc0", "sc1", "nt")}) for f in flags]
        stores = [x for op, x in flags if op == "global_store_dwordx2"]
        near, far = stores.count({"sc0"}), stores.count({"sc1"})
        assert far > 0 and all(not x or x in ({"sc0"}, {"sc1"}) for x in stores) and not any(op.startswith("flat") for op, _ in flags)
        assert near == far
        assert sum(x == {"sc1"} for op, x in flags if op == "global_load_dwordx2") > 0
