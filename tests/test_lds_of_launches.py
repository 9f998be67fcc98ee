"""Host test (no GPU): a launch whose LDS, what the kernel declares and what the launch adds, is beyond 64 KB has asked for it.  What kernels
declare is read from the compiler's output, what launches add from the calls of the stand-in for the HIP runtime of test_stream_order.py."""
import os
import re
import shutil
import subprocess
import sys

import pytest

from tests.test_stream_order import LIB, ROOT, STAND_IN, pytestmark  # noqa: F401

PROGRAM = r"""
import ctypes, sys
sys.path.insert(0, %r)
from paper_2503_10501_amd import binding as tc
lib, ptr = tc.load_library(), 1 << 20
for n in map(int, sys.argv[1].split(",")):
    p = tc.make_params(seq_len=n, vis_start=0, n_vis=n, n_heads=4, head_dim=128, hidden_dim=512, dtype=tc.TC_BF16, k_prune=2, k_final=2, batch=1)
    assert lib.tc_ipgs_score(ctypes.byref(p), ptr, ptr, ptr, None, None, None, ptr, tc.tc_workspace_bytes(p), None) == 0
"""
# around the sizes where td_orthogonalise_kernel (44 bytes a token and more) and td_twisted_kernel (16 and 24 KB) come to 64 KB
SIZES = [64, 576, 1344, 1352, 1353, 1354, 1360, 1728, 2576, 2592, 2593, 2608, 2609, 2640, 2880, 3000, 3456]


@pytest.fixture(scope="module")
def declared(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    from paper_2503_10501_amd import build
    out = tmp_path_factory.mktemp("declared") / "tdeig.s"   # (the kernels that do both)
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "tdeig.hip"), "-o", str(out)], check=True,
                   capture_output=True, timeout=600)
    return {re.search(r"\.name:\s*(\S+)", part)[1]: int(part.split()[0]) for part in out.read_text().split(".group_segment_fixed_size:")[1:]}


def test_what_is_beyond_64_kb_has_been_asked_for(declared, tmp_path):
    source = STAND_IN.replace('"@launch %lx %s\\n", (long)st, name);', '"@launch %ld %s\\n", (long)s, name);')
    source = source.replace("int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }", """
int hipFuncSetAttribute(const void* f, int a, int v) {
  for (int i = 0; i < nfn; i++) if (fn[i].f == f && a == 8) fprintf(stderr, "@allow %d %s\\n", v, fn[i].name);
  return 0;
}""")
    assert source.count("@launch %ld") == 1 and source.count("@allow") == 1
    (tmp_path / "s.c").write_text(source)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-O1", str(tmp_path / "s.c"), "-o", str(tmp_path / "s.so")], check=True)
    r = subprocess.run([sys.executable, "-c", PROGRAM % ROOT, ",".join(map(str, SIZES))], env=dict(os.environ, LD_PRELOAD=str(tmp_path / "s.so")),
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    allowed, seen = {}, 0
    for what, size, name in (line[1:].split() for line in r.stderr.splitlines() if line.startswith(("@launch", "@allow"))):
        if what == "allow":
            allowed[name] = int(size)
        elif name in declared and declared[name] + int(size) > 64 * 1024:
            seen += 1
            assert allowed.get(name, 0) >= int(size), (name, declared[name], size)
    assert seen > 10
