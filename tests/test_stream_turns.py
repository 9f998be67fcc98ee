"""Host test (no GPU): which launches of the reduction may run side by side when calls are enqueued on several streams.  The library runs
against the stand-in for the HIP runtime of test_stream_order.py; from what it asks for follows which launches are ordered."""
import itertools
import json
import os
import random
import re
import subprocess
import sys

import pytest

from tests.test_stream_order import LIB, ROOT, STAND_IN, pytestmark  # noqa: F401

PROGRAM = r"""
import ctypes, json, sys
sys.path.insert(0, %r)
from paper_2503_10501_amd import binding as tc
lib, ptr = tc.load_library(), 1 << 20
for n, batch, stream in json.loads(sys.stdin.read()):
    p = tc.make_params(seq_len=n, vis_start=0, n_vis=n, n_heads=4, head_dim=128, hidden_dim=512, dtype=tc.TC_BF16, k_prune=2, k_final=2, batch=batch, stream_groups=1)
    sys.stderr.write("@call %%d\n" %% batch); sys.stderr.flush()
    assert lib.tc_ipgs_score(ctypes.byref(p), ptr, ptr, ptr, None, None, None, ptr, tc.tc_workspace_bytes(p), ctypes.c_void_p(stream)) == 0
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """Calls [(tokens, images, stream)] -> their reductions' launches of groups [(P, most that may wait on an XCD, XCDs, stream, number in
    it, clock)], where clock says how many launches of every stream are over before it."""
    d = tmp_path_factory.mktemp("turns")
    say = 'fprintf(stderr, "@launch %lx %s\\n", (long)st, name);'   # and the number of the first XCD (groups of whole columns)
    assert STAND_IN.count(say) == 1
    (d / "s.c").write_text(STAND_IN.replace(say, say.replace("%s", "%s %d").replace("name)", 'name, strstr(name, "columns") ? *(int*)args[15] : 0)')))
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-O1", str(d / "s.c"), "-o", str(d / "s.so")], check=True)

    def run(todo):
        r = subprocess.run([sys.executable, "-c", PROGRAM % ROOT], env=dict(os.environ, LD_PRELOAD=str(d / "s.so")),
                           input=json.dumps(todo), capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        now, event, count, out, batch = {}, {}, {}, [], 0
        for w in (line.split() for line in r.stderr.splitlines() if line.startswith("@")):
            if w[0] == "@call":
                batch = int(w[1])
                continue
            clock = now.setdefault(w[1], {})
            if w[0] == "@launch":
                clock[w[1]] = count[w[1]] = count.get(w[1], 0) + 1
                columns = re.search(r"tridiag_columns_kernel.*TcShapeILi\d+ELi\d+ELi(\d+)E", w[2])
                triangle = re.search(r"14tridiag_kernelILi(\d+)E", w[2])
                P = int(columns[1]) if columns else 4 * int(triangle[1]) ** 2 if triangle else 1
                local = bool(columns) and P <= 16
                xcds = {(int(w[3]) + i) % 8 for i in range(min(batch, 8) if local else 8)}
                if P > 1:
                    out.append((P, P - 1 if local else -(-P * batch // 8), xcds, w[1], count[w[1]], dict(clock)))
            elif w[0] == "@record":
                event[w[2]] = dict(clock)
            elif w[0] == "@wait":
                for s, n in event.get(w[2], {}).items():
                    clock[s] = max(clock.get(s, 0), n)
        return out
    return run


def _side_by_side(a, b):
    return a[3] != b[3] and a[5].get(b[3], 0) < b[4] and b[5].get(a[3], 0) < a[4]


SHAPES = [(200, 8), (300, 8), (450, 40), (576, 8), (576, 16), (576, 64), (600, 1), (701, 1), (701, 2), (701, 4), (701, 9), (1152, 1), (1152, 2),
          (1499, 1), (1600, 1), (2000, 1), (2880, 8)]


@pytest.mark.parametrize("seed", range(4))
def test_what_may_wait_at_once_leaves_a_compute_unit(launches, seed):
    # an XCD has 32 compute units, a process four hardware queues; groups of four are not ordered, and three of their workgroups wait
    # at most in each queue
    rng = random.Random(seed)
    done = launches([(*rng.choice(SHAPES), 1 + rng.randrange(4)) for _ in range(60)])
    ordered = [x for x in done if x[0] > 4]
    assert len(ordered) > 100
    beside = [[_side_by_side(a, b) for b in ordered] for a in ordered]
    met = 0
    for x in range(8):
        here = [i for i, a in enumerate(ordered) if x in a[2]]
        for i in here:
            near = [j for j in here if j < i and beside[i][j]]
            for k in (1, 2, 3):
                for js in itertools.combinations(near, k):
                    if all(beside[a][b] for a, b in itertools.combinations(js, 2)):
                        met += 1
                        assert sum(ordered[j][1] for j in (i, *js)) + 3 * (3 - k) <= 31, [ordered[j][:4] for j in (i, *js)]
    assert met > 100


# Groups of eight have four of the nineteen places, or the last four in calls that have groups of sixteen, which have the first twelve.
# What fills the device takes all (32 images by eight, eight of 701 or 2880 tokens), and groups of four take none.
@pytest.mark.parametrize("n,batch,least", [(200, 8, 4), (300, 31, 4), (300, 32, 1), (576, 2, 4), (576, 4, 2), (701, 1, 4), (701, 8, 1),
                                           (2880, 8, 1), (576, 64, 4)])
def test_calls_that_leave_room_run_side_by_side(launches, n, batch, least):
    # so many of the first launches of four calls on four streams
    done = launches([(n, batch, s) for s in (1, 2, 3, 4)])
    first = [next(x for x in done if x[3] == "%d" % s) for s in (1, 2, 3, 4)]
    most = max(k for k in (1, 2, 3, 4) for some in itertools.combinations(first, k)
               if all(_side_by_side(a, b) for a, b in itertools.combinations(some, 2)))
    assert most >= least


@pytest.mark.parametrize("n,batch", [(576, 2), (576, 8), (576, 15)])
def test_small_groups_of_one_call_run_beside_large_groups_of_the_next(launches, n, batch):
    done = launches([(n, batch, s) for s in (1, 2, 3, 4)])
    calls = [[x for x in done if x[3] == "%d" % s] for s in (1, 2, 3, 4)]
    assert all(x[0] == 8 for x in (c[-1] for c in calls))
    assert all(_side_by_side(a[-1], next(x for x in b if x[0] == 16)) for a, b in zip(calls, calls[1:]))
