"""Host test (no GPU): the order that events impose on the launches of a call with stream groups, and what becomes of a call whose
events fail.  The library runs against a stand-in for the HIP runtime that launches nothing and writes down what it is asked for."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2503_10501_amd", "libtokencarve.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB) or not shutil.which("gcc"), reason="needs libtokencarve.so and gcc")

STAND_IN = r"""
#include <stdio.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static struct { const void* f; char name[200]; } fn[512];
static int nfn, calls[3], fail_at[3], last;   // 0 nothing, 1 record, 2 wait: the call with this number fails
static uintptr_t handles = 0x1000;
static dim3 cg, cb; static size_t cs; static void* cst;
int fake_arm(int kind, int at) { calls[1] = calls[2] = 0; fail_at[1] = fail_at[2] = 0; fail_at[kind] = at; return 0; }
static int outcome(int kind) { calls[kind]++; if (fail_at[kind] != calls[kind]) return 0; last = 1; return 1; }
static void say(const char* what, uintptr_t a, uintptr_t b, int bad) { fprintf(stderr, "@%s %lx %lx %d\n", what, (long)a, (long)b, bad); }
void** __hipRegisterFatBinary(const void* d) { static void* h; return &h; }
void __hipUnregisterFatBinary(void** m) {}
void __hipRegisterVar(void** m, void* v, char* h, const char* n, int e, size_t s, int c, int g) {}
void __hipRegisterFunction(void** m, const void* f, char* d, const char* name, unsigned t, void* a, void* b, void* c, void* e, int* w) {
  if (nfn < 512 && !strncmp(name, "_ZN2tc", 6)) {  /* (torch registers thousands of its own) */ fn[nfn].f = f; strncpy(fn[nfn++].name, name, 199); }
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void* st) { cg = g; cb = b; cs = s; cst = st; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** st) { *g = cg; *b = cb; *s = cs; *st = cst; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t s, void* st) {
  const char* name = "?";
  for (int i = 0; i < nfn; i++) if (fn[i].f == f) name = fn[i].name;
  fprintf(stderr, "@launch %lx %s\n", (long)st, name);
  return 0;
}
int hipGetLastError(void) { int e = last; last = 0; return e; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
int hipStreamIsCapturing(void* st, int* c) { *c = 0; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = (void*)(handles += 16); return 0; }
int hipEventDestroy(void* e) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { *s = (void*)(handles += 16); return 0; }
int hipStreamDestroy(void* s) { return 0; }
int hipStreamSynchronize(void* s) { say("sync", (uintptr_t)s, 0, 0); return 0; }
int hipEventRecord(void* e, void* st) { int bad = outcome(1); say("record", (uintptr_t)st, (uintptr_t)e, bad); return bad; }
int hipStreamWaitEvent(void* st, void* e, unsigned f) { int bad = outcome(2); say("wait", (uintptr_t)st, (uintptr_t)e, bad); return bad; }
"""

PROGRAM = r"""
import ctypes, json, sys
sys.path.insert(0, %r)
from paper_2503_10501_amd import binding as tc
lib, fake, ptr = tc.load_library(), ctypes.CDLL(None), 1 << 20
for kw, kind, at in json.loads(sys.stdin.read()):
    p = tc.make_params(seq_len=576, vis_start=0, n_vis=576, n_heads=32, head_dim=128, hidden_dim=4096, dtype=tc.TC_BF16, k_prune=2, k_final=2, **kw)
    need = tc.tc_workspace_bytes(p)
    fake.fake_arm(kind, at)
    sys.stderr.write("@call\n"); sys.stderr.flush()
    rc = lib.tc_ipgs_score(ctypes.byref(p), ptr, ptr, ptr, None, None, None, ptr, need, None)
    sys.stderr.write("@returns %%d\n" %% rc); sys.stderr.flush()
"""
RECORD, WAIT = 1, 2
CASES = [dict(batch=b, stream_groups=g, **kw) for b, g in ((130, 0), (64, 2), (64, 3), (64, 4)) for kw in ({}, {"eig_method": 1})]


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    """A process that makes some calls, [(parameters, RECORD or WAIT, which of these fails)]: [(what the call returned, its log)]."""
    d = tmp_path_factory.mktemp("standin")
    (d / "s.c").write_text(STAND_IN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-O1", str(d / "s.c"), "-o", str(d / "s.so")], check=True)

    def run(todo):
        r = subprocess.run([sys.executable, "-c", PROGRAM % ROOT], env=dict(os.environ, LD_PRELOAD=str(d / "s.so")),
                           input=json.dumps(todo), capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        out = []
        for w in (line.split() for line in r.stderr.splitlines() if line.startswith("@")):
            if w[0] == "@call":
                out.append([None, []])
            elif w[0] == "@returns":
                out[-1][0] = int(w[1])
            elif out:
                out[-1][1].append((w[0][1:], *w[1:]))
        assert len(out) == len(todo)
        return out
    return run


@pytest.fixture(scope="module")
def good(calls):
    return calls([(kw, 0, 0) for kw in CASES])


def _check(log, met):
    """Launches of the Gram step, which share the room for the digits, come one after the other on whatever stream; with `met` the
    caller's stream (0) waits for all launches, otherwise it does or the host has."""
    now, event, count, synced, gram = {}, {}, {}, {}, []
    for what, stream, *rest in log:
        clock = now.setdefault(stream, {})   # what is done before the stream's next launch: stream -> launches
        if what == "launch":
            if "gram" in rest[0]:
                assert all(clock.get(s, 0) >= n for s, n in gram)
            clock[stream] = count[stream] = count.get(stream, 0) + 1
            if "gram" in rest[0]:
                gram.append((stream, count[stream]))
        elif what == "record" and rest[1] == "0":
            event[rest[0]] = dict(clock)
        elif what == "wait" and rest[1] == "0":
            for s, n in event.get(rest[0], {}).items():
                clock[s] = max(clock.get(s, 0), n)
        elif what == "sync":
            synced[stream] = count.get(stream, 0)
    for s, n in count.items():
        assert s == "0" or now["0"].get(s, 0) >= n or (not met and synced.get(s, 0) >= n), s
    return count


@pytest.mark.parametrize("i", range(len(CASES)), ids=str)
def test_groups_share_the_digits_in_turn_and_meet_again(good, i):
    rc, log = good[i]
    assert rc == 0 and any(x[0] == "launch" and "gram_slice_kernel" in x[2] for x in log)
    assert len(_check(log, True)) > 1   # streams


@pytest.mark.parametrize("i", [4, 5])   # three groups
def test_a_call_whose_events_fail_says_so_and_leaves_nothing_running(calls, good, i):
    kinds = ((RECORD, "record"), (WAIT, "wait"))
    fail = [(k, n + 1) for k, name in kinds for n in range(sum(x[0] == name for x in good[i][1]))]
    assert len(fail) >= 7
    answers = calls([(CASES[i], *f) for at in fail for f in (at, (0, 0))])
    for at, (rc, log), (rc2, log2) in zip(fail, answers[::2], answers[1::2]):
        assert rc == -7, at
        _check(log, False)
        assert rc2 == 0 and [x[::2] for x in log2] == [x[::2] for x in good[i][1]], at   # the next call is as it should be
