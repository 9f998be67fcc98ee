"""Host test (no GPU): the frames of the register-resident reduction, their phases and which of them a device can hold, for whole
and partitioned devices.  csrc/tridiag_frames.h is host code; it is compiled here into a program that answers questions."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2503_10501_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "tridiag_frames.h"
using namespace tc;
int main() {
  int N, B, cus;
  while (std::scanf("%d %d %d", &N, &B, &cus) == 3) {
    TrPhase ph[TR_SIZES];
    size_t words;
    const int n = tr_phases(N, B, cus, ph, &words);
    std::printf("%d %d %zu %zu %d", tr_runs(N, cus, false), tr_runs(N, cus, true), words, tr_sync_words(N), n);
    for (int i = 0; i < n; i++)
      std::printf(" %d %d %d %d %d", TR_FRAMES[ph[i].size].F, TR_FRAMES[ph[i].size].P, ph[i].first, ph[i].last, tr_apart(TR_FRAMES[ph[i].size].P));
    std::printf("\n");
  }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("frames")
    src, exe = d / "frames.cpp", d / "frames"
    src.write_text(PROGRAM)
    subprocess.run([gxx, "-std=c++20", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def run(questions):
        out = subprocess.run([str(exe)], input="\n".join("%d %d %d" % q for q in questions), capture_output=True, text=True, check=True)
        rows = [[int(x) for x in line.split()] for line in out.stdout.splitlines()]
        assert len(rows) == len(questions)
        return [(r[0], r[1], r[2], r[3], [tuple(r[5 + 5 * i:10 + 5 * i]) for i in range(r[4])]) for r in rows]
    return run


SIZES = [1, 2, 255, 256, 257, 575, 576, 577, 701, 1024, 1152, 1153, 1728, 1729, 2304, 2305, 2880, 2881, 3456]


@pytest.mark.parametrize("cus", [256, 128, 64, 32, 8])
def test_phases_cover_every_column_once(ask, cus):
    questions = [(n, b, cus) for n in SIZES for b in (1, 2, 3, 7, 17, 64, 300)]
    for (n, b, _), (_, _, words, room, phases) in zip(questions, ask(questions)):
        assert phases[0][2] == 0 and phases[-1][3] == n
        for (F, P, first, last, _), nxt in zip(phases, phases[1:]):
            assert last == nxt[2] and last % 16 == 0   # blocks of sixteen reflectors
        for F, P, first, last, _ in phases:
            assert n - first <= F and first <= last
        assert words + len(phases) <= room


@pytest.mark.parametrize("cus,most,captured", [(256, 3456, 1728), (128, 2880, 1152), (64, 2304, 576), (32, 1152, 576), (8, 576, 256)])
def test_a_group_fits_the_device(ask, cus, most, captured):
    questions = [(n, 1, cus) for n in SIZES + [3457, 4096]]
    for (n, _, _), (runs, in_graph, _, _, phases) in zip(questions, ask(questions)):
        assert runs == (n <= most) and in_graph == (n <= captured), n
        if runs:
            assert all(P <= cus for _, P, _, _, _ in phases)
        # groups on one XCD leave at most three workgroups waiting there, with the four hardware queues of a process twelve of 32:
        # all others are kept apart
        assert all(apart == (P > 4) for _, P, _, _, apart in phases)


def test_the_end_of_the_frames(ask):
    assert [bool(r[4]) for r in ask([(3456, 1, 256), (3457, 1, 256)])] == [True, False]


# The same for captured streams too, with the rows that a frame has to leave to the next one.
CAPTURED = PROGRAM.replace("int N, B, cus;", "int N, B, cus, captured;").replace('"%d %d %d", &N, &B, &cus) == 3', '"%d %d %d %d", &N, &B, &cus, &captured) == 4')
CAPTURED = CAPTURED.replace("&words);", "&words, captured != 0);").replace("tr_apart(TR_FRAMES[ph[i].size].P)", "TR_FRAMES[ph[i].size].least")


@pytest.fixture(scope="module")
def ask_captured(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("captured")
    (d / "frames.cpp").write_text(CAPTURED)
    subprocess.run([gxx, "-std=c++20", "-O1", "-I", CSRC, str(d / "frames.cpp"), "-o", str(d / "frames")], check=True)

    def run(questions):
        out = subprocess.run([str(d / "frames")], input="\n".join("%d %d %d %d" % q for q in questions), capture_output=True, text=True, check=True)
        rows = [[int(x) for x in line.split()] for line in out.stdout.splitlines()]
        assert len(rows) == len(questions)
        return [(r[0], r[1], r[2], r[3], [tuple(r[5 + 5 * i:10 + 5 * i]) for i in range(r[4])]) for r in rows]
    return run


def test_the_room_for_exchanges_never_falls_and_is_small_where_there_are_none(ask_captured):
    rooms = [r[3] for r in ask_captured([(n, 1, 256, 0) for n in range(1, 3457)])]
    assert rooms == sorted(rooms)
    assert rooms[127] * 8 <= 256   # up to 128 tokens: one workgroup


# first and last size of every frame, and where that of the last 128 rows ends
EDGES = sorted({n + d for n in (128, 256, 320, 384, 448, 576, 768, 1152, 1536, 1728, 1920, 2112, 2304, 2880, 3456) for d in (-1, 0, 1, 2)} - {3457, 3458})


@pytest.mark.parametrize("captured", [0, 1])
@pytest.mark.parametrize("cus", [256, 128, 64, 32])
def test_phases_at_the_edges_of_the_frames(ask_captured, cus, captured):
    questions = [(n, b, cus, captured) for n in EDGES for b in (1, 2, 8, 16, 33, 64, 97, 300)]
    for (n, b, _, _), (runs, in_graph, words, room, phases) in zip(questions, ask_captured(questions)):
        if not (in_graph if captured else runs):
            continue
        assert phases[0][2] == 0 and phases[-1][3] == n and words + len(phases) <= room
        for (F, P, first, last, least), nxt in zip(phases, phases[1:]):
            assert last == nxt[2] and last % 16 == 0 and first < last and n - first <= F
            assert n - last >= least, (n, b)   # whole columns: every workgroup has one to publish up to the last
        assert n - phases[-1][2] <= phases[-1][0]
        assert all((7 if captured else 1) * P <= cus or P == 1 for _, P, _, _, _ in phases), (n, b)


def test_captured_phases_are_the_same_as_far_as_the_header_says(ask_captured):
    for cus, same in ((256, 768), (128, 576), (64, 448), (32, 128)):
        sizes = [n for n in range(1, 3457) if n <= same + 1]
        one, other = (ask_captured([(n, b, cus, c) for n in sizes for b in (1, 3, 16, 64, 300)]) for c in (0, 1))
        differ = [n for (n, _), x, y in zip(((n, b) for n in sizes for b in (1, 3, 16, 64, 300)), one, other) if x[4] != y[4]]
        assert differ and min(differ) == same + 1, cus
