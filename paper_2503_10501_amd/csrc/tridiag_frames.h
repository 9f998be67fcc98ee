// Frames of the register-resident reduction to tridiagonal form (tridiag.hip): geometry, exchange memory, phases, and
// which of them a device can hold.  Host code only.
#pragma once
#include <stddef.h>

namespace tc {

constexpr int TR_THREADS = 512;

// Geometry of a frame.
template <int PC>
struct TrShape {
  static constexpr int MODE = PC == 0 ? 0 : PC == 1 ? 1 : 2;
  static constexpr int PCC = PC < 2 ? 1 : PC;            // column classes of 64
  static constexpr int PR = PC == 0 ? 1 : 4 * PCC;       // row classes of 8
  static constexpr int LI = PC == 0 ? 32 : 18;           // rows and columns of a thread
  static constexpr int LK = PC == 0 ? 4 : 9;
  static constexpr int NS = 2;                           // rows are worked on in two sets of 16 or 9
  static constexpr int R = 8 * PR, C = 64 * PCC, RT = C / R;
  static constexpr int F = C * LK, P = PR * PCC;
  static constexpr int E = (F + TR_THREADS - 1) / TR_THREADS;  // vector elements of a thread
  static constexpr int OWN = 64 * LK;                    // columns of a workgroup; it has 8 LI rows
  // exchange words of one image: two slots of (partials, one set per column sum and row sum; next column; totals)
  static constexpr size_t WORDS = MODE == 0 ? 0 : MODE == 1 ? (size_t)2 * 5 * F : (size_t)2 * (5 * PCC + 2) * F;
  static constexpr size_t LDS = (size_t)(4 * (F + F / 32) + 8 * OWN + 16 * LI + 36) * 8 + (size_t)LI * 8 * 16 * 4 + 16;
  static_assert(LDS <= 160 * 1024, "LDS of a compute unit");
  static_assert(LI * R == F, "rows and columns must cover the same frame");
};

struct TrFrame { int mode, F, P; size_t words; };
constexpr int TR_SIZES = 7;  // frames: 0 the single workgroup, n: PC = n
inline const TrFrame TR_FRAMES[TR_SIZES] = {
#define TR_ENTRY(PC_) {TrShape<PC_>::MODE, TrShape<PC_>::F, TrShape<PC_>::P, TrShape<PC_>::WORDS}
    TR_ENTRY(0), TR_ENTRY(1), TR_ENTRY(2), TR_ENTRY(3), TR_ENTRY(4), TR_ENTRY(5), TR_ENTRY(6)
#undef TR_ENTRY
};

// The phases of a reduction: a frame works on the columns it is worth having, then hands the trailing matrix (through G)
// to a smaller one.  The next frame is the largest that needs fewer exchanges per column or lets more images run
// at once, so that the launch takes fewer rounds over the device's compute units.  (Hand-overs lie at multiples of 16
// columns: the blocks of sixteen reflectors.)
struct TrPhase { int size, first, last; size_t off; };  // off: where its exchange words start
inline int tr_phases(int N, int B, int cus, TrPhase* out, size_t* words) {
  auto rounds = [&](int s) { const int at_once = cus / TR_FRAMES[s].P > 1 ? cus / TR_FRAMES[s].P : 1; return (B + at_once - 1) / at_once; };
  int size = 0, n = 0, first = 0;
  while (size < TR_SIZES && TR_FRAMES[size].F < N) size++;
  *words = 0;
  if (size == TR_SIZES) return 0;
  while (true) {
    int next = size - 1;
    while (next >= 0 && TR_FRAMES[next].mode == TR_FRAMES[size].mode && rounds(next) >= rounds(size)) next--;
    const int last = next >= 0 ? (N - TR_FRAMES[next].F + 15) / 16 * 16 : N;
    out[n++] = TrPhase{size, first, last, *words};
    *words += TR_FRAMES[size].words;
    if (next < 0) return n;
    size = next;
    first = last;
  }
}

// Exchange memory of one image in words of 8 bytes: that of every frame that may take part (which do depends on the number of
// images; the size of a workspace must not fall when that or N grows), and an arrival counter per phase.
inline size_t tr_sync_words(int N) {
  size_t words = TR_SIZES;
  for (int size = 0; size < TR_SIZES; size++) {
    words += TR_FRAMES[size].words;
    if (TR_FRAMES[size].F >= N) break;
  }
  return words;
}

// Whether the reduction of N tokens runs on a device with `cus` compute units: a group must be able to be resident at once.
// Inside a captured graph (which may be replayed on several streams, where the host cannot keep launches apart) only where
// a stranded group (see tridiag.hip) holds a small part of the device: up to a seventh.
inline bool tr_runs(int N, int cus, bool captured) {
  int size = 0;
  while (size < TR_SIZES && TR_FRAMES[size].F < N) size++;
  return size < TR_SIZES && (captured ? 7 : 1) * TR_FRAMES[size].P <= (TR_FRAMES[size].P > 1 ? cus : 256);
}

// Launches that the host keeps apart: groups of a frame that spans several XCDs.
inline bool tr_apart(int P) { return P > 4; }

}  // namespace tc
