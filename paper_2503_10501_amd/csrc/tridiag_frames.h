// Frames of the register-resident reduction to tridiagonal form (tridiag.hip, tridiag_columns.hip): geometry, exchange memory,
// phases, and which of them a device can hold.  Host code only.
#pragma once
#include <stddef.h>

namespace tc {

constexpr int TR_THREADS = 512;

// Geometry of a frame that holds the lower triangle (tridiag.hip).
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

// Geometry of a frame that holds whole columns (tridiag_columns.hip): P workgroups of eight wavefronts, of which four hold the
// matrix, LK columns each with LI rows in a lane; the other four work on the vectors.
template <int LI_, int LK_, int P_>
struct TcShape {
  static constexpr int LI = LI_, LK = LK_, P = P_;
  static constexpr bool LOCAL = P <= 16;    // a group lies on one XCD
  static constexpr int F = 64 * LI;         // rows
  static constexpr int CW = 4 * P;          // columns of a class: one for every wavefront of the group that holds the matrix
  static constexpr int E = (F + 255) / 256, FP = 256 * E;  // vector elements of a thread; room of a vector
  static constexpr int RO = (F + P - 1) / P;    // rows of the reflectors that a workgroup writes
  static constexpr size_t WORDS = (size_t)6 * F;  // exchange: two slots of products, four of next columns
  static constexpr size_t LDS = (size_t)(5 * FP + 52) * 8 + (size_t)(RO * 16 + 16) * 4 + 16;
  static_assert(LK <= 32, "sums and columns of one wavefront");
  static_assert(LK * CW == F, "the classes must cover the frame");
  static_assert(LDS <= 160 * 1024, "LDS of a compute unit");
};

constexpr int TR_LAST = 128;  // rows that one workgroup of four wavefronts reduces (tridiag_last_kernel)

// mode: TrShape::MODE of a triangle, 3 the last columns, 4 whole columns;
// least: rows a frame leaves at least (all of its workgroups must have a column to publish); us: time of a column in microseconds,
// from which the phases are chosen.
struct TrFrame { int mode, F, P; size_t words; int least; double us; };
constexpr int TR_TRIANGLES = 7;  // frames: 0 the single workgroup, n: PC = n,
constexpr int TR_LAST_SIZE = TR_TRIANGLES;  // the last columns, and whole columns from here on: (number, LI, LK, P, us)
#define TC_FRAMES(X) \
  X(8, 6, 12, 8, 1.35) X(9, 9, 9, 16, 1.75) X(10, 12, 6, 32, 2.1) X(11, 18, 4, 72, 2.5) X(12, 24, 3, 128, 2.95) X(13, 30, 3, 160, 3.3) \
  X(14, 33, 3, 176, 3.5) X(15, 5, 20, 4, 1.45) X(16, 7, 14, 8, 1.65)
constexpr int TR_SIZES = 17;
inline const TrFrame TR_FRAMES[TR_SIZES] = {
#define TR_ENTRY(PC_, US_) {TrShape<PC_>::MODE, TrShape<PC_>::F, TrShape<PC_>::P, TrShape<PC_>::WORDS, 0, US_}
    TR_ENTRY(0, 3.05), TR_ENTRY(1, 5.5), TR_ENTRY(2, 6.4), TR_ENTRY(3, 7.35), TR_ENTRY(4, 7.4), TR_ENTRY(5, 8.3), TR_ENTRY(6, 9.0),
#undef TR_ENTRY
    {3, TR_LAST, 1, 0, 0, 0.93},
#define TR_ENTRY(N_, LI_, LK_, P_, US_) {4, TcShape<LI_, LK_, P_>::F, P_, TcShape<LI_, LK_, P_>::WORDS, TcShape<LI_, LK_, P_>::CW, US_},
    TC_FRAMES(TR_ENTRY)
#undef TR_ENTRY
};

// The smallest of the triangular frames that holds N rows (TR_TRIANGLES: none).
inline int tr_triangle(int N) {
  int size = 0;
  while (size < TR_TRIANGLES && TR_FRAMES[size].F < N) size++;
  return size;
}

// Inside a captured graph (which may be replayed on several streams, where the host cannot keep launches apart) a group that is
// stranded (see tridiag.hip) must hold a small part of the device: up to a seventh.
inline bool tr_holds(int P, int cus, bool captured) { return (captured ? 7 : 1) * P <= (P > 1 ? cus : 256); }

// The phases of a reduction: a frame works on the columns it is worth having, then hands the trailing matrix (through G) to a
// smaller one; the last TR_LAST rows are one workgroup's.  Chosen so that the sum over the phases is least: columns, times the
// rounds that the call's images make over the device, times the time of a column, and TR_HAND a round for handing over.
// (Hand-overs lie at multiples of 16 columns: the blocks of sixteen reflectors.)
struct TrPhase { int size, first, last; size_t off; };  // off: where its exchange words start
constexpr double TR_HAND = 12.0;
inline int tr_phases(int N, int B, int cus, TrPhase* out, size_t* words, bool captured = false) {
  const int top = tr_triangle(N);
  *words = 0;
  if (top == TR_TRIANGLES) return 0;
  const int most = TR_FRAMES[top].F > TR_FRAMES[1].F ? TR_FRAMES[top].F : TR_FRAMES[1].F;  // (what tr_sync_words counts)
  auto from = [&](int s) { return TR_FRAMES[s].F >= N ? 0 : (N - TR_FRAMES[s].F + 15) / 16 * 16; };  // first column of a frame
  auto rounds = [&](int P) { const int at_once = cus / P > 1 ? cus / P : 1; return (B + at_once - 1) / at_once; };
  double best[TR_SIZES];
  int next[TR_SIZES], start = -1;
  for (int s = 0; s < TR_SIZES; s++) best[s] = -1;
  best[TR_LAST_SIZE] = rounds(1) * TR_FRAMES[TR_LAST_SIZE].us * (N - from(TR_LAST_SIZE));
  next[TR_LAST_SIZE] = -1;
  for (int F = TR_LAST; F <= most; F += 64)  // by size
    for (int s = 0; s < TR_SIZES; s++) {
      const TrFrame& f = TR_FRAMES[s];
      if (f.F != F) continue;
      // (whether the device holds the smallest triangular frame for N is asked elsewhere: tr_runs)
      if (s != TR_LAST_SIZE && (s == top || tr_holds(f.P, cus, captured)))
        for (int t = 0; t < TR_SIZES; t++) {
          if (best[t] < 0 || TR_FRAMES[t].F >= F || from(t) <= from(s) || N - from(t) < f.least) continue;
          const double c = (from(t) - from(s)) * rounds(f.P) * f.us + TR_HAND * rounds(f.P) + best[t];
          if (best[s] < 0 || c < best[s]) { best[s] = c; next[s] = t; }
        }
      if (F >= N && best[s] >= 0 && (start < 0 || best[s] < best[start])) start = s;
    }
  if (start < 0) return 0;
  int n = 0;
  for (int s = start; s >= 0; s = next[s]) {
    out[n++] = TrPhase{s, from(s), next[s] >= 0 ? from(next[s]) : N, *words};
    *words += TR_FRAMES[s].words;
  }
  return n;
}

// Exchange memory of one image in words of 8 bytes: that of every frame that may take part (which do depends on the number of
// images; the size of a workspace must not fall when that or N grows), and an arrival counter per phase.  (Up to TR_LAST tokens one
// workgroup does all columns.)
inline size_t tr_sync_words(int N) {
  size_t words = TR_SIZES;
  if (N <= TR_LAST) return words;
  const int top = tr_triangle(N), F = top < 2 ? TR_FRAMES[1].F : TR_FRAMES[top < TR_TRIANGLES ? top : TR_TRIANGLES - 1].F;
  for (const TrFrame& f : TR_FRAMES)
    if (f.F <= F) words += f.words;
  return words;
}

// Whether the reduction of N tokens runs on a device with `cus` compute units: a group must be able to be resident at once.
inline bool tr_runs(int N, int cus, bool captured) {
  const int size = tr_triangle(N);
  return size < TR_TRIANGLES && tr_holds(TR_FRAMES[size].P, cus, captured);
}

// Launches that the host keeps apart (see TrTurn): most workgroups of one that may wait on an XCD at once, and how many of its
// places the launch takes there; all, too, where its workgroups would fill the XCD anyway.
constexpr int TR_PLACES = 19;
inline bool tr_apart(int P) { return P > 4; }
inline bool tr_local(int size) { return TR_FRAMES[size].mode == 4 && TR_FRAMES[size].P <= 16; }
inline int tr_places(int P, bool local, int images, int xcds) {
  const long long all = ((long long)P * images + xcds - 1) / xcds, waiting = local ? P - 1 : all;
  return all >= 32 || waiting - 3 > TR_PLACES ? TR_PLACES : waiting > 4 ? (int)waiting - 3 : 1;
}
// The first of these places.  Groups of sixteen take TR_SIXTEEN from 0 on; launches of their calls (sixteen) with groups that are spread make
// do with the rest, and so do groups of eight behind them on all XCDs.
constexpr int TR_SIXTEEN = 12;
inline int tr_first_place(int places, bool local, bool all, bool sixteen, unsigned slot) {
  constexpr int rest = TR_PLACES - TR_SIXTEEN;
  if (places > rest) return sixteen || 2 * places > TR_PLACES ? 0 : places * (int)(slot % 2);
  if (sixteen) return !local ? TR_SIXTEEN + places * (int)(slot % (rest / places)) : all ? TR_PLACES - places : 0;
  return TR_PLACES - places * (1 + (int)(slot % (TR_PLACES / places)));
}

}  // namespace tc
