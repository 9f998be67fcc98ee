// Direct symmetric eigensolver, stages 2 and 3 (stage 1, the reduction G = Q T Q^T, is tridiag.hip):
//   2a  eigenvalues of the tridiagonal T by bisection on Sturm counts, one lane per eigenvalue;
//   2b  eigenvector of every eigenvalue from the twisted factorisation of T - lambda I
//       (forward L D+ L^T, backward U D- U^T, joined at the index r that minimises |gamma_r|;
//       the vector solves (T - lambda I) z = gamma_r e_r), one lane per eigenvector;
//   3   back-transformation U = Q W = H_0 ... H_{N-2} W in float32 on the matrix cores, the reflectors sixteen
//       at a time in compact WY form, a strip of 16 eigenvectors held in accumulator registers; since U is
//       only needed for it, the information contribution score of Eq. 3-6, C(x) = sum_i |U[x][i]| sigma_i,
//       is accumulated right there: U is never written.
// T is first split where an off-diagonal element is negligible (|e_k| <= eps ||T||); each eigenpair then
// belongs to one unreduced block and its vector is zero outside that block, so equal eigenvalues of
// decoupled blocks (block-diagonal Gram matrices, null spaces) get orthogonal vectors for free.
// Eigenvectors of one block are computed independently of each other; a close pair that did not come out orthogonal is
// orthogonalised explicitly afterwards (td_pairs_kernel, td_orthogonalise_kernel).
#include <cfloat>
#include <utility>

#include "tc_internal.h"

namespace tc {

typedef unsigned long long u64;

constexpr double TD_EPS = 2.220446049250313e-16;

// ---- 2a -----------------------------------------------------------------------------------------------
// dvec, evec [B][Np] from the reduction.  Writes lam [B][Np] (eigenvalue of slot k: the (k - s)-th smallest
// of the block [s, t) that row k lies in), blk [B][Np] = (s, t), and tnorm [B] = ||T||_inf.
//
// The number of eigenvalues below x is the number of sign changes in the sequence of leading principal
// minors p_0 = 1, p_1 = d_s - x, p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}.  In this form the step from one row to the
// next is multiply-adds only; the quotient form q_i = d_i - x - e^2 / q_{i-1} puts a float64 division (thirty
// dependent instructions) on it, and with one eigenvalue per lane there is nothing to hide that latency behind.
// T is scaled by a power of two to ||T|| <= 1 so that the minors change by at most a
// factor 3 per step, and they are brought back into range every eight steps.
typedef double tb_pair __attribute__((ext_vector_type(2)));

// Scaled copy of T for the bisection, one workgroup per image: prep [B][prep_stride] doubles holds
// (d_i, -e_i^2) pairs for rows 0 .. N-1 (e_i = |coupling of rows i-1 and i|, e_0 = 0; the square is 0 where T
// is split), 32 zero pairs behind them, then the Gershgorin interval of T (scaled).  Also the block (s, t) of every row,
// tnorm [B] = ||T||_inf; bad[b] starts from the failure flag of the reduction, mark [B][Np] from N, any[b] and need[b] from 0.
__global__ __launch_bounds__(256) void td_prepare_kernel(const double* __restrict__ dvec, const double* __restrict__ evec,
                                                         double* __restrict__ prep, size_t prep_stride,
                                                         double* __restrict__ tnorm, int2* __restrict__ blk,
                                                         int32_t* __restrict__ bad, int32_t* __restrict__ mark,
                                                         int32_t* __restrict__ any, int32_t* __restrict__ need,
                                                         const int32_t* __restrict__ fail, int N, int Np) {
  __shared__ double wred[3][4];
  __shared__ u64 cut[MAX_NVIS / 64 + 1];  // bit i: a block starts at row i
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* db = dvec + (size_t)b * Np;
  const double* eb = evec + (size_t)b * Np;
  double rowmax = 0.0, lo = DBL_MAX, hi = -DBL_MAX;
  for (int i = tid; i < N; i += 256) {
    const double r = (i > 0 ? fabs(eb[i - 1]) : 0.0) + (i + 1 < N ? fabs(eb[i]) : 0.0), d = db[i];
    rowmax = fmax(rowmax, fabs(d) + r);
    lo = fmin(lo, d - r);
    hi = fmax(hi, d + r);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    rowmax = fmax(rowmax, __shfl_xor(rowmax, o, 64));
    lo = fmin(lo, __shfl_xor(lo, o, 64));
    hi = fmax(hi, __shfl_xor(hi, o, 64));
  }
  if (lane == 0) { wred[0][wave] = rowmax; wred[1][wave] = lo; wred[2][wave] = hi; }
  __syncthreads();
  const double tn = fmax(fmax(wred[0][0], wred[0][1]), fmax(wred[0][2], wred[0][3]));
  const double split = TD_EPS * tn;
  // power of two that brings ||T|| into (1/2, 1] (exact); a zero or non-finite norm leaves T as it is
  int ex = 0;
  if (tn > 0.0 && tn < DBL_MAX) (void)frexp(tn, &ex);
  const double down = ldexp(1.0, -ex);
  tb_pair* pr = reinterpret_cast<tb_pair*>(prep + (size_t)b * prep_stride);
  const int rows = round_up(N, 256);
  for (int i = tid; i < rows + 256; i += 256) {
    const double e = i > 0 && i < N ? fabs(eb[i - 1]) : 0.0;
    const bool start = i >= N || !(e > split);
    if (i < N + 32) pr[i] = i < N ? tb_pair{db[i] * down, start ? 0.0 : -(e * down) * (e * down)} : tb_pair{0.0, 0.0};
    const u64 m = __ballot(start);
    if (lane == 0 && (i >> 6) <= MAX_NVIS / 64) cut[i >> 6] = m;  // (rows past N count as starts: a block ends at N at the latest)
  }
  __syncthreads();
  for (int i = tid; i < N; i += 256) {
    int w = i >> 6;
    u64 m = cut[w] & (~0ull >> (63 - (i & 63)));  // starts at or before row i (row 0 is one)
    while (m == 0) m = cut[--w];
    const int s = 64 * w + 63 - __builtin_clzll(m);
    w = i >> 6;
    m = (i & 63) == 63 ? 0 : cut[w] & (~0ull << ((i & 63) + 1));
    while (m == 0) m = cut[++w];
    blk[(size_t)b * Np + i] = int2{s, min(64 * w + __builtin_ctzll(m), N)};
    mark[(size_t)b * Np + i] = N;
  }
  if (tid == 0) {
    tnorm[b] = tn;
    bad[b] = fail[b] ? 4 : 0;
    any[b] = 0;
    need[b] = 0;
    pr[N + 32] = tb_pair{fmin(fmin(wred[1][0], wred[1][1]), fmin(wred[1][2], wred[1][3])) * down,
                         fmax(fmax(wred[2][0], wred[2][1]), fmax(wred[2][2], wred[2][3])) * down};
  }
}

// d += (lane n of each row of 16 lanes of `row`) * c
template <int n>
__device__ __forceinline__ void td_fmac_bcast(double& d, double row, double c) {
  asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(row), "v"(c), "n"(n));
}

// One row of the recurrence: (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2} as -x p + (-e^2) pp + d p, the coefficients by broadcast:
// four instructions (46 cycles per row for a wavefront alone on its SIMD; with d - x formed first, one operation fewer
// on the chain but one instruction more, 50).  The rounding is that of a d_i off by eps |x| <= eps ||T||, what the
// entries of T carry anyway.
template <int n>
__device__ __forceinline__ void tb_row(double dr, double er, double x, double& p, double& pp, unsigned& signs) {
  double pn = -x * p;
  td_fmac_bcast<n>(pn, er, pp);
  td_fmac_bcast<n>(pn, dr, p);
  signs = __builtin_amdgcn_alignbit(signs, (unsigned)__double2hiint(pn), 31);
  pp = p;
  p = pn;
}

// The number of sign changes of the minors at x for rows s0 .. t0-1 (uniform over the wavefront), and the last minor as
// p 2^ex.  Sixteen rows' coefficients sit in the lanes of a row of 16, the next sixteen are in flight.  (Through the
// scalar unit, whose loads can only be waited for all together, a row cost 73 cycles.)
// Sign changes are counted on the sign bits.  The signs of the minors are shifted into one register, a bit
// per row (bit 0 = the newest); after eight rows the changes among them and against the minor before them
// are the set bits of (signs xor signs >> 1) in its low byte.  An exact zero needs no special case: its
// successor is -e^2 times its predecessor, so the three minors around it contain one sign change whichever
// sign the zero is given.  Every eight rows the minors are brought back into range by a power of two (which changes no
// sign) taken from the minors three rows before, off the chain.
__device__ __forceinline__ int tb_walk(const tb_pair* __restrict__ pr, int s0, int t0, int N, int lane, double x, double& p, int& ex) {
  double pp = 1.0;
  p = pr[s0].x - x;
  ex = 0;
  unsigned signs = (unsigned)__double2hiint(p) >> 31;  // p_0 = 1 is positive: bit 1 = 0
  int cnt = (int)signs;
  const tb_pair* q = pr + s0 + 1 + (lane & 15);
  const int nrow = t0 - s0 - 1, last = N + 31 - s0 - 1 - (lane & 15);  // (reads stay inside the zero pairs behind T)
  tb_pair cur = q[0];
  for (int i0 = 0; i0 < nrow; i0 += 16) {
    const tb_pair nxt = q[min(i0 + 16, last)];
    double dr = cur.x, er = cur.y;
    asm volatile("s_nop 1" : "+v"(dr), "+v"(er));
    const int left = nrow - i0;
#define TB_ROW(n) tb_row<n>(dr, er, x, p, pp, signs);
#define TB_ROW8(o)                                                            \
  {                                                                           \
    TB_ROW(o) TB_ROW(o + 1) TB_ROW(o + 2) TB_ROW(o + 3) TB_ROW(o + 4)         \
    const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pp)));        \
    TB_ROW(o + 5) TB_ROW(o + 6) TB_ROW(o + 7)                                 \
    cnt += __popc((signs ^ (signs >> 1)) & 0xffu);                            \
    p = __builtin_amdgcn_ldexp(p, -e);                                        \
    pp = __builtin_amdgcn_ldexp(pp, -e);                                      \
    ex += e;                                                                  \
  }
    if (left >= 8) TB_ROW8(0)
    if (left >= 16) {
      TB_ROW8(8)
    } else if ((left & 7) != 0) {  // the last rows of the block
      double d8 = left > 8 ? dr : __shfl_xor(dr, 8, 64), e8 = left > 8 ? er : __shfl_xor(er, 8, 64);
      asm volatile("s_nop 1" : "+v"(d8), "+v"(e8));
      const int r = left & 7;
#define TB_TAIL(n) if (r > n) tb_row<8 + n>(d8, e8, x, p, pp, signs);
      TB_TAIL(0) TB_TAIL(1) TB_TAIL(2) TB_TAIL(3) TB_TAIL(4) TB_TAIL(5) TB_TAIL(6)
#undef TB_TAIL
      cnt += __popc((signs ^ (signs >> 1)) & ((1u << r) - 1u));
    }
#undef TB_ROW8
#undef TB_ROW
    cur = nxt;
  }
  return cnt;
}

// The same from both ends: leading minors P of the first rows and trailing minors Q of the last ones, two chains that fill each
// other's waits, joined at row m:  det = P_m Q_{m+1} - e_m^2 P_{m-1} Q_{m+2},  and (inertia of the factorisation twisted at
// m) the count is that of the rows above, plus that of the rows below, plus one if det P_{m-1} Q_{m+1} < 0.  An exact zero of
// P_{m-1} or Q_{m+1} needs no special case here either: of its own change of sign and the one at the join exactly one counts.
// For blocks of TB_TWO rows or more: 124 -> 96 us for one image of 576 tokens, 237 -> 200 for 64, 2.02 -> 1.62 ms for 8 of 2880.
constexpr int TB_TWO = 40;
__device__ __forceinline__ int tb_walk_two(const tb_pair* __restrict__ pr, int s0, int t0, int N, int lane, double x, double& p, int& ex) {
  const int n = t0 - s0, L = (n - 1) / 2, nrow = L - 1;
  double pp = 1.0, q, qq = 1.0;
  p = pr[s0].x - x;
  q = pr[t0 - 1].x - x;
  ex = 0;
  unsigned sp = (unsigned)__double2hiint(p) >> 31, sq = (unsigned)__double2hiint(q) >> 31;
  int cnt = (int)(sp + sq);
  const int l15 = lane & 15, up = s0 + 1 + l15, dn = t0 - 2 - l15;  // first rows of the two chains (clamped reads are not used)
  tb_pair cu = pr[min(up, N + 31)];
  double cd = pr[max(dn, 0)].x, ce = pr[max(dn, 0) + 1].y;
  for (int i0 = 0; i0 < nrow; i0 += 16) {
    const int un = min(up + i0 + 16, N + 31), bn = max(dn - i0 - 16, 0);
    const tb_pair nu = pr[un];
    const double nd = pr[bn].x, ne = pr[bn + 1].y;
    double du = cu.x, eu = cu.y, dd = cd, ed = ce;
    asm volatile("s_nop 1" : "+v"(du), "+v"(eu), "+v"(dd), "+v"(ed));
    const int left = nrow - i0;
#define TB_ROW(k) tb_row<k>(du, eu, x, p, pp, sp); tb_row<k>(dd, ed, x, q, qq, sq);
#define TB_ROW8(o)                                                            \
  {                                                                           \
    TB_ROW(o) TB_ROW(o + 1) TB_ROW(o + 2) TB_ROW(o + 3) TB_ROW(o + 4)         \
    const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pp)));        \
    const int g = __builtin_amdgcn_frexp_exp(fmax(fabs(q), fabs(qq)));        \
    TB_ROW(o + 5) TB_ROW(o + 6) TB_ROW(o + 7)                                 \
    cnt += __popc((sp ^ (sp >> 1)) & 0xffu) + __popc((sq ^ (sq >> 1)) & 0xffu); \
    p = __builtin_amdgcn_ldexp(p, -e);                                        \
    pp = __builtin_amdgcn_ldexp(pp, -e);                                      \
    q = __builtin_amdgcn_ldexp(q, -g);                                        \
    qq = __builtin_amdgcn_ldexp(qq, -g);                                      \
    ex += e + g;                                                              \
  }
    if (left >= 8) TB_ROW8(0)
    if (left >= 16) {
      TB_ROW8(8)
    } else if ((left & 7) != 0) {  // the last rows of the chains
      const bool hi = left > 8;
      double d8 = hi ? du : __shfl_xor(du, 8, 64), e8 = hi ? eu : __shfl_xor(eu, 8, 64);
      double f8 = hi ? dd : __shfl_xor(dd, 8, 64), g8 = hi ? ed : __shfl_xor(ed, 8, 64);
      asm volatile("s_nop 1" : "+v"(d8), "+v"(e8), "+v"(f8), "+v"(g8));
      const int r = left & 7;
#define TB_TAIL(k) if (r > k) { tb_row<8 + k>(d8, e8, x, p, pp, sp); tb_row<8 + k>(f8, g8, x, q, qq, sq); }
      TB_TAIL(0) TB_TAIL(1) TB_TAIL(2) TB_TAIL(3) TB_TAIL(4) TB_TAIL(5) TB_TAIL(6)
#undef TB_TAIL
      cnt += __popc((sp ^ (sp >> 1)) & ((1u << r) - 1u)) + __popc((sq ^ (sq >> 1)) & ((1u << r) - 1u));
    }
#undef TB_ROW8
#undef TB_ROW
    cu = nu;
    cd = nd;
    ce = ne;
  }
  auto neg = [](double v) { return (unsigned)__double2hiint(v) >> 31; };
  const int m = t0 - L - 1;
  if ((n & 1) == 0) {  // one more row from above
    const tb_pair c = pr[m - 1];
    const double pn = fma(c.x - x, p, c.y * pp);
    cnt += (int)(neg(pn) ^ neg(p));
    pp = p;
    p = pn;
  }
  const tb_pair c = pr[m];
  const double det = fma(fma(c.x - x, p, c.y * pp), q, pr[m + 1].y * p * qq);
  cnt += (int)(neg(det) ^ neg(p) ^ neg(q));
  p = det;
  return cnt;
}

// The same for lanes in different blocks: every lane reads its own rows; rows past the block's end are replaced by the
// identity step p_i = p_{i-1}, which changes no sign.
__device__ __forceinline__ int tb_walk_own(const tb_pair* __restrict__ pr, int s, int t, int N, double x, double& p, int& ex) {
  double pp = 1.0;
  p = pr[s].x - x;
  ex = 0;
  unsigned signs = (unsigned)__double2hiint(p) >> 31;
  int cnt = (int)signs;
  for (int i0 = s + 1; __any(i0 < t); i0 += 8) {
    tb_pair c[8];
#pragma unroll
    for (int u = 0; u < 8; u++) c[u] = pr[min(i0 + u, N + 31)];
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const bool in = i0 + u < t;
      const double pn = fma(in ? c[u].x - x : 1.0, p, (in ? c[u].y : 0.0) * pp);
      signs = __builtin_amdgcn_alignbit(signs, (unsigned)__double2hiint(pn), 31);
      pp = in ? p : pp;
      p = pn;
    }
    cnt += __popc((signs ^ (signs >> 1)) & 0xffu);
    const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pp)));
    p = __builtin_amdgcn_ldexp(p, -e);
    pp = __builtin_amdgcn_ldexp(pp, -e);
    ex += e;
  }
  return cnt;
}

// G = 1 << gs lanes per eigenvalue (up to the whole wavefront); blockIdx.y = image.
// The kernel is bound by the chain of dependent operations of a walk over the rows, so it makes few walks:
//  - lanes whose eigenvalues still share one interval cut it together: n lanes evaluate n points that part it evenly, and
//    every lane takes the part that holds its eigenvalue (the neighbours of a wavefront lie close together: four or
//    five walks separate the noise part of a spectrum that spans 1e-6 of ||T||, where halving takes twenty);
//  - a lane alone with an interval that holds exactly one eigenvalue goes on with the secant through the last minor at
//    the two ends (Anderson-Bjoerck weights, Sturm counts keep the bracket), seven to twelve walks instead of thirty;
//  - several lanes alone with their eigenvalue (small calls) bracket the secant's estimate with points at distances that
//    fall geometrically, so that an interval shrinks to the error of the estimate in one walk.
// 18 walks at one lane per eigenvalue (55 by halving alone), 10 with 64 lanes: 0.75 -> 0.24 ms for 64 images of 576 tokens,
// 0.32 -> 0.11 ms for one.
// The search ends at a relative width of 2 eps: T is graded (the reduction meets the large eigenvalues first), its small
// eigenvalues are well determined relative to their size, and the vectors of close ones are as orthogonal as their
// relative gap allows.  What ends below the resolution of the reduction (8 eps ||T||) counts as zero and is left there.
__global__ __launch_bounds__(256) void td_bisect_kernel(const double* __restrict__ prep, size_t prep_stride,
                                                        const double* __restrict__ tnorm, double* __restrict__ lam,
                                                        const int2* __restrict__ blk, int N, int Np, int gs) {
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const tb_pair* __restrict__ pr = reinterpret_cast<const tb_pair*>(prep + (size_t)b * prep_stride);
  const double tn = tnorm[b];
  int ex = 0;
  if (tn > 0.0 && tn < DBL_MAX) (void)frexp(tn, &ex);
  const double up = ldexp(1.0, ex);
  const int G = 1 << gs;
  // whole groups of G lanes past the last eigenvalue repeat it (every lane stays active: the walks read across lanes)
  const int kk = (blockIdx.x * 256 + tid) >> gs, k = min(kk, N - 1);
  const int2 st = blk[(size_t)b * Np + k];
  const int s = st.x, t = st.y, m = k - s;
  // Gershgorin interval of T, slightly widened (scaled units: ||T|| <= 1; blocks need no interval of their own, the
  // search ends at an absolute width)
  const tb_pair ger = pr[N + 32];
  const double widen = 2.0 * TD_EPS * N + 2.0 * DBL_MIN;
  double lo = ger.x - widen, hi = ger.y + widen;
  int clo = 0, chi = t - s;       // eigenvalues of the block below the ends
  double flo = 0.0, fhi = 0.0;    // last minor at the ends (0: not evaluated), times 2^elo, 2^ehi
  int elo = 0, ehi = 0, side = 0, steps = 0;
  double xs = lo, found = 0.0;
  bool done = false, has = false;
  const int s0 = __builtin_amdgcn_readfirstlane(s), t0 = __builtin_amdgcn_readfirstlane(t);
  const bool uniform = __all(s == s0 && t == t0);
  const int up_lane = lane == 0 ? 0 : lane - 1;
  for (int it = 0; it < 160; it++) {
    const double mid = 0.5 * (lo + hi), width = hi - lo;
    done = done || !(mid > lo && mid < hi) || width <= 2.0 * TD_EPS * fabs(mid) || hi <= 2.0 * TD_EPS;
    if (__all(done)) break;
    // the run of lanes that share this interval
    const double ulo = __shfl(lo, up_lane, 64), uhi = __shfl(hi, up_lane, 64);
    const int us = __shfl(s, up_lane, 64);
    const u64 first = __ballot((lane == 0) | (ulo != lo) | (uhi != hi) | (us != s));
    const int r0 = 63 - __builtin_clzll(first & (~0ull >> (63 - lane)));
    const u64 after = lane == 63 ? 0 : first & (~0ull << (lane + 1));
    const int r1 = after ? __builtin_ctzll(after) : 64, n = r1 - r0;
    double x = n > 1 ? lo + width * ((double)(lane - r0 + 1) / (double)(n + 1)) : mid;
    bool secant = false;
    if (n == G && clo == m && chi == m + 1 && flo != 0.0 && fhi != 0.0 && steps < 20 && !done) {
      const double fh = __builtin_amdgcn_ldexp(fhi, min(max(ehi - elo, -2000), 2000));
      const double ratio = fabs(fh / flo);
      const double xe = lo + width * (flo / (flo - fh));
      // a polynomial of this degree is only close to a line near its root: until the ends' values come within a factor
      // of 8 of each other the interval is cut evenly
      if (steps > 0 || (ratio > 0.125 && ratio < 8.0)) {
        steps++;
        if (n > 1) {  // points on both sides of the estimate, from a quarter of the interval down to 2^-38 of it
          const int half = G / 2, sec = lane - r0, q = sec < half ? sec : G - 1 - sec;
          const double off = __builtin_amdgcn_ldexp(width, half == 1 ? -6 : -2 - 36 * q / (half - 1));
          x = fmin(fmax(sec < half ? xe - off : xe + off, lo), hi);
        } else if (steps > 1 && (!(xe > lo && xe < hi) || fabs(xe - xs) <= 2.0 * TD_EPS * fabs(xe))) {
          done = has = true;
          found = xe;
        } else if (xe > lo && xe < hi) {
          secant = true;
          x = xs = xe;
        }
      }
    }
    double p;
    int pe;
    const int cnt = !uniform ? tb_walk_own(pr, s, t, N, x, p, pe)
                    : t0 - s0 >= TB_TWO ? tb_walk_two(pr, s0, t0, N, lane, x, p, pe) : tb_walk(pr, s0, t0, N, lane, x, p, pe);
    // the last point of the run with at most m eigenvalues below it, and the first with more (the counts rise with the point)
    int ms = r0;
    if (n > 1) {
      int step = 32, lo_i = r0 - 1;  // lo_i: largest lane known to have cnt <= m
      for (; step > 0; step >>= 1) {
        const int c = min(lo_i + step, 63);
        const int v = __shfl(cnt, c, 64);
        if (lo_i + step < r1 && v <= m) lo_i += step;
      }
      {  // (a run of 64 needs one more probe)
        const int v = __shfl(cnt, min(lo_i + 1, 63), 64);
        if (lo_i + 1 < r1 && v <= m) lo_i += 1;
      }
      ms = lo_i + 1;
    } else {
      ms = cnt <= m ? r1 : r0;
    }
    const int la = max(ms - 1, 0), ha = min(ms, 63);
    const double xl = __shfl(x, la, 64), xh = __shfl(x, ha, 64), pl = __shfl(p, la, 64), ph = __shfl(p, ha, 64);
    const int el = __shfl(pe, la, 64), eh = __shfl(pe, ha, 64), cl = __shfl(cnt, la, 64), ch = __shfl(cnt, ha, 64);
    if (secant && p == 0.0) { done = has = true; found = x; }
    if (ms > r0 && !done) {  // the lower end moves
      if (secant) {
        if (side == -1) {  // twice in a row: the other end's value is weighed down
          const double w = 1.0 - __builtin_amdgcn_ldexp(pl, min(max(el - elo, -2000), 2000)) / flo;
          fhi *= w > 0.0 ? w : 0.5;
        }
        side = -1;
      }
      lo = xl; flo = pl; elo = el; clo = cl;
    }
    if (ms < r1 && !done) {
      if (secant) {
        if (side == 1) {
          const double w = 1.0 - __builtin_amdgcn_ldexp(ph, min(max(eh - ehi, -2000), 2000)) / fhi;
          flo *= w > 0.0 ? w : 0.5;
        }
        side = 1;
      }
      hi = xh; fhi = ph; ehi = eh; chi = ch;
    }
  }
  if ((lane & (G - 1)) == 0 && kk < N) lam[(size_t)b * Np + k] = (has ? found : 0.5 * (lo + hi)) * up;
}

// ---- 2b -----------------------------------------------------------------------------------------------
// One lane per eigenvector: T - l I = L D+ L^T from the top (pivots dp), = U D- U^T from the bottom (pivots dm), joined at the row r
// with the smallest |gamma|, gamma_i = dp_i + dm_i - (d_i - l); z_r = 1, upwards z_i = -(e_i / dp_i) z_{i+1}, downwards
// z_i = -(e_{i-1} / dm_i) z_{i-1}.
// The pivots are ratios of neighbouring minors, dp_i = P_i / P_{i-1} with P_i = (d_i - l) P_{i-1} - e_{i-1}^2 P_{i-2}, and so are the
// steps of the vector: z_i = c_i P_{i-1} with c_r = 1 / P_{r-1} and c_i = -e_i c_{i+1} (from the bottom with Q_{i+1} the same).  A row
// so takes a multiply-add on the chain and no division, where dp_{i+1} = d_{i+1} - l - e_i (e_i / dp_i) has a reciprocal
// with its Newton steps there, and no pivot needs to be kept off zero.  (The error of either form is that of T's entries off by a few eps each.)
// Divisions are left in gamma, off the chain.
// T is scaled to ||T|| <= 1 by a power of two and the minors are brought back into range every sixteen rows, at which they have
// fallen by 2^-850 at most (from two rows to the next two by e^2, and e > eps / 2) or grown by 3^16.  Where T is
// split they begin anew; segments with such a row have their own instance of the walk.
// W [B][Np][Np] float receives the unnormalised vector of slot k in column k (rows outside its block are zero); rn
// [B][Np] its reciprocal norm (0 if the vector is not finite: weakly coupled parts of T that share an eigenvalue to the last bit;
// that raises any[b], and td_orthogonalise_kernel makes the vector anew).
//
// All lanes of a wavefront walk over the same row at the same time, whatever block their eigenvalue belongs
// to and wherever its twist index lies (a lane ignores rows that are not its own): every access to memory is one
// contiguous run per row.  Two chains, one per wavefront, in each of three walks: minors, gamma (four
// wavefronts, a quarter of the segments each), vector.
// Only the minors at the ends of segments of sixteen rows are kept (ck [4][row / 16][slot]: P of the segment's first row and of the one
// before, Q of its last row and of the one behind); the later walks form the others again from there.
// What bounds it is the instructions of a row, at 7 clocks each (one wavefront on a SIMD): minors 5, vector 8 more, gamma 35.  Before
// (pivots by division, vectors masked row by row and stored by the wavefronts that form them) and now, us: one image of 576 tokens
// 111 and 66, 64 images 178 and 144, two of 1499 287 and 166, one of 64 13.9 and 10.8; by walk for the first: 11, 15 and 35.
constexpr int TW_SEG = 16;

// 1 / x to the last bit or so: hardware estimate and two Newton steps
__device__ __forceinline__ double tw_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// LDS beyond 64 KB, what the kernel itself declares (fixed) and what its launch adds, has to be asked for.
static bool td_lds(const void* kernel, size_t fixed, size_t added) {
  return fixed + added <= 64 * 1024 || hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)added) == hipSuccess;
}

constexpr size_t TW_FIXED = 3 * 4 * 64 * 8 + 4 * 64 * 4 + 64 * 8 + 2 * 2 * TW_SEG * 64 * 4;
static size_t td_twisted_lds(int N) {
  const int nseg = (N + TW_SEG - 1) / TW_SEG;
  return (size_t)(nseg * TW_SEG + 1) * 16 + (size_t)nseg * 4;
}

__global__ __launch_bounds__(256) void td_twisted_kernel(const double* __restrict__ dvec, const double* __restrict__ evec,
                                                        const double* __restrict__ lam, const int2* __restrict__ blk,
                                                        const double* __restrict__ tnorm, double* __restrict__ ckpt,
                                                        size_t ckpt_stride, float* __restrict__ W,
                                                        double* __restrict__ rn, int32_t* __restrict__ any, int N,
                                                        int Np) {
  extern __shared__ __attribute__((aligned(16))) unsigned char tw_smem[];
  __shared__ double gs[4][64], ps[4][64], qs[4][64];
  __shared__ int rs[4][64];
  __shared__ double ns[64];
  __shared__ float zs[2][2][TW_SEG * 64];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, nseg = (N + TW_SEG - 1) / TW_SEG, rows = nseg * TW_SEG;
  tb_pair* de = reinterpret_cast<tb_pair*>(tw_smem);   // [rows + 1]: d_i, and e_{i-1} that couples rows i - 1 and i (0 where T is split)
  int* cut = reinterpret_cast<int*>(de + rows + 1);    // [nseg]: T is split in the segment or at one of its ends
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double* db = dvec + (size_t)b * Np;
  const double* eb = evec + (size_t)b * Np;
  const double tn = tnorm[b], split = TD_EPS * tn;
  int ex = 0;
  if (tn > 0.0 && tn < DBL_MAX) (void)frexp(tn, &ex);
  const double down = ldexp(1.0, -ex);
  for (int c = tid; c < nseg; c += 256) cut[c] = 0;
  __syncthreads();
  for (int i = tid; i <= rows; i += 256) {  // rows behind the last stand alone (4 is nobody's eigenvalue)
    const double e = i > 0 && i < N ? eb[i - 1] : 0.0, es = fabs(e) > split ? e * down : 0.0;
    de[i] = tb_pair{i < N ? db[i] * down : 4.0, es};
    if (es == 0.0 && i > 0 && i < rows) cut[(i - 1) / TW_SEG] = cut[i / TW_SEG] = 1;
  }
  __syncthreads();
  const int k = blockIdx.x * 64 + lane, kr = min(k, N - 1);  // (lanes past the last vector repeat it and store nothing but minors)
  const int2 st = blk[(size_t)b * Np + kr];
  const int s = st.x, t = st.y;
  const double l = lam[(size_t)b * Np + kr] * down;
  const size_t part = (size_t)nseg * Np;
  double* ck = ckpt + (size_t)b * ckpt_stride + k;
  float* w = W + (size_t)b * Np * Np + k;

  // Minors of the rows of segment c (f) and of the row before each (g), from those of its first row; then those of the row behind the
  // segment, times 2^-k.  With `split` they begin anew where T is split.
  auto leading = [&](auto split, int c, double& p, double& pp, double* f, double* g) __attribute__((always_inline)) {
    const tb_pair* a = de + c * TW_SEG + 1;
#pragma unroll
    for (int u = 0; u < TW_SEG; u++) {
      f[u] = p;
      g[u] = pp;
      const tb_pair r = a[u];
      const double m = split && r.y == 0.0 ? 1.0 : p;
      p = fma(r.x - l, m, -r.y * r.y * pp);
      pp = m;
    }
    const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pp)));
    p = __builtin_amdgcn_ldexp(p, -e);
    pp = __builtin_amdgcn_ldexp(pp, -e);
    return e;
  };
  // The same from the last row upwards (g: of the row behind), up to the row before the segment (not for segment 0).
  auto trailing = [&](auto split, int c, double& q, double& qq, double* f, double* g) __attribute__((always_inline)) {
    const tb_pair* a = de + c * TW_SEG;
    double y = a[TW_SEG - 1].y;
#pragma unroll
    for (int u = TW_SEG - 1; u >= 0; u--) {
      f[u] = q;
      g[u] = qq;
      if (u == 0 && c == 0) break;
      const tb_pair r = a[u - 1];
      const double m = split && y == 0.0 ? 1.0 : q;
      q = fma(r.x - l, m, -y * y * qq);
      qq = m;
      y = r.y;
    }
    const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(q), fabs(qq)));
    q = __builtin_amdgcn_ldexp(q, -e);
    qq = __builtin_amdgcn_ldexp(qq, -e);
    return e;
  };
  auto segment = [&](int c, auto work) __attribute__((always_inline)) {
    if (__builtin_amdgcn_readfirstlane(cut[c])) work(std::true_type{});
    else work(std::false_type{});
  };

  if (wv == 0) {
    double p = de[0].x - l, pp = 1.0;
    for (int c = 0; c < nseg; c++) {
      ck[(size_t)c * Np] = p;
      ck[part + (size_t)c * Np] = pp;
      if (c + 1 < nseg)
        segment(c, [&](auto split) __attribute__((always_inline)) {
          double f[TW_SEG], g[TW_SEG];
          leading(split, c, p, pp, f, g);
        });
    }
  } else if (wv == 1) {
    double q = de[rows - 1].x - l, qq = 1.0;
    for (int c = nseg - 1; c >= 0; c--) {
      ck[2 * part + (size_t)c * Np] = q;
      ck[3 * part + (size_t)c * Np] = qq;
      if (c > 0)
        segment(c, [&](auto split) __attribute__((always_inline)) {
          double f[TW_SEG], g[TW_SEG];
          trailing(split, c, q, qq, f, g);
        });
    }
  }
  __syncthreads();
  // twist index: the row with the smallest |gamma| (the last of equal ones wins); a quarter of the segments each
  double gbest = DBL_MAX, pbest = 0.0, qbest = 0.0;
  int r = -1;
  const int c0 = nseg * wv / 4, c1 = nseg * (wv + 1) / 4;
  if (c0 < c1) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; u++) v[u] = ck[u * part + (size_t)c0 * Np];
    for (int c = c0; c < c1; c++) {
      const int cn = min(c + 1, c1 - 1);
      double vn[4];
#pragma unroll
      for (int u = 0; u < 4; u++) vn[u] = ck[u * part + (size_t)cn * Np];
      segment(c, [&](auto split) __attribute__((always_inline)) {
        double f[TW_SEG], fp[TW_SEG], h[TW_SEG], hq[TW_SEG];
        leading(split, c, v[0], v[1], f, fp);
        trailing(split, c, v[2], v[3], h, hq);
#pragma unroll
        for (int u = 0; u < TW_SEG; u++) {
          const int i = c * TW_SEG + u;
          const double g = fabs(f[u] * tw_rcp(fp[u]) + h[u] * tw_rcp(hq[u]) - (de[i].x - l));
          const bool take = i >= s && i < t && g <= gbest;  // (a minor of zero before or behind the row: not a number, not taken)
          gbest = take ? g : gbest;
          pbest = take ? fp[u] : pbest;
          qbest = take ? hq[u] : qbest;
          r = take ? i : r;
        }
      });
#pragma unroll
      for (int u = 0; u < 4; u++) v[u] = vn[u];
    }
  }
  gs[wv][lane] = gbest;
  ps[wv][lane] = pbest;
  qs[wv][lane] = qbest;
  rs[wv][lane] = r;
  __syncthreads();
  r = t - 1;
  gbest = DBL_MAX;
  pbest = qbest = 0.0;  // (no row taken, each having a minor of zero before or behind it: the vector comes out not finite)
#pragma unroll
  for (int u = 0; u < 4; u++) {
    const double g = gs[u][lane];
    const int ru = rs[u][lane];
    const bool take = ru >= 0 && g <= gbest;
    gbest = take ? g : gbest;
    pbest = take ? ps[u][lane] : pbest;
    qbest = take ? qs[u][lane] : qbest;
    r = take ? ru : r;
  }
  // The vector: wavefront 0 upwards from r over the segments from the last to the first, wavefront 1 downwards from the first to
  // the last, and the other two store what these had a segment ago.  (A wavefront that stores waits for its stores with its next
  // read.)  c is zero behind r and, as T is split there, outside the block: nothing is masked but what is stored.  (A vector that is not
  // finite stays so across the split: see the end.)
  const bool on = k < N;
  double nrm = 0.0, cc = 0.0, start = 0.0, p = 0.0, pp = 0.0;
  auto couplings = [&](int c, double* y) __attribute__((always_inline)) {  // (before the selects, which would be branches around the reads)
#pragma unroll
    for (int u = 0; u < TW_SEG; u++) y[u] = de[c * TW_SEG + u].y;
#pragma unroll
    for (int u = 0; u < TW_SEG; u++) asm volatile("" : "+v"(y[u]));
  };
  if (wv < 2) {
    start = 1.0 / (wv == 0 ? pbest : qbest);
    const double* from = ck + (wv == 0 ? (size_t)(nseg - 1) * Np : 2 * part);
    p = from[0];
    pp = from[part];
  }
  asm volatile("" : "+v"(p), "+v"(pp));
  for (int it = 0; it <= nseg; it++) {
    if (wv == 0 && it < nseg) {
      const int c = nseg - 1 - it, cn = max(c - 1, 0);
      const double pn = ck[(size_t)cn * Np], ppn = ck[part + (size_t)cn * Np];
      float* z = zs[0][it & 1] + lane;
      segment(c, [&](auto split) __attribute__((always_inline)) {
        double f[TW_SEG], g[TW_SEG], en[TW_SEG];
        couplings(c, en);
        const double last = de[(c + 1) * TW_SEG].y;
        const int e = leading(split, c, p, pp, f, g);
        cc = __builtin_amdgcn_ldexp(cc, -e);  // (the minors of this segment are 2^e of the next one's)
#pragma unroll
        for (int u = TW_SEG - 1; u >= 0; u--) {
          const int i = c * TW_SEG + u;
          const double down = -(u + 1 < TW_SEG ? en[u + 1 < TW_SEG ? u + 1 : u] : last) * cc;
          cc = i == r ? start : down;
          const double y = g[u] * cc;
          nrm = fma(y, y, nrm);
          z[64 * u] = (float)y;
        }
      });
      p = pn;
      pp = ppn;
      asm volatile("" : "+v"(p), "+v"(pp));  // (waited for here, not behind the branches, where those that store would wait too)
    } else if (wv == 1 && it < nseg) {
      const int c = it, cn = min(c + 1, nseg - 1);
      const double pn = ck[2 * part + (size_t)cn * Np], ppn = ck[3 * part + (size_t)cn * Np];
      float* z = zs[1][it & 1] + lane;
      segment(c, [&](auto split) __attribute__((always_inline)) {
        double f[TW_SEG], g[TW_SEG], en[TW_SEG];
        couplings(c, en);
        const int e = trailing(split, c, p, pp, f, g);
        if (c > 0) cc = __builtin_amdgcn_ldexp(cc, -e);
#pragma unroll
        for (int u = 0; u < TW_SEG; u++) {
          const int i = c * TW_SEG + u;
          const double down = -en[u] * cc;
          cc = i == r ? start : down;
          const double y = g[u] * cc;
          nrm = fma(y, y, nrm);
          z[64 * u] = (float)y;
        }
      });
      p = pn;
      pp = ppn;
      asm volatile("" : "+v"(p), "+v"(pp));  // (waited for here, not behind the branches, where those that store would wait too)
    } else if (wv >= 2 && it > 0) {
      const int c = wv == 2 ? nseg - it : it - 1;
      const float* z = zs[wv - 2][(it - 1) & 1] + lane;
      const int i0 = wv == 2 ? 0 : r + 1, i1 = !on ? 0 : wv == 2 ? r + 1 : N;  // rows this wavefront stores
      float y[TW_SEG];
#pragma unroll
      for (int u = 0; u < TW_SEG; u++) y[u] = z[64 * u];
#pragma unroll
      for (int u = 0; u < TW_SEG; u++)
        if (c * TW_SEG + u >= i0 && c * TW_SEG + u < i1) w[(size_t)(c * TW_SEG + u) * Np] = y[u];
    }
    __syncthreads();
  }
  if (wv == 1) ns[lane] = nrm;
  __syncthreads();
  if (wv != 0 || !on) return;
  nrm += ns[lane] - 1.0;  // (row r is in both)
  const bool fin = nrm == nrm && nrm < DBL_MAX && nrm < 1e60;  // float storage of z holds |z| < 3e38 relative to z_r = 1
  rn[(size_t)b * Np + k] = fin ? 1.0 / sqrt(nrm) : 0.0;
  if (!fin) {  // made anew in its block only; the back-transformation reads all rows, also of a vector without weight
    atomicOr(&any[b], 1);
    for (int i = 0; i < s; i++) w[(size_t)i * Np] = 0.f;
    for (int i = t; i < N; i++) w[(size_t)i * Np] = 0.f;
  }
}

// ---- close eigenvalues inside one block -----------------------------------------------------------------
// The vectors of one block are computed independently of each other.  A run is a set of neighbouring slots of one block,
// each closer than 1e-10 ||T|| to the next; vectors of different runs are orthogonal to about eps / 1e-10 and are left as they
// are.  td_pairs_kernel compares every two vectors of a run; where two are not orthogonal to 1e-6 (T is not graded there, or
// the eigenvalues agree to their last bits), td_orthogonalise_kernel orthogonalises all from the one to the other: comparing
// neighbours only, or mending single slots, leaves pairs further apart as they were (up to 7e-5 in groups of four).  The rest of
// the run, hundreds of vectors where rows have been averaged by attention, came out orthogonal and stays.  Eigenvalues that
// count as zero (below the resolution of the reduction) get weight 0 in Eq. 3-6: their vectors are left as they are, however
// many of them there are (the null space of a rank-deficient matrix).
constexpr double TD_CLOSE = 1e-10;             // of ||T||
constexpr float TD_ORTHOGONAL = 1e-6f;         // largest scalar product of two unit vectors that passes
__device__ inline double td_zero_floor(double tn) { return tn > 0.0 ? 8.0 * TD_EPS * tn : DBL_MAX; }  // (every eigenvalue of an all-zero matrix is zero)
// slot k belongs to the run of slot k - 1
__device__ inline bool td_close(const double* lb, const int2* bb, double tn, int k, int N) {
  const double zero = td_zero_floor(tn);
  return k > 0 && k < N && bb[k].x == bb[k - 1].x && lb[k] - lb[k - 1] <= TD_CLOSE * tn && lb[k] > zero && lb[k - 1] > zero;
}

// A product of all vectors in runs, U^T (U r) - r with r of no particular values, shows whether any two are not orthogonal for the
// price of two passes over the vectors; four such r leave a pair that is off by 1e-5 a chance of 1e-4 to hide (by 1e-4, of
// 1e-8).  Above 576 tokens the pairs of an image are compared only where this finds something: for eight images of 2880
// tokens with runs of two thousand the comparison is 0.9 ms on the matrix cores, the product 0.11.
constexpr int TP_R = 4;
constexpr int TP_ABOVE = 576;
__device__ inline double td_probe_weight(int p, int k) {  // between 0.5 and 1 in size
  uint32_t h = (uint32_t)(TP_R * k + p + 1) * 0x9e3779b1u;
  h = (h ^ (h >> 16)) * 0xa3b1956bu;
  h ^= h >> 13;
  const double v = 0.5 + (double)(h & 0x7fffffu) * 0x1p-24;
  return (h >> 31) ? -v : v;
}
__device__ inline bool td_in_run(const double* lb, const int2* bb, double tn, int k, int N) {
  return td_close(lb, bb, tn, k, N) || td_close(lb, bb, tn, k + 1, N);
}

// y = U r of 64 rows (y [Np][TP_R] of the image in `ckpt`, which td_twisted_kernel is done with).
constexpr int TP_THREADS = 1024, TP_WAVES = TP_THREADS / 64;
__global__ __launch_bounds__(TP_THREADS) void td_probe_rows_kernel(const double* __restrict__ lam, const int2* __restrict__ blk,
                                                            const double* __restrict__ tnorm, const float* __restrict__ W,
                                                            const double* __restrict__ rn, double* __restrict__ ckpt,
                                                            size_t ckpt_stride, int N, int Np) {
  extern __shared__ float weight[];  // [TP_R][N]: over the vector's norm, 0 outside runs
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* lb = lam + (size_t)b * Np;
  const int2* bb = blk + (size_t)b * Np;
  const double tn = tnorm[b];
  int found = 0;
  for (int k = tid; k < N; k += TP_THREADS) {
    const bool in = td_in_run(lb, bb, tn, k, N);
    found |= in;
    for (int p = 0; p < TP_R; p++) weight[p * N + k] = in ? (float)(td_probe_weight(p, k) * rn[(size_t)b * Np + k]) : 0.f;
  }
  if (!__syncthreads_or(found)) return;
  double* y = ckpt + (size_t)b * ckpt_stride;
  for (int r = wave; r < 64; r += TP_WAVES) {
    const int i = 64 * blockIdx.x + r;
    if (i >= N) break;
    const float* row = W + ((size_t)b * Np + i) * Np;
    double s[TP_R] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int k = lane; k < N; k += 64) {
      const double v = (double)row[k];
#pragma unroll
      for (int p = 0; p < TP_R; p++) s[p] = fma(v, (double)weight[p * N + k], s[p]);
    }
#pragma unroll
    for (int p = 0; p < TP_R; p++) {
      const double t = wave_sum_dpp(s[p]);
      if (lane == 0) y[(size_t)i * TP_R + p] = t;
    }
  }
}

// need[b] becomes 1 where U^T y is not r.  One workgroup per 64 slots.
__global__ __launch_bounds__(TP_THREADS) void td_probe_slots_kernel(const double* __restrict__ lam, const int2* __restrict__ blk,
                                                             const double* __restrict__ tnorm, const float* __restrict__ W,
                                                             const double* __restrict__ rn, const double* __restrict__ ckpt,
                                                             size_t ckpt_stride, int32_t* __restrict__ need, int N, int Np) {
  __shared__ double part[TP_WAVES][TP_R][64];
  const int b = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), k = 64 * blockIdx.x + lane;
  const bool in = td_in_run(lam + (size_t)b * Np, blk + (size_t)b * Np, tnorm[b], k, N);
  if (!__any(in)) return;  // the same in all wavefronts
  const int r0 = blk[(size_t)b * Np + 64 * blockIdx.x].x, r1 = blk[(size_t)b * Np + min(64 * (int)blockIdx.x + 63, N - 1)].y;
  const double* y = ckpt + (size_t)b * ckpt_stride;
  const float* col = W + (size_t)b * Np * Np + k;
  double s[TP_R] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
  for (int i = r0 + wave; i < r1; i += TP_WAVES) {
    const double v = (double)col[(size_t)i * Np];
#pragma unroll
    for (int p = 0; p < TP_R; p++) s[p] = fma(v, y[(size_t)i * TP_R + p], s[p]);
  }
#pragma unroll
  for (int p = 0; p < TP_R; p++) part[wave][p][lane] = s[p];
  __syncthreads();
  if (wave != 0) return;
  bool off = false;
  if (in)
#pragma unroll
    for (int p = 0; p < TP_R; p++) {
      double z = 0.0;
      for (int w = 0; w < TP_WAVES; w++) z += part[w][p][lane];
      z *= rn[(size_t)b * Np + k];
      off = off || !(fabs(z - td_probe_weight(p, k)) <= TD_ORTHOGONAL);
    }
  if (__any(off) && lane == 0) need[b] = 1;
}

// One workgroup per two tiles of 64 slots, the first not before the second; most find no run that reaches from one to the
// other and end.  (Rows that attention has averaged have hundreds of eigenvalues below 1e-10 ||T||: with one workgroup per
// tile and all tiles before it, on the vector units, 227 us for four images of 701 tokens and 473 for two of 1499.)  The
// vectors are read as operands of the float32 matrix cores, at unit length: the products are off by a few 2^-24.
// mark [B][Np], N before, becomes the first slot of the run whose vector is not orthogonal to that of the slot (which need not
// be looked at where td_twisted_kernel found no vector); any [B] collects.
typedef __attribute__((ext_vector_type(4))) float f4;
__global__ __launch_bounds__(256) void td_pairs_kernel(const double* __restrict__ lam, const int2* __restrict__ blk,
                                                       const double* __restrict__ tnorm, const float* __restrict__ W,
                                                       const double* __restrict__ rn, int32_t* __restrict__ mark,
                                                       int32_t* __restrict__ any, const int32_t* __restrict__ need, int N,
                                                       int Np) {
  constexpr int ST = 8;      // steps of four rows in flight
  __shared__ int start[64];  // the first slot, of this run of slot k0 + i, that lies in the second tile or behind it
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (need && !need[b]) return;
  int tj = blockIdx.x, ti = 0;
  while (tj >= ti + 1) { tj -= ti + 1; ti++; }
  const int k0 = 64 * ti, j0 = 64 * tj;
  const double* lb = lam + (size_t)b * Np;
  const int2* bb = blk + (size_t)b * Np;
  const double* rb = rn + (size_t)b * Np;
  const double tn = tnorm[b];
  const u64 cl = __ballot(td_close(lb, bb, tn, k0 + lane, N));  // the same in all four wavefronts
  if (cl == 0) return;
  int before = k0;
  if (ti != tj) {  // does the run of slot k0 begin in the second tile or before it?
    if (!(cl & 1)) return;
    for (int t = k0 - 64; t > j0; t -= 64)
      if (~__ballot(td_close(lb, bb, tn, t + lane, N))) return;
    const u64 open = ~__ballot(td_close(lb, bb, tn, j0 + lane, N));
    before = open ? j0 + 63 - __builtin_clzll(open) : j0;
  }
  if (wave == 0) {
    const u64 open = ~cl & (~0ull >> (63 - lane));
    start[lane] = open ? k0 + 63 - __builtin_clzll(open) : before;
  }
  __syncthreads();
  // a wavefront compares 32 slots of the first tile with 32 of the second
  const int kw = 32 * (wave >> 1), ka = k0 + kw, ja = j0 + 32 * (wave & 1), l31 = lane & 31;
  if (!__any(ka + l31 < N && ja < ka + l31 && start[kw + l31] <= ja + 31)) return;
  const int l15 = lane & 15, q4 = lane >> 4;
  const int r0 = bb[j0].x, r1 = bb[min(k0 + 63, N - 1)].y;  // rows of the blocks that meet here (a vector is zero outside its own)
  const float* Wb = W + (size_t)b * Np * Np;
  const float* src[4] = {Wb + ka + l15, Wb + ka + 16 + l15, Wb + ja + l15, Wb + ja + 16 + l15};
  float unit[4];
#pragma unroll
  for (int u = 0; u < 4; u++) unit[u] = (float)rb[min((u < 2 ? ka : ja) + 16 * (u & 1) + l15, N - 1)];
  f4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int y = 0; y < 2; y++) acc[x][y] = f4{0.f, 0.f, 0.f, 0.f};
  float cur[ST][4], nxt[ST][4];
  auto load = [&](int r, float (*d)[4]) {
#pragma unroll
    for (int t = 0; t < ST; t++)
#pragma unroll
      for (int u = 0; u < 4; u++) d[t][u] = src[u][(size_t)min(r + 4 * t + q4, r1 - 1) * Np];
  };
  load(r0, cur);
  for (int r = r0; r < r1; r += 4 * ST) {
    load(r + 4 * ST, nxt);
#pragma unroll
    for (int t = 0; t < ST; t++) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; u++) v[u] = r + 4 * t + q4 < r1 ? cur[t][u] * unit[u] : 0.f;
#pragma unroll
      for (int x = 0; x < 2; x++)
#pragma unroll
        for (int y = 0; y < 2; y++) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[x], v[2 + y], acc[x][y], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < ST; t++)
#pragma unroll
      for (int u = 0; u < 4; u++) cur[t][u] = nxt[t][u];
  }
  bool found = false;
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int y = 0; y < 2; y++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int i = 16 * x + 4 * q4 + e, k = ka + i, j = ja + 16 * y + l15;
        if (k < N && j < k && j >= start[kw + i] && !(fabsf(acc[x][y][e]) <= TD_ORTHOGONAL) && rb[k] > 0.0 && rb[j] > 0.0) {
          atomicMin(&mark[(size_t)b * Np + k], j);
          found = true;
        }
      }
  if (__any(found) && lane == 0) atomicOr(&any[b], 1);
}

// What td_pairs_kernel and td_twisted_kernel have marked (few calls have any), a workgroup for the runs that begin in its
// TO_SLOTS slots.  Slots from a marked one back to its mark, and those that overlap, form a cluster: every vector of it is
// orthogonalised, in float64 and twice, against the earlier ones.  Where less than a tenth of a vector is left (two eigenvalues
// that agree to their last bits may come out with one vector), or there was none, it is made anew by inverse iteration: a
// vector of no particular direction is made orthogonal to the others of the run (but those of the cluster that are still to
// come), multiplied by (T - lambda)^-1 and made orthogonal again, three times.  lambda is taken 64 eps ||T|| off the eigenvalue,
// which multiplies all that agree with it alike (at the eigenvalue itself, one of them comes out again and again, however much
// of it the earlier vectors hold) and what lies outside the run by 1.4e-4 of that.  An image for which this fails (T is not
// finite) gets bad[b], and the caller's info turns negative.
constexpr int TO_THREADS = 512, TO_WAVES = TO_THREADS / 64;
constexpr int TO_SLOTS = 16;  // of a workgroup (288 pairs in one image of 577 tokens: a chain of 0.4 ms each)
constexpr size_t TO_FIXED = TO_WAVES * 8;
static size_t td_orthogonalise_lds(int N) { return (size_t)N * 5 * 8 + (TO_WAVES + 1) * 64 * 8 + round_up(N, 16) + (size_t)N * 4; }

__global__ __launch_bounds__(TO_THREADS) void td_orthogonalise_kernel(const double* __restrict__ dvec, const double* __restrict__ evec,
                                                                      const double* __restrict__ lam, const int2* __restrict__ blk,
                                                                      const double* __restrict__ tnorm, const int32_t* __restrict__ mark,
                                                                      const int32_t* __restrict__ any, float* __restrict__ W,
                                                                      double* __restrict__ rn, int32_t* __restrict__ bad, int N, int Np) {
  const int b = blockIdx.y;
  if (!any[b]) return;
  extern __shared__ __attribute__((aligned(16))) unsigned char to_smem[];
  double* x = reinterpret_cast<double*>(to_smem);  // [N] the vector in hand
  double* pd = x + N;                              // [N] factors of T - lambda: pivots,
  double* pu = pd + N;                             // [N] first
  double* pv = pu + N;                             // [N] and second superdiagonal,
  double* pl = pv + N;                             // [N] multipliers,
  double* part = pl + N;                           // [TO_WAVES][64]
  double* coef = part + TO_WAVES * 64;             // [64]
  int* low = reinterpret_cast<int*>(coef + 64);    // [N] the smallest mark of slot i and all behind it
  uint8_t* sw = reinterpret_cast<uint8_t*>(low + N);  // [N] 1: rows i and i + 1 have changed places
  __shared__ double wsum[TO_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* db = dvec + (size_t)b * Np;
  const double* eb = evec + (size_t)b * Np;
  const double* lb = lam + (size_t)b * Np;
  const int2* bb = blk + (size_t)b * Np;
  const int32_t* mb = mark + (size_t)b * Np;
  double* rb = rn + (size_t)b * Np;
  float* Wb = W + (size_t)b * Np * Np;
  const double tn = tnorm[b], tiny = TD_EPS * tn;

  auto norm2 = [&](int n) {  // of x, the same in every thread
    double v = 0.0;
    __syncthreads();
    for (int i = tid; i < n; i += TO_THREADS) v = fma(x[i], x[i], v);
    v = wave_sum(v);
    if (lane == 0) wsum[wave] = v;
    __syncthreads();
    double t = 0.0;
    for (int q = 0; q < TO_WAVES; q++) t += wsum[q];
    return t;
  };
  auto scale = [&](int n, double f) {
    for (int i = tid; i < n; i += TO_THREADS) x[i] *= f;
    __syncthreads();
  };
  // x less its parts along the vectors of slots j0 .. j1 - 1 (rows s .. s + n - 1), 64 at a time
  auto project = [&](int j0, int j1, int s, int n) {
    for (int j = j0; j < j1; j += 64) {
      const int cnt = min(64, j1 - j), jl = j + min(lane, cnt - 1);
      double v = 0.0;
      __syncthreads();
      for (int i = wave; i < n; i += TO_WAVES) v = fma((double)Wb[(size_t)(s + i) * Np + jl], x[i], v);
      part[wave * 64 + lane] = v;
      __syncthreads();
      if (wave == 0) {
        double t = 0.0;
        for (int q = 0; q < TO_WAVES; q++) t += part[q * 64 + lane];
        coef[lane] = lane < cnt && rb[jl] > 0.0 ? t * rb[jl] * rb[jl] : 0.0;  // column j has norm 1 / rb[j], or is none (0)
      }
      __syncthreads();
      for (int i = tid; i < n; i += TO_THREADS) {
        const float* row = Wb + (size_t)(s + i) * Np + j;
        double v2 = x[i];
        for (int c = 0; c < cnt; c++) v2 = coef[c] != 0.0 ? fma(-coef[c], (double)row[c], v2) : v2;
        x[i] = v2;
      }
    }
    __syncthreads();
  };
  // T - lambda of rows s .. s + n - 1 as triangular factors, rows exchanged for the larger pivot (one thread: a chain)
  auto factor = [&](int s, int n, double l) {
    double d = db[s] - l, u = n > 1 ? eb[s] : 0.0;
    for (int i = 0; i + 1 < n; i++) {
      const double e = eb[s + i], dn = db[s + i + 1] - l, un = i + 2 < n ? eb[s + i + 1] : 0.0;
      if (fabs(d) >= fabs(e)) {
        const double m = e / d;
        pd[i] = d; pu[i] = u; pv[i] = 0.0; pl[i] = m; sw[i] = 0;
        d = dn - m * u;
        u = un;
      } else {
        const double m = d / e;
        pd[i] = e; pu[i] = dn; pv[i] = un; pl[i] = m; sw[i] = 1;
        d = u - m * dn;
        u = -m * un;
      }
    }
    pd[n - 1] = fabs(d) < tiny ? tiny : d;
    pu[n - 1] = pv[n - 1] = 0.0;
  };
  auto solve = [&](int n) {
    double p = x[0];
    for (int i = 0; i + 1 < n; i++) {
      const double q = x[i + 1], m = pl[i];
      if (sw[i]) { x[i] = q; p = p - m * q; }
      else { x[i] = p; p = q - m * p; }
    }
    double y1 = p / pd[n - 1], y2 = 0.0;
    x[n - 1] = y1;
    for (int i = n - 2; i >= 0; i--) {
      const double y = (x[i] - pu[i] * y1 - pv[i] * y2) / pd[i];
      x[i] = y;
      y2 = y1;
      y1 = y;
    }
  };

  // low: each thread its own stretch from the back, then what lies behind the stretch (part as 512 ints)
  {
    int* tail = reinterpret_cast<int*>(part);
    const int per = (N + TO_THREADS - 1) / TO_THREADS, i0 = min(N, tid * per), i1 = min(N, i0 + per);
    int m = N;
    for (int i = i1 - 1; i >= i0; i--) low[i] = m = min(m, mb[i]);
    tail[tid] = m;
    __syncthreads();
    m = N;
    for (int t = tid + 1; t < TO_THREADS; t++) m = min(m, tail[t]);
    for (int i = i0; i < i1; i++) low[i] = min(low[i], m);
    __syncthreads();
  }

  for (int begin = blockIdx.x * TO_SLOTS; begin < min(N, (int)(blockIdx.x + 1) * TO_SLOTS); begin++) {
    if (td_close(lb, bb, tn, begin, N)) continue;  // (uniform, as all that follows)
    const int s = bb[begin].x, n = bb[begin].y - s;
    if (rb[begin] == 0.0 && !(lb[begin] > td_zero_floor(tn))) {  // (a run of its own) its weight is zero
      for (int i = tid; i < n; i += TO_THREADS) Wb[(size_t)(s + i) * Np + begin] = 0.f;
      continue;
    }
    int stop = begin + 1;  // end of the run
    while (td_close(lb, bb, tn, stop, N)) stop++;
    for (int first = begin, end; first < stop; first = end) {
      end = first + 1;  // end of the cluster
      while (end < stop && low[end] < end) end++;
      for (int k = first; k < end; k++) {
        const double r = rb[k];
        if (k == first && r > 0.0) continue;
        double left = 0.0;
        if (r > 0.0) {
          __syncthreads();
          for (int i = tid; i < n; i += TO_THREADS) x[i] = (double)Wb[(size_t)(s + i) * Np + k] * r;
          __syncthreads();
          project(first, k, s, n);
          project(first, k, s, n);
          left = norm2(n);
        }
        if (!(left >= 0.01)) {
          __syncthreads();
          if (tid == 0) factor(s, n, lb[k] + 64.0 * tiny);
          for (int i = tid; i < n; i += TO_THREADS) {
            uint32_t h = (uint32_t)(i + 1) * 0x9e3779b1u ^ (uint32_t)(k + 1) * 0xa3b1956bu;
            h = (h ^ (h >> 15)) * 0x5f8c2e17u;
            x[i] = (double)(int32_t)(h ^ (h >> 13)) * 0x1p-31;
          }
          __syncthreads();
          auto others = [&]() {
            project(begin, k, s, n);
            project(end, stop, s, n);
          };
          others();
          bool ok = false;
          for (int it = 0; it < 6 && !ok; it++) {
            scale(n, 1.0 / sqrt(norm2(n)));
            if (tid == 0) solve(n);
            const double y2 = norm2(n);
            if (!(y2 > 0.0 && y2 < DBL_MAX)) break;
            scale(n, 1.0 / sqrt(y2));
            others();
            others();
            left = norm2(n);
            ok = it > 1 && left >= 0.25;
          }
          if (!ok) {
            if (tid == 0) {
              bad[b] = 1;
              rb[k] = 0.0;
            }
            __syncthreads();
            continue;
          }
        }
        const double f = 1.0 / sqrt(left);
        __syncthreads();
        for (int i = tid; i < n; i += TO_THREADS) {
          const float y = (float)(x[i] * f);
          Wb[(size_t)(s + i) * Np + k] = y;
          x[i] = (double)y;
        }
        const double v = norm2(n);
        if (tid == 0) rb[k] = 1.0 / sqrt(v);
        __syncthreads();
      }
    }
  }
}

// ---- weights of Eq. 3-6 -----------------------------------------------------------------------------------
// sigma_k = sqrt(max(lambda_k, 0)); wgt[k] = sigma_k * rn[k] (0 for terms dropped by sv_rtol): the factor that
// turns the unnormalised vector of slot k into its term of C.  Also the optional outputs of tc_ipgs_score that
// do not need the vectors: sigma sorted in descending order, and info.
__global__ __launch_bounds__(256) void td_weights_kernel(const double* __restrict__ lam, const double* __restrict__ rn,
                                                         const double* __restrict__ tnorm,
                                                         const int32_t* __restrict__ bad, float sv_rtol,
                                                         double* __restrict__ sig, double* __restrict__ wgt,
                                                         float* __restrict__ sigma_out, int32_t* __restrict__ info_out,
                                                         int N, int Np) {
  extern __shared__ float key[];  // pow2 >= N floats, only when sigma_out != nullptr
  __shared__ double wmax[4];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* lb = lam + (size_t)b * Np;
  double* sb = sig + (size_t)b * Np;
  // Eigenvalues come out of the reduction and the bisection with an absolute error of a few eps ||T||: what lies
  // below that is zero (an all-zero matrix, the null space of a rank-deficient one).
  const double floor0 = td_zero_floor(tnorm[b]);
  double mx = 0.0;
  int nanflag = 0;
  for (int i = tid; i < Np; i += 256) {
    double s = 0.0;
    if (i < N) {
      const double l = lb[i];
      nanflag |= (l == l) ? 0 : 1;
      s = l > floor0 ? sqrt(l) : 0.0;
    }
    sb[i] = s;
    mx = fmax(mx, s);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    mx = fmax(mx, __shfl_xor(mx, o, 64));
    nanflag |= __shfl_xor(nanflag, o, 64);
  }
  __shared__ int wnan[4];
  if (lane == 0) { wmax[wave] = mx; wnan[wave] = nanflag; }
  __syncthreads();
  const double thr = sv_rtol > 0.f ? (double)sv_rtol * fmax(fmax(wmax[0], wmax[1]), fmax(wmax[2], wmax[3])) : -1.0;
  if (wgt)
    for (int i = tid; i < Np; i += 256) {
      const double s = sb[i];
      wgt[(size_t)b * Np + i] = (i < N && s > thr) ? s * rn[(size_t)b * Np + i] : 0.0;
    }
  if (tid == 0 && info_out)  // 1: done (the method does not iterate); negative: an eigenvector could not be found or the reduction gave up
    info_out[b] = (bad[b] | wnan[0] | wnan[1] | wnan[2] | wnan[3]) ? -1 : 1;
  if (!sigma_out) return;
  int n2 = 1;
  while (n2 < N) n2 <<= 1;
  for (int i = tid; i < n2; i += 256) key[i] = i < N ? (float)sb[i] : -1.0f;
  __syncthreads();
  for (int k = 2; k <= n2; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = tid; i < n2; i += 256) {
        const int l = i ^ j;
        if (l > i) {
          const float a = key[i], c = key[l];
          const bool desc = (i & k) == 0;
          if (desc ? (a < c) : (a > c)) { key[i] = c; key[l] = a; }
        }
      }
      __syncthreads();
    }
  for (int i = tid; i < N; i += 256) sigma_out[(size_t)b * N + i] = key[i];
}

// ---- 3 ------------------------------------------------------------------------------------------------
// U = H_0 H_1 ... H_{N-2} W, sixteen reflectors at a time in compact WY form (the scheme of LAPACK's
// dlarft/dlarfb): H_j0 ... H_j0+15 = I - V T V^T with V the 16 reflectors and T upper triangular,
//     T[c][c] = tau_c,   T[0:c, c] = -tau_c T[0:c, 0:c] (V[:, 0:c]^T v_c).
constexpr int BT_K = 16;  // reflectors per block

// T of every block of 16 reflectors, one workgroup per (block, image).  S = V^T V on the matrix cores: a lane's element
// V[4 s + lane / 16][lane % 16] is operand A and operand B of step s alike, the wavefronts take the steps in turn and
// their parts are added in a fixed order.  Then lane a forms row a of T in registers.  Also clears the rows of the block
// behind the last token (up to a multiple of 16), which the back-transformation reads.
__global__ __launch_bounds__(256) void td_tfactor_kernel(float* __restrict__ Vc, const float* __restrict__ tauv,
                                                         float* __restrict__ Tf, int N, int Np, int npanel) {
  __shared__ float part[4][BT_K][BT_K];
  __shared__ float S[BT_K][BT_K];
  const int p = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, q4 = lane >> 4;
  const int j0 = BT_K * p, rows = N - j0;
  float* Vb = Vc + (size_t)b * Np * Np + (size_t)p * Np * BT_K + (size_t)j0 * BT_K;
  f4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int r = 4 * wave + q4; r - q4 < rows; r += 16) {
    const float v = r < rows ? Vb[(size_t)r * BT_K + l15] : 0.f;
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v, v, acc, 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < 4; j++) part[wave][4 * q4 + j][l15] = acc[j];
  {  // rows N .. round_up(N, 16) - 1
    const int r = rows + (tid >> 4);
    if (r < round_up(N, 16) - j0) Vb[(size_t)r * BT_K + l15] = 0.f;
  }
  __syncthreads();
  {
    const int x = tid / BT_K, c = tid % BT_K;
    S[x][c] = (part[0][x][c] + part[1][x][c]) + (part[2][x][c] + part[3][x][c]);
  }
  __syncthreads();
  if (tid < BT_K) {
    float t[BT_K];
    float* out = Tf + ((size_t)b * npanel + p) * (BT_K * BT_K) + tid * BT_K;
#pragma unroll
    for (int c = 0; c < BT_K; c++) {
      const float tau = j0 + c <= N - 2 ? tauv[(size_t)b * Np + j0 + c] : 0.f;
      float sum = 0.f;
#pragma unroll
      for (int r = 0; r < c; r++) sum += t[r] * S[r][c];  // (t[r] is zero for r < this row)
      t[c] = tid < c ? -tau * sum : (tid == c ? tau : 0.f);
      out[c] = t[c];
    }
  }
}

// A strip of 16 eigenvectors (columns k0 .. k0 + 15 of W) lives in the accumulator registers of NW wavefronts for the
// whole kernel: wavefront w of the strip owns the row tiles rt = NW t + w (16 rows each), t < TPW; element j of a lane is
// (row 4 (lane / 16) + j, column lane % 16) of its tile.  Per block of reflectors, last block first:
//   Z  = V^T U     contraction over rows; the B operand of matrix-core step j is accumulator element j itself
//                  (rows j, 4 + j, 8 + j, 12 + j of the tile), the A operand the matching rows of V;
//                  with NW > 1 the wavefronts' parts are added in a fixed order through LDS
//   Z2 = T Z       one 16x16x16 product, same trick on the accumulator of Z
//   U -= V Z2      likewise on the accumulator of Z2.
// A wavefront reads the rows of V that it owns straight from the L2, BT_AHEAD tiles ahead of the matrix cores (no other
// wavefront of the workgroup uses them in the same strip; staging them in LDS for four strips together cost two barriers
// and a transposing copy per block and kept one wavefront per SIMD: 0.52 ms for 64 images of 576 tokens against the 0.16 ms
// that the matrix cores need).  The tiles are walked from the last one up and the walk ends at the block's own rows, so
// that it is straight code whose loads in flight the compiler can count.
// At the end the strip's share of Eq. 3-6, Cpart[strip][x] = sum_k |U[x][k]| wgt[k],
// is reduced across the 16 lanes of a row and written; U itself is not.
constexpr int BT_AHEAD = 6;
// f(n - 1), f(n - 2), ... f(0) with the index as a constant, until one of them returns false.
template <int n, typename F>
__device__ __forceinline__ void walk_down(F f) {
  [&]<int... i>(std::integer_sequence<int, i...>) { (void)(f(std::integral_constant<int, n - 1 - i>{}) && ...); }(std::make_integer_sequence<int, n>{});
}
template <int TPW, int NW, int SPW>  // SPW strips per workgroup
__global__ __launch_bounds__(64 * NW * SPW) __attribute__((amdgpu_waves_per_eu(2))) void td_backtransform_kernel(const float* __restrict__ W, const float* __restrict__ Vc,
                                                                         const float* __restrict__ Tf,
                                                                         const double* __restrict__ wgt,
                                                                         double* __restrict__ Cpart, int B, int N, int Np, int nstrip,
                                                                         int npanel) {
  __shared__ __attribute__((aligned(16))) float zbuf[NW > 1 ? 2 : 1][SPW][NW > 1 ? NW : 1][NW > 1 ? 256 : 4];
  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, q4 = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), w = wv % NW, sl = wv / NW;
  int b, group;
  if (!group_on_xcd(blockIdx.x, (nstrip + SPW - 1) / SPW, B, &b, &group)) return;  // an image's strips share its reflectors: one XCD
  const int strip = min(group * SPW + sl, nstrip - 1);  // a strip too many repeats the last one (its wavefronts must meet the barriers)
  const int k0 = strip * 16, ntile = (N + 15) >> 4;
  const float* Wb = W + (size_t)b * Np * Np;
  const float* Vb = Vc + (size_t)b * Np * Np;
  const int tl = (ntile - 1 - w) / NW;  // this wavefront's last tile (ntile > w, or it has none)
  const bool any = ntile > w;
  f4 acc[TPW];
#pragma unroll
  for (int t = 0; t < TPW; t++)
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int row = 16 * (NW * t + w) + 4 * q4 + j, col = k0 + l15;
      acc[t][j] = (row < N && col < N) ? Wb[(size_t)row * Np + col] : 0.f;
    }
  for (int p = npanel - 1; p >= 0; p--) {
    const float* Vp = Vb + (size_t)p * Np * BT_K;
    const int tf = p > w ? (p - w + NW - 1) / NW : 0;  // first tile that reaches the block's rows
    const f4 tt = *reinterpret_cast<const f4*>(Tf + ((size_t)b * npanel + p) * (BT_K * BT_K) + l15 * BT_K + 4 * q4);
    constexpr int TS = 16 * NW * BT_K;                              // from one of the wavefront's tiles to the next
    const float* Vt = Vp + 16 * w * BT_K;                           // its tile 0 (uniform)
    const int oz = 4 * q4 * BT_K + l15;                             // rows 4 q4 + j, reflector l15
    const int ou = l15 * BT_K + 4 * q4;                             // row l15, reflectors 4 q4 + j
    auto load_z = [&](int t) {
      const float* s = Vt + t * TS;
      return f4{s[oz], s[oz + BT_K], s[oz + 2 * BT_K], s[oz + 3 * BT_K]};
    };
    auto load_u = [&](int t) { return *reinterpret_cast<const f4*>(Vt + t * TS + ou); };
    f4 ring[BT_AHEAD];
    f4 z = {0.f, 0.f, 0.f, 0.f}, za = z;
    if (any && tl >= tf) {
      // static walk over t = TPW-1 .. 0; tiles past tl are skipped, the walk ends below tf
#pragma unroll
      for (int u = 0; u < BT_AHEAD; u++) ring[(TPW - 1 - u + 16 * BT_AHEAD) % BT_AHEAD] = load_z(min(max(TPW - 1 - u, tf), tl));
      walk_down<TPW>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        if (t < tf) return false;
        const f4 v = ring[t % BT_AHEAD];
        ring[t % BT_AHEAD] = load_z(min(max(t - BT_AHEAD, tf), tl));
        if (t <= tl) {
#pragma unroll
          for (int j = 0; j < 4; j++) {
            if (t & 1) za = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j], acc[t][j], za, 0, 0, 0);
            else z = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j], acc[t][j], z, 0, 0, 0);
          }
        }
        return true;
      });
#pragma unroll
      for (int u = 0; u < BT_AHEAD; u++) ring[(TPW - 1 - u + 16 * BT_AHEAD) % BT_AHEAD] = load_u(min(max(TPW - 1 - u, tf), tl));
    }
    z += za;
    if constexpr (NW > 1) {  // (two buffers in turn: one barrier per block)
      f4* zb = reinterpret_cast<f4*>(&zbuf[p & 1][sl][0][0]);
      zb[w * 64 + lane] = z;
      __syncthreads();
      z = zb[lane];
#pragma unroll
      for (int q = 1; q < NW; q++) z += zb[q * 64 + lane];
    }
    f4 z2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; j++) z2 = __builtin_amdgcn_mfma_f32_16x16x4f32(-tt[j], z[j], z2, 0, 0, 0);
    if (any && tl >= tf) {
      walk_down<TPW>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        if (t < tf) return false;
        const f4 v = ring[t % BT_AHEAD];
        ring[t % BT_AHEAD] = load_u(min(max(t - BT_AHEAD, tf), tl));
        if (t <= tl) {
#pragma unroll
          for (int j = 0; j < 4; j++) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j], z2[j], acc[t], 0, 0, 0);
        }
        return true;
      });
    }
  }
  // Eq. 3-6, this strip's share
  const int col = k0 + l15;
  const double wk = col < N ? wgt[(size_t)b * Np + col] : 0.0;
  double* Cp = Cpart + ((size_t)b * nstrip + strip) * Np;
#pragma unroll
  for (int t = 0; t < TPW; t++)
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const double term = row16_sum_dpp(fabs((double)acc[t][j]) * wk);
      const int row = 16 * (NW * t + w) + 4 * q4 + j;
      if (l15 == 0 && row < N) Cp[row] = term;
    }
}

// C(x) = sum over the strips of their shares, in a fixed order.
__global__ __launch_bounds__(256) void td_ics_finish_kernel(const double* __restrict__ Cpart, float* __restrict__ C,
                                                            float* __restrict__ C_out, int N, int Np, int nstrip) {
  const int b = blockIdx.y, x = blockIdx.x * 256 + threadIdx.x;
  if (x >= N) return;
  double s = 0.0;
#pragma unroll 12
  for (int t = 0; t < nstrip; t++) s += Cpart[((size_t)b * nstrip + t) * Np + x];
  C[(size_t)b * N + x] = (float)s;
  if (C_out) C_out[(size_t)b * N + x] = (float)s;
}

int launch_td_eigen(const Plan& pl, const double* dvec, const double* evec, const float* tauv, float* Vc,
                    double* lam, int2* blk, double* tnorm, double* scratch, float* W, double* rn, int32_t* bad, int32_t* mark, const int32_t* fail,
                    double* sig, double* wgt, double* Cpart, float* Tf, float sv_rtol, bool vectors, float* C, float* C_out,
                    float* sigma_out, int32_t* info_out, hipStream_t st) {
  const int N = pl.N, Np = pl.Np, B = pl.B;
  // The image's part of `scratch` (Np^2 doubles) holds the scaled copy of T first, the minors at the ends of segments later.
  const size_t stride = (size_t)Np * Np;
  int32_t* any = mark + (size_t)B * Np;  // (two words per image behind the marks of the group's images)
  int32_t* need = any + B;
  TC_TIMED(PK_BISECT, 0, st, (td_prepare_kernel<<<B, 256, 0, st>>>(dvec, evec, scratch, stride, tnorm, blk, bad, mark, any, need, fail, N, Np)));
  // lanes per eigenvalue: as many as keep the launch near one wavefront per SIMD (by the size of the whole call, so
  // that an image's result does not depend on how the call is cut into stream groups)
  int gs = 0;
  while (gs < 6 && ((long long)N * pl.batch_call << (gs + 1)) <= 64 * 1024) gs++;
  TC_TIMED(PK_BISECT, 0, st, (td_bisect_kernel<<<dim3(((N << gs) + 255) / 256, B), 256, 0, st>>>(scratch, stride, tnorm, lam, blk, N, Np, gs)));
  int n2 = 1;
  while (n2 < N) n2 <<= 1;
  const size_t shm_sig = sigma_out ? (size_t)n2 * sizeof(float) : 0;
  if (!vectors) {  // eigenvalues only (the information-quantity tool)
    TC_TIMED(PK_BISECT, 1, st, (td_weights_kernel<<<B, 256, shm_sig, st>>>(lam, nullptr, tnorm, bad, 0.f, sig, nullptr, sigma_out, info_out, N, Np)));
    return check_launch();
  }
  {
    const size_t shm = td_twisted_lds(N);
    if (!td_lds(reinterpret_cast<const void*>(td_twisted_kernel), TW_FIXED, shm)) return TC_ERR_HIP;
    TC_TIMED(PK_TWISTED, 0, st, (td_twisted_kernel<<<dim3((N + 63) / 64, B), 256, shm, st>>>(dvec, evec, lam, blk, tnorm, scratch, stride, W, rn, any, N, Np)));
  }
  const int nt = (N + 63) / 64;
  const bool probe = N > TP_ABOVE;
  if (probe) {
    const size_t shm = (size_t)TP_R * N * 4;
    TC_TIMED(PK_TWISTED, 1, st, (td_probe_rows_kernel<<<dim3(nt, B), TP_THREADS, shm, st>>>(lam, blk, tnorm, W, rn, scratch, stride, N, Np)));
    TC_TIMED(PK_TWISTED, 1, st, (td_probe_slots_kernel<<<dim3(nt, B), TP_THREADS, 0, st>>>(lam, blk, tnorm, W, rn, scratch, stride, need, N, Np)));
  }
  TC_TIMED(PK_TWISTED, 1, st, (td_pairs_kernel<<<dim3(nt * (nt + 1) / 2, B), 256, 0, st>>>(lam, blk, tnorm, W, rn, mark, any, probe ? need : nullptr, N, Np)));
  {
    const size_t shm = td_orthogonalise_lds(N);
    if (!td_lds(reinterpret_cast<const void*>(td_orthogonalise_kernel), TO_FIXED, shm)) return TC_ERR_HIP;
    TC_TIMED(PK_TWISTED, 2, st, (td_orthogonalise_kernel<<<dim3((N + TO_SLOTS - 1) / TO_SLOTS, B), TO_THREADS, shm, st>>>(dvec, evec, lam, blk, tnorm, mark, any, W, rn, bad, N, Np)));
  }
  TC_TIMED(PK_BISECT, 1, st, (td_weights_kernel<<<B, 256, shm_sig, st>>>(lam, rn, tnorm, bad, sv_rtol, sig, wgt, sigma_out, info_out, N, Np)));
  const int npanel = (N - 1 + BT_K - 1) / BT_K, nstrip = (N + 15) / 16;  // blocks of reflectors, strips of eigenvectors
  if (npanel > 0) TC_TIMED(PK_BACKTF, 0, st, (td_tfactor_kernel<<<dim3(npanel, B), 256, 0, st>>>(Vc, tauv, Tf, N, Np, npanel)));
#define TC_BACKTF(TPW_, NW_, SPW_)                                                                                                   \
  TC_TIMED(PK_BACKTF, 1, st, (td_backtransform_kernel<TPW_, NW_, SPW_><<<grid_for_groups((nstrip + SPW_ - 1) / SPW_, B), 64 * NW_ * SPW_, 0, st>>>(W, Vc, Tf, wgt, Cpart, B, N, Np, nstrip, npanel)))
  // Wavefronts per strip: as few as hold it (up to 36 row tiles in a wavefront's registers) once the strips alone fill the
  // chip, four (by the size of the whole call: the order of a sum must not depend on stream groups) before that.
  const bool few = (long long)nstrip * pl.batch_call <= 512;
  if (N <= 64) TC_BACKTF(4, 1, 4);
  else if (N <= 256 && few) TC_BACKTF(4, 4, 1);
  else if (N <= 256) TC_BACKTF(16, 1, 4);
  else if (N <= 576 && few) TC_BACKTF(9, 4, 1);
  else if (N <= 576) TC_BACKTF(36, 1, 4);
  else if (N <= 1152) TC_BACKTF(18, 4, 1);
  else if (N <= 2304) TC_BACKTF(18, 8, 1);
  else if (N <= 4096) TC_BACKTF(32, 8, 1);
  else return TC_ERR_SHAPE;
#undef TC_BACKTF
  TC_TIMED(PK_ICS, 0, st, (td_ics_finish_kernel<<<dim3((N + 255) / 256, B), 256, 0, st>>>(Cpart, C, C_out, N, Np, nstrip)));
  return check_launch();
}

}  // namespace tc
