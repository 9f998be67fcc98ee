// Direct symmetric eigensolver, stage 1: reduction of the Gram matrix to tridiagonal form,
//     G = Q T Q^T,   Q = H_0 H_1 ... H_{N-3},   H_j = I - tau_j v_j v_j^T  (Householder reflectors),
// so that the singular vectors of Section 3.3.1 (Z = U Sigma V^T, Z Z^T = U Sigma^2 U^T) become
// U = Q W with T W = W Sigma^2 (stages 2 and 3: tdeig.hip).
//
// Column j needs p = A v_j over the whole trailing matrix, then A <- A - v w^T - w v^T.  From memory that is one
// pass over the matrix per column (or a pass for the product and one for the update per panel), and one compute unit
// per image is bound by what its memory path delivers: 3.5 us of steps plus up to 16 us of product per column at 576
// tokens.  Here the trailing matrix never leaves the registers: a group of P workgroups, one per compute unit, holds
// the lower triangle of one image in its vector registers (90 doubles per thread of 512, 368 KB per compute unit:
// four compute units for 576 tokens, so 64 images fill the 256 of the chip) and updates it in place.  What is left per
// column is latency: one exchange of the partial products between the workgroups of the group (about 1.1 us inside an
// XCD), three barriers with their scalars, and the arithmetic (4 fused multiply-adds per element of the triangle, one
// every 4.3 clocks of a SIMD).  The update runs while the partial products are on their way.  Measured at 576 tokens:
// 2.1 ms for one image, 2.1 to 2.3 for 64 (5.6 and 8.8 ms with the matrix in memory), 40 ms for eight images of 2880 tokens (470 ms), all
// columns by this form.
//
// (tridiag_columns.hip does the same with whole columns, in less than half of the time a column and with twice the compute units; this
// form is for calls whose images fill the device, for more than 2112 tokens, and for small devices.)
//
// Frame.  The matrix is placed at the end of a frame of F x F (row f of the frame is row f + base of the matrix).
// Wavefront w of workgroup (a, b) owns the rows f = i R + 8 a + w (i < LI) and lane l the columns k C + 64 b + l (k < LK), R = 8 PR
// rows and C = 64 PC columns per step, cyclic in both directions so that every thread keeps its share as the trailing
// matrix shrinks; element (i, k) is kept when i >= RT k, RT = C / R: the blocks below the diagonal, and in full
// (both triangles) the C x C blocks on the diagonal.  An element below the diagonal blocks counts twice (row sum and
// column sum), one inside them only for the column sum; no element needs a mask.
//   MODE 0  one workgroup, F = 256: no exchange at all
//   MODE 1  PC = 1, four workgroups, F = 576: every workgroup publishes its partial of p and its rows of the next
//           column, everybody reads the four partials and adds them in the same order
//   MODE 2  PC >= 2, P = 4 PC^2, F = 576 PC: the partials of an element (PR column sums, PC row sums) are added by one
//           workgroup, which publishes the total (two exchanges, but every workgroup reads F values, not 5 PC F)
// The O(F) part of a column (w, the next column, its reflector) is done by every workgroup for itself, bit for bit
// the same.
//
// Exchange.  Values are published with relaxed agent-scope stores and polled with relaxed agent-scope loads; the lowest
// mantissa bit of a value carries the parity of its use of the slot (two slots, used in turn), so a value announces
// itself and no fence or flag is needed.  A slot is written again two columns later, when every workgroup has
// published the column in between and therefore read this one.
// A group waits for its own members, which must all be resident.  Nothing promises that: the hardware deals a launch to the
// XCDs by id and every XCD starts its share by itself, other streams, other processes and replays of graphs compete for the
// compute units.  So the members count themselves in first, and a group that is not complete after a while gives its
// compute units back before it has written anything; tridiag_alone_kernel then reduces the image by one workgroup.  A
// group that is complete stays resident and its waits end.  (They are bounded all the same, TD_SPIN polls: a workgroup that gives up
// raises the image's failure flag, its group follows, and the caller reports the image as failed.)
// Launches of this library that would strand each other are kept apart by the host (see TrTurn).
#include <mutex>

#include "tc_internal.h"
#include "tridiag_device.h"
#include "tridiag_frames.h"

namespace tc {

// d += (value of `row` in lane n of each row of 16 lanes) * c.  `row` holds one matrix row per lane of a row of 16:
// the multiply-add reads the broadcast lane itself, so a row's value costs no instruction of its own.
template <int N>
__device__ __forceinline__ void fmac_bcast(double& d, double row, double c) {
  asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(row), "v"(c), "n"(N));
}

template <int N>
__device__ __forceinline__ void fmac_bcast_neg(double& d, double row, double c) {
  asm("v_fmac_f64_dpp %0, %1, -%2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(row), "v"(c), "n"(N));
}

// Two wait states must lie between a write of a register and its use as a broadcast, and the compiler keeps none for an asm
// operand.  As inputs, the rows are written before the wait; that nothing else writes them on the way to the multiply-adds is
// checked in the compiler's output by a test.  (Tied to the multiply-adds as well, through an operand that passes through,
// a call of one image of 576 tokens takes 2.54 ms in place of 2.52.)
__device__ __forceinline__ void settle(double a, double b) { asm volatile("s_nop 1" : : "v"(a), "v"(b)); }
__device__ __forceinline__ void settle(double a, double b, double c) { asm volatile("s_nop 1" : : "v"(a), "v"(b), "v"(c)); }
__device__ __forceinline__ void settle(double a, double b, double c, double d) { asm volatile("s_nop 1" : : "v"(a), "v"(b), "v"(c), "v"(d)); }

// Sums of 8 or 16 values over the 64 lanes by recursive halving (fixed order).  On return lane L holds the total of value
// *which: the halves and the rows of 16 lanes trade with the swap instructions, then L and L^8, (16 values) L and 7-L
// through lane permutations; what is left of a row of lanes is added.
template <int n>
__device__ __forceinline__ double reduce_many(double* x, int lane, int* which) {
  typedef __attribute__((ext_vector_type(2))) unsigned int u2;
  static_assert(n == 8 || n == 16, "");
#pragma unroll
  for (int u = 0; u < n / 2; u++) {
    const u2 lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x[u]), (unsigned)__double2loint(x[u + n / 2]), false, false);
    const u2 hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x[u]), (unsigned)__double2hiint(x[u + n / 2]), false, false);
    x[u] = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
  }
#pragma unroll
  for (int u = 0; u < n / 4; u++) {
    const u2 lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x[u]), (unsigned)__double2loint(x[u + n / 4]), false, false);
    const u2 hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x[u]), (unsigned)__double2hiint(x[u + n / 4]), false, false);
    x[u] = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
  }
  const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0;
#pragma unroll
  for (int u = 0; u < n / 8; u++)
    x[u] = (b3 ? x[u + n / 8] : x[u]) + dpp_f64<0x128>(b3 ? x[u] : x[u + n / 8]);  // row_ror:8, L <-> L^8
  double t;
  if (n == 16) t = (b2 ? x[1] : x[0]) + dpp_f64<0x141>(b2 ? x[0] : x[1]);  // row_half_mirror, L <-> 7-L
  else t = x[0] + dpp_f64<0x141>(x[0]);
  t += dpp_f64<0xB1>(t);  // quad_perm [1,0,3,2]
  t += dpp_f64<0x4E>(t);  // quad_perm [2,3,0,1]
  *which = ((lane & 32) ? n / 2 : 0) + ((lane & 16) ? n / 4 : 0) + (b3 ? n / 8 : 0) + (n == 16 && b2 ? 1 : 0);
  return t;
}

// Exchange memory of the launch that follows: cleared, so that no value carries the tag of its first use (1).
__global__ __launch_bounds__(256) void tridiag_clear_kernel(u64* __restrict__ sync, size_t stride, size_t words,
                                                            int32_t* __restrict__ fail) {
  u64* p = sync + (size_t)blockIdx.y * stride;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256) p[i] = 0;
  if (fail && blockIdx.x == 0 && threadIdx.x == 0) fail[blockIdx.y] = 0;
}

// G      [B][Np][Np]  in: the Gram matrix (full != 0: stored in full, else the lower triangle of the trailing matrix that the
//                     phase before left); out: the trailing matrix from column last on, lower triangle (mirror != 0: both)
// dvec   [B][Np]      out: diagonal of T
// evec   [B][Np]      out: evec[j] = T[j+1][j], j < N-1
// tauv   [B][Np]      out: tau_j (0 for a reflector that is the identity)
// Vc     [B][Np/16][Np][16] out, float: the reflectors in blocks of sixteen, Vc[j / 16][i][j % 16] = v_j[i] (zeros up to
//                     i = j, 1 at j + 1) -- the layout stage 3 copies into LDS; reflectors j >= N-1 are not written
// sync                exchange memory, cleared
__device__ __forceinline__ int tr_at(int f) { return f + (f >> 5); }

template <int PC>  // 0: the single-workgroup frame
__global__ __launch_bounds__(TR_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void tridiag_kernel(
    double* __restrict__ G, int N, int Np, int B, int first, int last, int full, int mirror, double* __restrict__ dvec,
    double* __restrict__ evec, float* __restrict__ tauv, float* __restrict__ Vc, u64* __restrict__ sync, size_t sync_stride,
    u64* __restrict__ arrived, int patience, int xcds, int32_t* __restrict__ fail) {
  typedef TrShape<PC> S;
  constexpr int LI = S::LI, LK = S::LK, RT = S::RT, NS = S::NS, SR = S::LI / S::NS, E = S::E, MODE = S::MODE;
  constexpr int PR = S::PR, pc = S::PCC, R = S::R, C = S::C, F = S::F, P = S::P, OWN = S::OWN;
  static_assert(SR * R % 32 == 0, "a set of rows must be whole units of the padded vectors");
  static_assert(SR <= 16 && SR * NS == LI, "the rows of a set must fit the 16 lanes of a row");
  extern __shared__ __attribute__((aligned(16))) unsigned char tr_smem[];
  // The three vectors are read by rows (a wavefront's rows, R apart) and by columns (64 in a row): with a double skipped
  // after every 32 both are free of bank conflicts.
  constexpr int FX = F + F / 32;
  double* Va = reinterpret_cast<double*>(tr_smem);  // [FX] reflector of the even columns
  double* Vb = Va + FX;                              // [FX] of the odd ones
  double* Wv = Vb + FX;                              // [FX] w of the column before
  double* X = Wv + FX;                               // [FX] the column being reduced below its head (zero up to and with the head)
  double* csb = X + FX;                              // [8][OWN] column sums per wavefront
  double* rsb = csb + 8 * OWN;                       // [LI * 8] row sums
  double* colb = rsb + 8 * LI;                       // [LI * 8] this workgroup's rows of the next column
  double* red = colb + 8 * LI;                       // [4][8] partial sums of the block reductions
  double* one = red + 32;                            // [4] p at the reflector's first row, head of the next column; v and w of the column before at that row
  float* vblk = reinterpret_cast<float*>(one + 4);   // [LI * 8][16] the last sixteen reflectors, this workgroup's rows
  int* quit = reinterpret_cast<int*>(vblk + LI * 8 * 16);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // workgroup -> (image, member): in the four-workgroup frame the members of a group have ids that differ by multiples
  // of the number of XCDs (one XCD, one L2); larger groups are spread over all XCDs anyway
  int img, mem;
  if (MODE == 1) {
    const int t = (int)blockIdx.x / xcds;
    img = t / P * xcds + (int)blockIdx.x % xcds;
    mem = t % P;
  } else {
    img = blockIdx.x / P;
    mem = blockIdx.x % P;
  }
  if (img >= B) return;
  if (first > 0 && fail[img] != 0) return;  // (the phase before has not been)
  if (MODE != 0 && tid == 0) __hip_atomic_fetch_add(arrived + (size_t)img * sync_stride, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int a = mem % PR, b = mem / PR;
  double* A0 = G + (size_t)img * Np * Np;
  double* dout = dvec + (size_t)img * Np;
  double* eout = evec + (size_t)img * Np;
  float* tout = tauv + (size_t)img * Np;
  float* Vout = Vc + (size_t)img * Np * Np;
  u64* sy = sync + (size_t)img * sync_stride;
  const int base = N - F;                 // row of the matrix = row of the frame + base
  const int js = first - base, je = last - base;  // columns of the frame

  // ---- the workgroup's share of the matrix ---------------------------------------------------------------
  double A[LI][LK];
#pragma unroll
  for (int k = 0; k < LK; k++)
#pragma unroll
    for (int i = 0; i < LI; i++)
      if (i >= RT * k) {
        const int r = i * R + 8 * a + w + base, c = k * C + 64 * b + lane + base;
        double x = 0.0;
        if (r >= first && c >= first) x = full ? A0[(size_t)r * Np + c] : A0[(size_t)max(r, c) * Np + min(r, c)];
        A[i][k] = x;
      }
  for (int e = tid; e < 4 * FX; e += TR_THREADS) Va[e] = 0.0;  // the four vectors
  for (int e = tid; e < LI * 8 * 16; e += TR_THREADS) vblk[e] = 0.f;
  if (tid == 0) *quit = MODE != 0 && tr_stranded(arrived + (size_t)img * sync_stride, P, patience) ? 1 : 0;

  // this thread's elements of the vectors: frame rows F - 1 - tid - 512 u, so that the live ones stay in the low threads
  {
    double part = 0.0;
    __syncthreads();  // (X has been cleared)
    if (MODE != 0 && *quit) {  // uniform; nothing has been written
      if (tid == 0) __hip_atomic_store(fail + img, 1 + first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
#pragma unroll
    for (int u = 0; u < E; u++) {
      const int f = F - 1 - tid - TR_THREADS * u;
      if (f < js) continue;
      const double x = A0[(size_t)(f + base) * Np + first];
      if (f > js + 1) X[tr_at(f)] = x;
      if (f >= js + 2) part += x * x;
      if (f == js + 1) one[1] = x;
      if (f == js && mem == 0) dout[first] = x;
    }
    part = wave_sum_dpp(part);
    if (lane == 0) red[8 + w] = part;
  }
  __syncthreads();

  // place of a thread's element u in the vectors (tr_at of F - 1 - t - 512 u, as one address and a constant)
  auto own_at = [](int t, int u) { return tr_at(F - 1 - t - TR_THREADS * (E - 1)) + (TR_THREADS + TR_THREADS / 32) * (E - 1 - u); };
  bool bad = false;
  for (int j = js; j < min(je, F - 1); j++) {
    // (what hangs on the thread index is formed anew in every stage: kept across the sweeps, it would push the matrix out
    // of the registers)
    int tj = tid;
    fresh<MODE != 0>(tj);
    int lj = tj & 63;
    double* Vn = (j & 1) ? Vb : Va;        // this column's reflector
    const double* Vo = (j & 1) ? Va : Vb;  // the one before
    const int jr = j + base;               // column of the matrix
    // (with more than three elements a thread, the vectors are read again where they are wanted: no registers hold them)
    constexpr int K = E > 3 ? 1 : E;
    double p[E], col[E], v[K], vo[K], wo[K], dot[3] = {0.0, 0.0, 0.0};  // p^T v, w_o^T v, v_o^T v
    double beta, tau, scal;
    // Householder reflector that maps x[j+1:] onto beta e_1 (every workgroup and every wavefront for itself), and this
    // thread's elements of the vectors
    auto own_values = [&]() {
      const double xn2 = sum8(red + 8);
      const double alpha = one[1];
      beta = alpha;
      tau = scal = 0.0;
      if (xn2 > 0.0) {
        const double n2 = fma(alpha, alpha, xn2), rb = fast_rsq(n2);
        double nb = n2 * rb;
        nb = fma(0.5 * rb, fma(-nb, nb, n2), nb);          // |beta| = sqrt(n2)
        beta = -copysign(nb, alpha);
        tau = fma(fabs(alpha), rb, 1.0);                   // (beta - alpha) / beta
        scal = copysign(fast_rcp(fabs(alpha) + nb), alpha);  // 1 / (alpha - beta)
      }
#pragma unroll
      for (int u = 0; u < E; u++) {
        const int f = F - 1 - tj - TR_THREADS * u, g = own_at(tj, u);
        const int q = min(u, K - 1);
        v[q] = vo[q] = wo[q] = 0.0;
        if (f > j) {
          v[q] = f == j + 1 ? 1.0 : X[g] * scal;
          Vn[g] = v[q];
          if (b == 0 && (MODE == 0 || ((f >> 3) % PR) == a)) vblk[(f / R * 8 + (f & 7)) * 16 + (jr & 15)] = (float)v[q];
          if (MODE != 0) {
            vo[q] = Vo[g];
            wo[q] = Wv[g];
            dot[1] = fma(wo[q], v[q], dot[1]);
            dot[2] = fma(vo[q], v[q], dot[2]);
          }
        }
      }
      if (MODE != 0) {
        dot[1] = wave_sum_dpp(dot[1]);
        dot[2] = wave_sum_dpp(dot[2]);
      }
      if (tj == 0) {
        Vn[tr_at(j)] = 0.0;
        if (j > 0) Vn[tr_at(j - 1)] = 0.0;
        if (mem == 0) {
          eout[jr] = beta;
          tout[jr] = (float)tau;
        }
      }
    };
    // ---- A x, this workgroup's part -----------------------------------------------------------------------
    // The reflector is v = e_(j+1) + scal x with x the column below its head, so p = A v is the next column plus scal A x:
    // the sweep waits for no norm, and the chain of a square root, a reciprocal and the scaling runs while the parts are on
    // their way.  (With v in the sweep it stood before it: eight images of 2880 tokens 59.6 ms, now 55.6; four of 701 3.45,
    // now 3.39; one of 576 2.53 either way, where issuing the instructions is what takes the time.)
    // MODE 0: nothing is on its way, so the chain is issued in front of the sweep, which hides it (256 tokens: 602 us with v in
    // the sweep, 620 with the chain behind it, 590 so).  The update with the column before is applied in the same sweep.
    // Otherwise the product is formed with the matrix as it is and published, and the update follows while the other workgroups'
    // parts are on their way (below): p and the next column then still lack it, which costs two scalar products.
    if (MODE == 0) own_values();
    const int kmin = (j + 1) / C;
    const bool owner = MODE != 2 || (((j + 1) >> 6) % pc) == b;
    const int l0 = (j + 1) & 63;
    {
      const int fc0 = tr_at(64 * b + lj);
      // MODE 0 goes through its 32 rows in two sweeps (fewer sums in flight), the other modes through 18 in one
      constexpr int SW = MODE == 0 ? 2 : 1, RW = LI / SW;
      double cs[SW > 1 ? LK : 1];
      if (SW > 1)
#pragma unroll
        for (int k = 0; k < LK; k++) cs[SW > 1 ? k : 0] = 0.0;
      walk_up<0, SW>([&](auto sc) {
        constexpr int sw = decltype(sc)::value, i0 = sw * RW, i1 = i0 + RW;  // rows of the sweep
        if (sw + 1 < SW && RT * kmin >= i1) return;                         // every row of the sweep is done with
        constexpr int s0 = i0 / SR, s1 = (i1 - 1) / SR;                     // sets of rows it takes in
        // column values of the first live class; the next class's are on their way while one is worked on
        double vc = X[fc0 + kmin * (C + C / 32)], oc = 0.0, wc = 0.0;
        if (MODE == 0) { oc = Vo[fc0 + kmin * (C + C / 32)]; wc = Wv[fc0 + kmin * (C + C / 32)]; }
        const int gr0 = tr_at(min(lj & 15, SR - 1) * R + 8 * a + w);
        double vn[s1 - s0 + 1], vo[s1 - s0 + 1], wo[s1 - s0 + 1];
#pragma unroll
        for (int s = s0; s <= s1; s++) {
          const int g = gr0 + s * (SR * R + SR * R / 32);
          vn[s - s0] = X[g];
          if (MODE == 0) { vo[s - s0] = Vo[g]; wo[s - s0] = Wv[g]; }
        }
        constexpr int j0 = i0 > RT ? i0 : RT, NR = i1 - j0;  // rows with a row sum (those of the first diagonal block have none)
        double rs[NR];
#pragma unroll
        for (int q = 0; q < NR; q++) rs[q] = 0.0;
        walk_up<0, LK>([&](auto kc) {
          constexpr int k = decltype(kc)::value, r0 = RT * k > i0 ? RT * k : i0;
          if constexpr (r0 < i1) {
            if (k < kmin) return;
            constexpr int fn = (k + 1 < LK ? k + 1 : k) * (C + C / 32);
            const double xn = X[fc0 + fn], on = MODE == 0 ? Vo[fc0 + fn] : 0.0, wn = MODE == 0 ? Wv[fc0 + fn] : 0.0;
            double c0 = SW > 1 ? cs[SW > 1 ? k : 0] : 0.0, c1 = 0.0;
            if constexpr (MODE == 0) settle(vn[0], vo[0], wo[0]);
            else settle(vn[0], vn[1]);
            walk_up<r0, i1>([&](auto ic) {
              constexpr int i = decltype(ic)::value, s = i / SR - s0, q = i % SR;
              if constexpr (MODE == 0) {
                fmac_bcast_neg<q>(A[i][k], vo[s], wc);
                fmac_bcast_neg<q>(A[i][k], wo[s], oc);
              }
              if constexpr (i >= RT * (k + 1)) rs[i - j0] = fma(A[i][k], vc, rs[i - j0]);
              fmac_bcast<q>(i & 1 ? c1 : c0, vn[s], A[i][k]);
            });
            if constexpr (sw + 1 < SW) cs[SW > 1 ? k : 0] = c0 + c1;
            else csb[w * OWN + 64 * k + lj] = c0 + c1;
            if (k == kmin && owner && lj == l0) {
#pragma unroll
              for (int i = r0; i < i1; i++) colb[i * 8 + w] = A[i][k];
            }
            vc = xn;
            oc = on;
            wc = wn;
          }
        });
        // row sums (rows up to the end of the live diagonal block have none), the last eight alone where they are all
        int which;
        const int live = RT * (kmin + 1);
        if (NR == 16 && live < i1 - 8) {
          const double t = reduce_many<16>(rs, lj, &which);
          if ((lj & 3) == 0) rsb[(j0 + which) * 8 + w] = t;
        } else if (live < i1) {
          const double t = reduce_many<8>(rs + NR - 8, lj, &which);
          if ((lj & 7) == 0) rsb[(i1 - 8 + which) * 8 + w] = t;
        }
      });
    }
    __syncthreads();

    // ---- p in every workgroup -------------------------------------------------------------------------------
    const unsigned tag = (((j - js) >> 1) & 1) ^ 1;
    const int slot = (j - js) & 1;
    fresh<MODE != 0>(tj);
    lj = tj & 63;
    auto column_sum = [&](int o) {  // over the wavefronts
      const double* c = csb + o;
      return ((c[0] + c[OWN]) + (c[2 * OWN] + c[3 * OWN])) + ((c[4 * OWN] + c[5 * OWN]) + (c[6 * OWN] + c[7 * OWN]));
    };
    auto update = [&]() {  // A <- A - v w^T - w v^T with the column before
      fresh<true>(tj);
      lj = tj & 63;
      const int fc0 = tr_at(64 * b + lj);
      const int gr0 = tr_at(min(lj & 15, SR - 1) * R + 8 * a + w);
      double ro[NS], rw[NS];
      double oc = Vo[fc0 + kmin * (C + C / 32)], wc = Wv[fc0 + kmin * (C + C / 32)];
#pragma unroll
      for (int s = 0; s < NS; s++) {
        const int fr = gr0 + s * (SR * R + SR * R / 32);
        ro[s] = Vo[fr];
        rw[s] = Wv[fr];
      }
      walk_up<0, LK>([&](auto kc) {
        constexpr int k = decltype(kc)::value, fn = (k + 1 < LK ? k + 1 : k) * (C + C / 32);
        if (k < kmin) return;
        const double on = Vo[fc0 + fn], wn = Wv[fc0 + fn];
        settle(ro[0], ro[1], rw[0], rw[1]);
        walk_up<RT * k, LI>([&](auto ic) {
          constexpr int i = decltype(ic)::value, s = i / SR, q = i % SR;
          fmac_bcast_neg<q>(A[i][k], ro[s], wc);
          fmac_bcast_neg<q>(A[i][k], rw[s], oc);
        });
        oc = on;
        wc = wn;
      });
      fresh<true>(tj);
      lj = tj & 63;
    };
    if (MODE == 0) {
#pragma unroll
      for (int u = 0; u < E; u++) {
        const int f = F - 1 - tj - TR_THREADS * u;
        p[u] = col[u] = 0.0;
        if (f > j) {
          col[u] = colb[f];
          p[u] = fma(scal, column_sum(f) + ((f >> 3) >= RT * (kmin + 1) ? rsb[f] : 0.0), col[u]);
        }
      }
    } else if (MODE == 1) {
      u64* Y = sy + (size_t)slot * 5 * F;  // [4][F] partials, then [F] the next column
#pragma unroll
      for (int u = 0; u < E; u++) {
        const int f = F - 1 - tj - TR_THREADS * u, g = own_at(tj, u);
        if (f > j) {
          const bool mine = ((f >> 3) & 3) == a;  // a row of this workgroup
          const int o = (f >> 5) * 8 + (f & 7);
          const double s = column_sum(f) + (mine && (o >> 3) >= RT * (kmin + 1) ? rsb[o] : 0.0);
          publish(Y + (size_t)a * F + f, s, tag);
          if (mine) publish(Y + (size_t)4 * F + f, colb[o], tag);
        }
      }
      update();
      own_values();
#pragma unroll
      for (int u = 0; u < E; u++) {
        const int f = F - 1 - tj - TR_THREADS * u, g = own_at(tj, u);
        p[u] = col[u] = 0.0;
        if (f > j) {
          u64 y[5];
          for (int spin = 0;; spin++) {
            bool ok = true;
#pragma unroll
            for (int q = 0; q < 5; q++) y[q] = peek(Y + (size_t)q * F + f);
#pragma unroll
            for (int q = 0; q < 5; q++) ok &= (y[q] & 1) == tag;
            if (ok) break;
            if (tr_give_up(spin, fail + img)) { bad = true; break; }
          }
          col[u] = received(y[4]);
          p[u] = fma(scal, (received(y[0]) + received(y[1])) + (received(y[2]) + received(y[3])), col[u]);
        }
      }
    } else {
      u64* YC = sy + (size_t)slot * (5 * pc + 2) * F;  // [PR][F] column sums by row class
      u64* YR = YC + (size_t)PR * F;                   // [PC][F] row sums by column class
      u64* YN = YR + (size_t)pc * F;                   // [F] the next column
      u64* YT = YN + F;                                // [F] totals
      for (int o = tj; o < OWN; o += TR_THREADS) {
        const int f = (o >> 6) * C + 64 * b + (o & 63);
        if (f > j) publish(YC + (size_t)a * F + f, column_sum(o), tag);
      }
      if (tj < 8 * LI) {
        const int f = (tj >> 3) * R + 8 * a + (tj & 7);
        if (f > j) {
          publish(YR + (size_t)b * F + f, (tj >> 3) >= RT * (kmin + 1) ? rsb[tj] : 0.0, tag);
          if (owner) publish(YN + f, colb[tj], tag);
        }
      }
      update();
      // totals of this workgroup's share of its rows: four lanes per element
      constexpr int NQ = 5 * pc, PER = (NQ + 3) / 4;
      const int o = (tj >> 2) * pc + b;
      const int ft = (o >> 3) * R + 8 * a + (o & 7);
      if (o < 8 * LI && ft > j) {
        u64 y[PER];
        for (int spin = 0;; spin++) {
          bool ok = true;
#pragma unroll
          for (int q = 0; q < PER; q++) y[q] = peek(YC + (size_t)min(4 * q + (tj & 3), NQ - 1) * F + ft);  // (YR follows YC)
#pragma unroll
          for (int q = 0; q < PER; q++) ok &= (y[q] & 1) == tag;
          if (ok) break;
          if (tr_give_up(spin, fail + img)) { bad = true; break; }
        }
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < PER; q++) s += 4 * q + (tj & 3) < NQ ? received(y[q]) : 0.0;
        s += dpp_f64<0xB1>(s);  // the quad
        s += dpp_f64<0x4E>(s);
        if ((tj & 3) == 0) publish(YT + ft, s, tag);
      }
      auto collect = [&](const u64* src, double* dst) {
        for (int spin = 0;; spin++) {
          u64 y[E];
          bool ok = true;
#pragma unroll
          for (int u = 0; u < E; u++) {
            const int f = F - 1 - tj - TR_THREADS * u, g = own_at(tj, u);
            y[u] = f > j ? peek(src + f) : tag;
          }
#pragma unroll
          for (int u = 0; u < E; u++) {
            ok &= (y[u] & 1) == tag;
            dst[u] = received(y[u]);
          }
          if (ok) break;
          if (tr_give_up(spin, fail + img)) { bad = true; break; }
        }
      };
      collect(YN, col);  // (published together with the partials: it has arrived by the time the totals are)
      own_values();
      collect(YT, p);
#pragma unroll
      for (int u = 0; u < E; u++) p[u] = fma(scal, p[u], col[u]);
    }
    if (MODE != 0 && bad) *quit = 1;

    // ---- w = p - (tau/2) (p^T v) v with p <- tau p; the next column -------------------------------------------
#pragma unroll
    for (int u = 0; u < E; u++) {
      const int f = F - 1 - tj - TR_THREADS * u, g = own_at(tj, u);
      if (K == E) dot[0] = fma(p[u], v[min(u, K - 1)], dot[0]);  // (v is zero where f <= j)
      else if (f > j) dot[0] = fma(p[u], Vn[g], dot[0]);
      if (f == j + 1) {
        one[0] = p[u];
        if (MODE != 0) {
          one[2] = K == E ? vo[min(u, K - 1)] : Vo[g];
          one[3] = K == E ? wo[min(u, K - 1)] : Wv[g];
        }
      }
    }
    dot[0] = wave_sum_dpp(dot[0]);
    if (lj == 0) {
      red[w] = dot[0];
      if (MODE != 0) {
        red[16 + w] = dot[1];
        red[24 + w] = dot[2];
      }
    }
    __syncthreads();
    if (MODE != 0 && *quit) break;  // uniform
    double pv = sum8(red), p1 = one[0], sw = 0.0, sv = 0.0, vo1 = 0.0, wo1 = 0.0;
    if (MODE != 0) {  // the update with the column before that p lacks: p - v_o (w_o^T v) - w_o (v_o^T v)
      sw = sum8(red + 16);
      sv = sum8(red + 24);
      vo1 = one[2];
      wo1 = one[3];
      p1 -= vo1 * sw + wo1 * sv;
      pv -= 2.0 * sw * sv;
    }
    fresh<(E > 3)>(tj);
    lj = tj & 63;
    const double half = 0.5 * tau * tau * pv, w1 = tau * p1 - half;
    double part = 0.0;
#pragma unroll
    for (int u = 0; u < E; u++) {
      const int f = F - 1 - tj - TR_THREADS * u, g = own_at(tj, u);
      if (f > j) {
        double pf = p[u], xf = col[u];
        const double vf = K == E ? v[min(u, K - 1)] : Vn[g];
        if (MODE != 0) {
          const double vof = K == E ? vo[min(u, K - 1)] : Vo[g], wof = K == E ? wo[min(u, K - 1)] : Wv[g];
          pf -= vof * sw + wof * sv;
          xf -= vof * wo1 + wof * vo1;
        }
        const double wf = tau * pf - half * vf;
        Wv[g] = wf;
        const double x = xf - vf * w1 - wf;  // (the reflector's first entry is 1)
        X[g] = f <= j + 2 ? 0.0 : x;
        if (f >= j + 3) part = fma(x, x, part);
        if (f == j + 2) one[1] = x;
        if (f == j + 1 && mem == 0) dout[jr + 1] = x;
      }
    }
    if (tj == 0) Wv[tr_at(j)] = 0.0;
    part = wave_sum_dpp(part);
    if (lj == 0) red[8 + w] = part;
    // ---- sixteen reflectors complete: this workgroup's rows of them leave in 16-byte pieces ---------------------
    if ((jr & 15) == 15 || j == min(je, F - 1) - 1) {
      if (b == 0)
        for (int e = tj; e < LI * 8 * 4; e += TR_THREADS) {
          const int o = e >> 2, r = (o >> 3) * R + 8 * a + (o & 7) + base;
          if (r >= (jr & ~15) && r >= 0) {
            float4* src = reinterpret_cast<float4*>(vblk + o * 16 + 4 * (e & 3));
            *reinterpret_cast<float4*>(Vout + ((size_t)(jr >> 4) * Np + r) * 16 + 4 * (e & 3)) = *src;
            *src = float4{0.f, 0.f, 0.f, 0.f};
          }
        }
    }
    __syncthreads();
  }
  if (MODE != 0 && *quit) {
    if (tid == 0) __hip_atomic_store(fail + img, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  if (last == N) {
    if (tid == 0 && mem == 0) {
      eout[N - 1] = 0.0;
      tout[N - 1] = 0.f;
    }
    return;
  }
  // ---- the trailing matrix with the last column's update, for the next phase --------------------------------------
  const double* Vo = (je & 1) ? Va : Vb;
#pragma unroll
  for (int k = 0; k < LK; k++)
#pragma unroll
    for (int i = 0; i < LI; i++)
      if (i >= RT * k) {
        const int fr = i * R + 8 * a + w, fc = k * C + 64 * b + lane;
        if (fr >= je && fc >= je && fr >= fc) {
          const double y = A[i][k] - Vo[tr_at(fr)] * Wv[tr_at(fc)] - Wv[tr_at(fr)] * Vo[tr_at(fc)];
          A0[(size_t)(fr + base) * Np + fc + base] = y;
          if (mirror) A0[(size_t)(fc + base) * Np + fr + base] = y;
        }
      }
}

// ---- a stranded image -----------------------------------------------------------------------------------------
// The reduction by one workgroup with the matrix in memory: from the column the stranded phase would have begun with, one
// pass over the trailing matrix per column (the update with the column before and the product).  It waits for nobody.  Rare,
// so plain: 18 ms for an image of 576 tokens, 0.12 s for one of 1024, 2.6 s for one of 2880.
constexpr int AL_THREADS = 1024, AL_WAVES = AL_THREADS / 64;
static size_t alone_lds(int N) { return (size_t)(4 * N + 2 * AL_WAVES) * 8; }

__global__ __launch_bounds__(AL_THREADS) void tridiag_alone_kernel(double* __restrict__ G, int N, int Np, double* __restrict__ dvec,
                                                                   double* __restrict__ evec, float* __restrict__ tauv,
                                                                   float* __restrict__ Vc, int32_t* __restrict__ fail) {
  const int img = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (fail[img] <= 0) return;
  const int first = fail[img] - 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char al_smem[];
  double* v = reinterpret_cast<double*>(al_smem);  // [N] the reflector (x before it)
  double* p = v + N;                               // [N] A v
  double* vo = p + N;                              // [N] reflector and w of the column before
  double* wo = vo + N;
  double* red = wo + N;  // [2][AL_WAVES]
  double* A = G + (size_t)img * Np * Np;
  float* V = Vc + (size_t)img * Np * Np;
  // (a hand-over leaves the lower triangle)
  if (first > 0)
    for (int r = first + wave; r < N; r += AL_WAVES)
      for (int c = first + lane; c < r; c += 64) A[(size_t)c * Np + r] = A[(size_t)r * Np + c];
  for (int i = tid; i < N; i += AL_THREADS) vo[i] = wo[i] = 0.0;
  auto sum = [&](double x, int which) {
    x = wave_sum(x);
    if (lane == 0) red[which * AL_WAVES + wave] = x;
    __syncthreads();
    double t = 0.0;
    for (int q = 0; q < AL_WAVES; q++) t += red[which * AL_WAVES + q];
    return t;
  };
  __syncthreads();
  for (int j = first; j < N - 1; j++) {
    const double* row = A + (size_t)j * Np;
    double n2 = 0.0;
    for (int i = j + tid; i < N; i += AL_THREADS) {
      const double x = row[i] - vo[j] * wo[i] - wo[j] * vo[i];
      v[i] = x;
      if (i >= j + 2) n2 = fma(x, x, n2);
    }
    n2 = sum(n2, 0);
    const double alpha = v[j + 1];
    double beta = alpha, tau = 0.0, scal = 0.0;
    if (n2 > 0.0) {
      beta = -copysign(sqrt(fma(alpha, alpha, n2)), alpha);
      tau = (beta - alpha) / beta;
      scal = 1.0 / (alpha - beta);
    }
    if (tid == 0) {
      dvec[(size_t)img * Np + j] = v[j];
      evec[(size_t)img * Np + j] = beta;
      tauv[(size_t)img * Np + j] = (float)tau;
    }
    __syncthreads();
    float* out = V + (size_t)(j >> 4) * Np * 16 + (j & 15);
    const bool end = j == N - 2;  // (the places behind the last reflector are zero)
    for (int i = (j & ~15) + tid; i < N; i += AL_THREADS) {
      const double y = i <= j ? 0.0 : i == j + 1 ? 1.0 : v[i] * scal;
      v[i] = y;
      out[(size_t)i * 16] = (float)y;
      if (end)
        for (int c = (j & 15) + 1; c < 16; c++) out[(size_t)i * 16 + c - (j & 15)] = 0.f;
    }
    __syncthreads();
    double pv = 0.0;
    for (int i = j + 1 + wave; i < N; i += AL_WAVES) {
      double* a = A + (size_t)i * Np;
      const double vi = vo[i], wi = wo[i];
      double s = 0.0;
      for (int k = j + 1 + lane; k < N; k += 64) {
        const double x = a[k] - vi * wo[k] - wi * vo[k];
        a[k] = x;
        s = fma(x, v[k], s);
      }
      s = wave_sum(s);
      if (lane == 0) p[i] = s;
      pv = fma(s, v[i], pv);
    }
    pv = sum(lane == 0 ? pv : 0.0, 1);
    const double half = 0.5 * tau * tau * pv;
    for (int i = j + 1 + tid; i < N; i += AL_THREADS) {
      vo[i] = v[i];
      wo[i] = tau * p[i] - half * v[i];
    }
    __syncthreads();
  }
  if (tid == 0) {
    dvec[(size_t)img * Np + N - 1] = A[(size_t)(N - 1) * Np + N - 1] - 2.0 * vo[N - 1] * wo[N - 1];
    evec[(size_t)img * Np + N - 1] = 0.0;
    tauv[(size_t)img * Np + N - 1] = 0.f;
    fail[img] = 0;
  }
}

// ---- host ---------------------------------------------------------------------------------------------------
}  // namespace tc

// Polls before a group gives up waiting for its members (a quarter of a second; a round of the largest frame over the chip
// takes 25 ms).  A variable for the tests, no part of the interface: -n strands the groups from phase n - 1 of a call on.
constexpr int TR_PATIENCE = 1 << 18;
extern "C" __attribute__((visibility("default"))) int tc_group_patience = TR_PATIENCE;

namespace tc {
bool tridiag_fits(int N) { return N <= TR_FRAMES[TR_TRIANGLES - 1].F; }
int tridiag_most() { return TR_FRAMES[TR_TRIANGLES - 1].F; }
size_t tridiag_sync_bytes(int N) { return align256(tr_sync_words(N) * 8); }

static int compute_units() {  // of the current device
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  return n;
}

static bool tr_capturing(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone;
}

bool tridiag_allowed(int N, hipStream_t st) { return tr_runs(N, compute_units(), tr_capturing(st)); }

// Which launches are kept apart.  Groups that wait for members without a compute unit hold theirs, and an XCD deals out its
// workgroups by itself, in the order of their ids: launches side by side on several streams could strand each other's groups,
// where all 32 compute units of an XCD are held by workgroups that wait.  So what may wait there at once has to be
// less: of a launch whose groups lie on one XCD, the one group that is not complete, less a member; of a launch whose groups are
// spread over the XCDs, any of its workgroups.  A process has four hardware queues, so with three waiting in each, 19 more may.  An
// XCD has as many places, and a launch takes one for each workgroup above three (tr_places) on each XCD that it uses, behind the
// last launches there.  Groups of four take none and need no order.  A launch that could fill the XCD takes all: it is alone but for groups
// of four, and the image with the lowest number that is not complete finds its compute units, at most 22 of the 23 that are left.
// Which places and XCDs a launch takes depends on its shape and its stream only (the streams are counted as they come, which matters for
// nothing else).  Groups of sixteen have twelve places, and the other launches of their calls share the other seven: the groups of eight of
// one call run beside the groups of sixteen of another.  In calls without groups of sixteen each of four streams has places of its own.
// Launches with few images of groups on one XCD use as many XCDs as they have images, each stream its own.
// ms a call on two and on four streams, each with a hardware queue, when a launch took whole XCDs and now: 576 tokens, 2 images 0.62 and 0.62,
// 0.36 and 0.35; 8 images 0.73 and 0.74, 0.72 and 0.50; 701 tokens, 1 image 0.96 and 0.77, 0.96 and 0.41; 2 images 0.97 and 0.80, 0.96 and 0.47;
// 1152 tokens, 1 image 2.05 and 1.48, 2.04 and 1.37; 300 tokens, 8 images 0.35 and 0.34, 0.26 and 0.21.  (16 images of 576 tokens: 1.14 and 1.15, 1.05
// and 1.06; 32 images 1.81 and 1.81, 1.84 and 1.84: a call fills the device.  Two such calls side by side, 32 images on four streams: 1.96.)
// Captured launches cannot be kept apart; tr_runs and the frames allowed there bound what a stranded group holds.
// An event is known by the first place of the launch behind which it is recorded; every launch waits for the event it is going to
// record, so who waits for an event that has moved on waits for more.  (And for those of launches that take all, and of groups of sixteen
// where it needs a place of theirs: which events a call waits for does not depend on calls before it.)
constexpr int TR_STREAMS = 64, TR_ALL = 8 * TR_PLACES, TR_EVENTS = TR_ALL + 1;
struct TrDevice {
  hipEvent_t ev[TR_EVENTS];               // XCD x, place p: TR_PLACES x + p; TR_ALL: launches that take all
  unsigned char last[8 * TR_PLACES];      // event of the last launch there, and one (0: none)
  bool made;
  hipStream_t streams[TR_STREAMS];        // the last ones that were new
  unsigned seen;
};
static std::mutex tr_mx;
static TrDevice tr_devices[64];

TrTurn::TrTurn(int P, bool local, int images, bool sixteen, int xcds_, hipStream_t st_) : xcds(xcds_ < 8 ? xcds_ : 8), st(st_) {
  captured = tr_capturing(st);
  apart = tr_apart(P) && !captured;
  rc = TC_OK;
  if (!apart) return;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { apart = false; rc = TC_ERR_HIP; return; }
  tr_mx.lock();
  TrDevice& d = tr_devices[dev];
  for (int u = 0; u < TR_EVENTS && !d.made; u++)
    if (!d.ev[u] && hipEventCreateWithFlags(&d.ev[u], hipEventDisableTiming) != hipSuccess) rc = TC_ERR_HIP;
  if (rc == TC_OK) d.made = true;
  unsigned slot = 0;
  while (slot < d.seen && slot < TR_STREAMS && d.streams[slot] != st) slot++;
  if (slot == d.seen || slot == TR_STREAMS) {
    slot = d.seen++ % TR_STREAMS;
    d.streams[slot] = st;
  }
  places = tr_places(P, local, images, xcds);
  count = local && images < xcds ? images : xcds;
  first = count < xcds ? (int)(slot * count % xcds) : 0;
  from = tr_first_place(places, local, count == xcds, sixteen, slot);
  event = places == TR_PLACES && count == xcds ? TR_ALL : unit(0);
  bool waits[TR_EVENTS] = {};
  waits[event] = waits[TR_ALL] = true;
  if (from < TR_SIXTEEN) waits[unit(0) - from] = true;
  for (int i = 0; i < count * places; i++)
    if (d.last[unit(i)]) waits[d.last[unit(i)] - 1] = true;
  for (int e = 0; e < TR_EVENTS && rc == TC_OK; e++)
    if (waits[e] && hipStreamWaitEvent(st, d.ev[e], 0) != hipSuccess) rc = TC_ERR_HIP;
  if (rc != TC_OK) {
    (void)hipGetLastError();  // it is reported here, not by the next launch
    tr_mx.unlock();
    apart = false;
  }  // otherwise the lock is held until the event is recorded behind the launch
}

int TrTurn::done() {
  if (!apart) return TC_OK;
  TrDevice& d = tr_devices[dev];
  const bool ok = hipEventRecord(d.ev[event], st) == hipSuccess;
  if (!ok) {
    (void)hipStreamSynchronize(st);  // nobody can wait for this launch, so it is over
    (void)hipGetLastError();
  }
  for (int i = 0; i < count * places; i++) d.last[unit(i)] = (unsigned char)(event + 1);
  tr_mx.unlock();
  return ok ? TC_OK : TC_ERR_HIP;
}

int launch_columns(const Plan& pl, const TrPhase& ph, double* G, double* dvec, double* evec, float* tauv, float* Vc, u64* sync,
                   size_t stride, u64* arrived, int patience, bool sixteen, int xcds, int32_t* fail, hipStream_t st);  // tridiag_columns.hip

template <int PC>
static int tr_launch(const Plan& pl, const TrPhase& ph, int mirror, double* G, double* dvec, double* evec, float* tauv, float* Vc,
                     u64* sync, size_t stride, u64* arrived, int patience, bool sixteen, int xcds, int32_t* fail, hipStream_t st) {
  typedef TrShape<PC> S;
  if (S::LDS > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(tridiag_kernel<PC>),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS) != hipSuccess)
    return TC_ERR_HIP;
  const int grid = (S::MODE == 1 ? (pl.B + xcds - 1) / xcds * xcds : pl.B) * S::P;
  TrTurn turn(S::P, false, pl.B, sixteen, xcds, st);
  if (turn.rc != TC_OK) return turn.rc;
  TC_TIMED(PK_TRIDIAG, 0, st, (tridiag_kernel<PC><<<grid, TR_THREADS, S::LDS, st>>>(G, pl.N, pl.Np, pl.B, ph.first, ph.last, ph.first == 0, mirror, dvec, evec, tauv, Vc, sync, stride, arrived, patience, xcds, fail)));
  const int rc = check_launch(), rc2 = turn.done();
  return rc != TC_OK ? rc : rc2;
}

int launch_tridiag(const Plan& pl, double* G, double* dvec, double* evec, float* tauv, float* Vc, void* sync, size_t sync_bytes,
                   int32_t* fail, hipStream_t st) {
  const int cus = compute_units(), xcds = cus >= 64 ? cus / 32 : 1;  // (32 compute units each)
  TrPhase ph[TR_SIZES];
  size_t words;
  const int n = tr_phases(pl.N, pl.batch_call, cus, ph, &words, tr_capturing(st));
  if (n == 0) return TC_ERR_SHAPE;
  const size_t stride = sync_bytes / 8;
  if (words + TR_SIZES > stride) return TC_ERR_WORKSPACE;
  u64* sy = static_cast<u64*>(sync);
  const unsigned per = (unsigned)((words + TR_SIZES + 1023) / 1024);
  TC_TIMED(PK_TRIDIAG_UPDATE, 0, st, (tridiag_clear_kernel<<<dim3(per > 64 ? 64 : per, pl.B), 256, 0, st>>>(sy, stride, words + TR_SIZES, fail)));
  bool alone = false, sixteen = false;
  for (int i = 0; i < n; i++) sixteen |= tr_local(ph[i].size) && TR_FRAMES[ph[i].size].P == 16;
  for (int i = 0; i < n; i++) {
    const int set = tc_group_patience, patience = set >= 0 ? set : i + 1 >= -set ? -1 : TR_PATIENCE;
    const int mirror = i + 1 < n && ph[i + 1].size >= TR_TRIANGLES;  // whole columns want both triangles
    u64* words_of = sy + ph[i].off;
    u64* arrived = sy + words + i;
    int rc;
    alone |= TR_FRAMES[ph[i].size].P > 1;
#define TR_CASE(PC_) case PC_: rc = tr_launch<PC_>(pl, ph[i], mirror, G, dvec, evec, tauv, Vc, words_of, stride, arrived, patience, sixteen, xcds, fail, st); break;
    switch (ph[i].size) {
      TR_CASE(0) TR_CASE(1) TR_CASE(2) TR_CASE(3) TR_CASE(4) TR_CASE(5) TR_CASE(6)
      default: rc = launch_columns(pl, ph[i], G, dvec, evec, tauv, Vc, words_of, stride, arrived, patience, sixteen, xcds, fail, st);
    }
#undef TR_CASE
    if (rc != TC_OK) return rc;
  }
  if (alone) {
    const size_t shm = alone_lds(pl.N);
    if (shm > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(tridiag_alone_kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) != hipSuccess)
      return TC_ERR_HIP;
    TC_TIMED(PK_TRIDIAG_UPDATE, 1, st, (tridiag_alone_kernel<<<pl.B, AL_THREADS, shm, st>>>(G, pl.N, pl.Np, dvec, evec, tauv, Vc, fail)));
  }
  return check_launch();
}

}  // namespace tc
