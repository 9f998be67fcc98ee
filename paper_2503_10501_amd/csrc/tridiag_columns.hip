// Direct symmetric eigensolver, stage 1: reduction of the Gram matrix to tridiagonal form by groups of workgroups that hold whole
// columns of the trailing matrix in registers, and the last 128 columns by one workgroup.  (tridiag.hip holds the triangle: half the
// registers, and so half the compute units an image, but more than twice the time a column.  tr_phases chooses.)
//
// What bounds a column is latency: its steps hang on each other, and the arithmetic is small.  So this form has as few steps as it
// can, and each of them few instructions.
//   - A wavefront owns columns (both triangles are stored), a lane 64-cyclic rows of them: the product A x of a column is summed in
//     a lane and over the lanes of one wavefront, which publishes it.  No partial sums travel, and a reader finds one value per
//     row (the triangle: four, or totals in a second exchange).
//   - Four wavefronts, one per SIMD, hold the matrix and have the other registers of the chip's halves to themselves; the other four
//     have the vectors, one element in every 256 a thread, in registers from column to column.  While the first form A x, these add
//     up the norm and what else the reflector needs; while those update, these wait for the products.  (All eight doing both:
//     7000 clocks a column at 576 tokens, so 4000.)
//   - The next column is published a column ahead, when the update is done.
//   - The loops over columns are written out for every class of 64 (4 P) columns that is live, so no element's register is chosen at
//     run time and no branch parts the multiply-adds (with branches around rows that are done with: update 2800 clocks, so 900).
// As in tridiag.hip the product is formed with the matrix before the update of the column before and with the column below its
// head, unscaled: p = A v = (the next column) + scal A x, less what the update would have taken: v_o (w_o^T v) + w_o (v_o^T v).
// Column j, between two barriers A (a column ago) and B:
//   matrix:   A | A x, published | 0 | A <- A - v_o w_o^T - w_o v_o^T, next column published | B
//   vectors:  A | w_o, its sums with x | 0 | reflector v, waiting for A x, p, its product with v | B | next column
// Measured at 576 tokens on one XCD, clocks (2.4 GHz): A x 900 - 1300, reflector 900, waiting 600, p 500, next column 350: 3500 -
// 4000; with the loads and stores at the ends of a phase 1.7 us a column of the 576 frame and 1.3 of the 384 frame (the triangle 4.5 us, one
// workgroup for 256 tokens 2.3 us).  The whole reduction, ms, triangle and now: 64 tokens
// 0.097 and 0.051, 300 x 3 0.78 and 0.34, 576 x 1 2.05 and 0.80, x 16 2.07 and 0.83, x 64 2.2 and 1.8, 1152 x 1 5.4 and 2.1, 1499 x 2
// 7.4 and 3.2, 2880 x 1 17.5 and 11.5.
// Batches that fill the chip take the fewest workgroups an image that the registers allow: 320 rows by four, 448 by eight (100 and
// 98 elements a lane).  64 images of 576 tokens up to the last 128 rows, us: 192 columns of the triangle and 256 of 384 rows by
// eight in two rounds 1091 + 736; now 128 of the triangle, 64 of 448, 64 of 384 and 192 of 320 rows 774 + 282 + 243 + 325.
//
// Exchange: as in tridiag.hip, a value's lowest mantissa bit carries the parity of its use of the slot.  Products have two slots
// in turn: who publishes for column j + 2 has read all products of column j + 1, so every workgroup had published those and was
// done with column j.  (So every workgroup must have a live column: a frame leaves at least `least` rows.)  The next column, which
// is published one column earlier, has four.
#include "tc_internal.h"
#include "tridiag_device.h"
#include "tridiag_frames.h"

namespace tc {

typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

// Lower lanes: the sum of x in a lane and in the one 32 (16) further; upper lanes: that of y.
__device__ __forceinline__ double trade32(double x, double y) {
  const u32x2 lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
  const u32x2 hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double trade16(double x, double y) {
  const u32x2 lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
  const u32x2 hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// Sums of n values over the 64 lanes by recursive halving (fixed order); place_of_sum says which of them a lane returns.
template <int n>
__device__ __forceinline__ double reduce_lanes(double* x, int lane) {
  constexpr int h5 = (n + 1) / 2, h4 = (h5 + 1) / 2, h3 = (h4 + 1) / 2;
  static_assert(n <= 16, "");
#pragma unroll
  for (int u = 0; u < h5; u++) x[u] = trade32(x[u], u + h5 < n ? x[u + h5] : 0.0);
#pragma unroll
  for (int u = 0; u < h4; u++) x[u] = trade16(x[u], u + h4 < h5 ? x[u + h4] : 0.0);
  const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0;
  if constexpr (h4 == 1) x[0] += dpp_f64<0x128>(x[0]);  // row_ror:8, L <-> L^8
  else
#pragma unroll
    for (int u = 0; u < h3; u++) {
      const double y = u + h3 < h4 ? x[u + h3] : 0.0;
      x[u] = (b3 ? y : x[u]) + dpp_f64<0x128>(b3 ? x[u] : y);
    }
  double t;
  if constexpr (h3 == 1) t = x[0] + dpp_f64<0x141>(x[0]);  // row_half_mirror, L <-> 7-L
  else t = (b2 ? x[1] : x[0]) + dpp_f64<0x141>(b2 ? x[0] : x[1]);
  t += dpp_f64<0xB1>(t);  // quad_perm [1,0,3,2]
  t += dpp_f64<0x4E>(t);  // quad_perm [2,3,0,1]
  return t;
}

// Which of the n sums reduce_lanes leaves in a lane that is to publish it (-1: none).
template <int n>
__device__ __forceinline__ int place_of_sum(int lane) {
  constexpr int h5 = (n + 1) / 2, h4 = (h5 + 1) / 2, h3 = (h4 + 1) / 2;
  int at = 0;
  bool ok = (lane & 3) == 0;
  if (h3 > 1 && (lane & 4)) at = 1;
  if (h4 > 1 && (lane & 8)) { at += h3; ok &= at < h4; }
  if (lane & 16) { at += h4; ok &= at < h5; }
  if (lane & 32) { at += h5; ok &= at < n; }
  return ok ? at : -1;
}

// Sums over the 64 lanes on the matrix cores: in the 4x4x4 form lane i + 4 b + 16 k holds A[i][k] and B[k][i] of block b, lane
// j + 4 b + 16 i gets D[i][j].  A product with ones from the right adds the four rows of lanes, one with ones from the left
// what that has left in the quads; the four blocks are added through lane permutations.  Every lane returns the same bits.
__device__ __forceinline__ double lanes_of_blocks(double d) {
  double e = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, d, 0.0, 0, 0, 0);
  e += dpp_f64<0x124>(e);  // row_ror:4
  e += dpp_f64<0x128>(e);  // row_ror:8
  return e;
}
__device__ __forceinline__ double sum_lanes(double x) { return lanes_of_blocks(__builtin_amdgcn_mfma_f64_4x4x4f64(x, 1.0, 0.0, 0, 0, 0)); }
// Lane L returns the sum of x, y, z (L % 4 = 0, 1, 2; 0 elsewhere).
__device__ __forceinline__ double sum_lanes(double x, double y, double z, int lane) {
  const int q = lane & 3;
  double d = __builtin_amdgcn_mfma_f64_4x4x4f64(x, q == 0 ? 1.0 : 0.0, 0.0, 0, 0, 0);
  d = __builtin_amdgcn_mfma_f64_4x4x4f64(y, q == 1 ? 1.0 : 0.0, d, 0, 0, 0);
  d = __builtin_amdgcn_mfma_f64_4x4x4f64(z, q == 2 ? 1.0 : 0.0, d, 0, 0, 0);
  return lanes_of_blocks(d);
}

// A store that the other members can poll.  Members on one XCD (known from XCC_ID, not assumed) share its L2: the store ends there and
// the polls find it.  Elsewhere it has to go on to memory (one way from store to poll, measured with 64 lanes: 800 clocks and 1300 to
// 1700).  The near store stands on the machine, not on the memory model, which promises a store of workgroup scope to its own workgroup
// only: L1 writes through, so global_store with sc0 and without sc1 ends in the L2 of the XCD, and a load with sc1 passes L1 by.  The value
// carries its own tag, so nothing else has to be ordered with it.
__device__ __forceinline__ void publish_to(bool near, u64* p, double v, unsigned tag) {
  const u64 y = tagged(v, tag);
  if (near) __hip_atomic_store(p, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(p, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class S>
__global__ __launch_bounds__(TR_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void tridiag_columns_kernel(
    double* __restrict__ G, int N, int Np, int B, int first, int last, double* __restrict__ dvec, double* __restrict__ evec,
    float* __restrict__ tauv, float* __restrict__ Vc, u64* __restrict__ sync, size_t sync_stride, u64* __restrict__ arrived,
    int patience, int xcds, int shift, int32_t* __restrict__ fail) {
  constexpr int LI = S::LI, LK = S::LK, P = S::P, F = S::F, CW = S::CW, E = S::E, RO = S::RO;
  constexpr int OT = 256, FP = S::FP, OFF = FP - F;   // the vectors have room for elements that no row belongs to
  extern __shared__ __attribute__((aligned(16))) unsigned char tc_smem[];
  double* Va = reinterpret_cast<double*>(tc_smem);  // [FP] reflector of the even columns
  double* Vb = Va + FP;                             // [FP] of the odd ones
  double* Wv = Vb + FP;                             // [FP] w of the column before
  double* X = Wv + FP;                              // [FP] the column being reduced: diagonal, head and what is below
  double* PV = X + FP;                              // [FP] tau p
  double* red = PV + FP;                            // [4][4] sums x x, w x, v x of a wavefront; [4] tau p v
  double* ebuf = red + 20;                          // [16] results until they leave, by column
  double* dbuf = ebuf + 16;                         // [16]
  float* tbuf = reinterpret_cast<float*>(dbuf + 16);  // [16]
  float* vblk = tbuf + 16;                          // [RO][16] the last sixteen reflectors, this workgroup's rows
  int* quit = reinterpret_cast<int*>(vblk + RO * 16);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int img, m;
  if (S::LOCAL && shift >= 0) {  // the members on one XCD, the first image on the one with number `shift`
    const int t = (int)blockIdx.x / xcds;
    img = t / P * xcds + ((int)blockIdx.x + xcds - shift) % xcds;
    m = t % P;
  } else {
    img = blockIdx.x / P;
    m = blockIdx.x % P;
  }
  if (img >= B) return;
  if (first > 0 && fail[img] != 0) return;  // (the phase before has not been)
  // the members count themselves in, in all (the lowest eight bits) and by XCD (six bits each)
  const unsigned xcc = __builtin_amdgcn_s_getreg(20 | 3 << 11) & 7;  // XCC_ID
  if (tid == 0)
    __hip_atomic_fetch_add(arrived + (size_t)img * sync_stride, 1ull + (1ull << (8 + 6 * xcc)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  double* A0 = G + (size_t)img * Np * Np;
  u64* Y = sync + (size_t)img * sync_stride;  // [2][F] products
  u64* Cn = Y + 2 * F;                        // [4][F] next columns
  const int base = N - F;                     // row of the matrix = row of the frame + base
  const int js = first - base;  // columns of the frame, from here
  int je = last - base;         // ... to here

  for (int e = tid; e < 5 * FP + 20; e += TR_THREADS) Va[e] = 0.0;  // the vectors and the sums
  if (tid == 0) {
    u64 n = 0;
    quit[0] = tr_stranded(arrived + (size_t)img * sync_stride, P, patience, 255, &n) ? 1 : 0;
    quit[1] = S::LOCAL && ((n >> (8 + 6 * xcc)) & 63) == P ? 1 : 0;
  }
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(*quit)) {  // uniform; nothing has been written
    if (tid == 0) __hip_atomic_store(fail + img, 1 + first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  const bool near = __builtin_amdgcn_readfirstlane(quit[1]) != 0;
  for (int f = js + tid; f < F; f += TR_THREADS) X[OFF + f] = A0[(size_t)first * Np + f + base];

  if (w >= 4) {  // ==== a wavefront of the matrix =========================================================================
    const int cw = m * 4 + w - 4;  // column of class k: cw + k CW
    double A[LI][LK];
#pragma unroll
    for (int k = 0; k < LK; k++)
#pragma unroll
      for (int i = 0; i < LI; i++) {
        const int r = i * 64 + lane + base, c = k * CW + cw + base;
        A[i][k] = r >= first && c >= first ? A0[(size_t)c * Np + r] : 0.0;
      }
    // The wavefront that owns column c, which is of class K or the one after that, publishes it for the column before that (its rows
    // from c on).
    auto publish_column = [&](auto kc, int c) __attribute__((always_inline)) {
      constexpr int K = decltype(kc)::value;
      const int k = c / CW;
      if (c - k * CW != cw) return;
      const int n = c - 1 - js;  // use of the slots
      const unsigned tag = ((n >> 2) & 1) ^ 1;
      u64* dst = Cn + (size_t)(n & 3) * F;
      int l = lane;
      fresh<true>(l);
#pragma unroll
      for (int i = 0; i < LI; i++)
        if (64 * i + 63 >= c) {
          const double y = K + 1 < LK && k > K ? A[i][K + 1 < LK ? K + 1 : K] : A[i][K];
          if (64 * i + l >= c) publish_to(near, dst + 64 * i + l, y, tag);
        }
    };
    walk_up<0, LK>([&](auto kc) __attribute__((always_inline)) {
      if ((js + 1) / CW == decltype(kc)::value) publish_column(kc, js + 1);
    });
    __builtin_amdgcn_s_waitcnt(0);  // (the matrix is there: no wait for it inside the loop)
    __syncthreads();
    int j = js;
    walk_up<0, LK>([&](auto kc) __attribute__((always_inline)) {
      // columns whose product needs the classes from K on
      constexpr int K = decltype(kc)::value, n = LK - K, i0 = K * CW / 64, end = (K + 1) * CW - 1;
      if (j >= end) return;
      // Sums of M columns at a time: more take registers that the matrix needs.  ypl: byte offsets of the products that this lane
      // publishes (0: none)
      constexpr int M = n > 14 ? (n + 1) / 2 : n, PARTS = (n + M - 1) / M;
      int ypl[PARTS];
#pragma unroll
      for (int h = 0; h < PARTS; h++) {
        const int q = place_of_sum<M>(lane);
        ypl[h] = q < 0 || h * M + q >= n ? 0 : 8 * ((K + h * M + q) * CW + cw);
      }
      for (; j < min(je, end); j++) {
        int lj = lane;
        fresh<true>(lj);
        const double* Vo = (j & 1) ? Va : Vb;  // reflector of the column before
        const unsigned tag = (((j - js) >> 1) & 1) ^ 1;
        u64* Yj = Y + (size_t)((j - js) & 1) * F;
        // ---- A x, this wavefront's columns --------------------------------------------------------------------
        {
          constexpr int NA = n > 2 || LI - i0 < 2 ? 1 : 2;  // (few columns: two chains each)
          // (rows in turns: what is read ahead is bounded, so that the matrix stays in the registers; the 1920 and 2112 frames
          // have 2 and 40 registers too few: the compiler puts one store to scratch into the kernel, and twenty)
          constexpr int T = LI <= 12 ? LI : 6;
          auto below = [&](int i) {  // (zero up to and with the head)
            const double x = X[OFF + 64 * i + lj];
            return 64 * i <= end && 64 * i + lj <= j + 1 ? 0.0 : x;
          };
          double xr[2][T];
#pragma unroll
          for (int r = 0; r < T; r++)
            if (i0 + r < LI) xr[0][r] = below(i0 + r);
          walk_up<0, PARTS>([&](auto hc) __attribute__((always_inline)) {
            constexpr int q0 = decltype(hc)::value * M, m = n - q0 < M ? n - q0 : M;
            static_assert(PARTS == 1 || T >= LI, "the rows are there for every part");
            double acc[NA][M];
#pragma unroll
            for (int i = i0; i < LI; i++) {
              const int r = (i - i0) % T, b = (i - i0) / T % 2;
              if (r == 0) {
#pragma unroll
                for (int s = 0; s < T; s++)
                  if (i + T + s < LI) xr[1 - b][s] = below(i + T + s);
                if (T < LI - i0) __builtin_amdgcn_sched_barrier(0);
              }
#pragma unroll
              for (int q = 0; q < m; q++) {
                double& a = acc[(i - i0) % NA][q];
                a = i - i0 < NA ? A[i][K + q0 + q] * xr[b][r] : fma(A[i][K + q0 + q], xr[b][r], a);
              }
            }
            if (NA == 2)
#pragma unroll
              for (int q = 0; q < m; q++) acc[0][q] += acc[NA - 1][q];
#pragma unroll
            for (int q = m; q < M; q++) acc[0][q] = 0.0;
            const double t = reduce_lanes<M>(acc[0], lj);
            const int y = ypl[decltype(hc)::value];
            if (y > 8 * j) publish_to(near, reinterpret_cast<u64*>(reinterpret_cast<char*>(Yj) + (unsigned)y), t, tag);
          });
        }
        __syncthreads();
        // ---- the update with the column before ------------------------------------------------------------------
        fresh<true>(lj);
        // the columns' values: lane k reads those of class k, which then come from scalar registers
        const int cl = OFF + min(lj, LK - 1) * CW + cw;
        const double vcl = -Vo[cl], wcl = -Wv[cl];
        constexpr int T = 3;  // rows read ahead
#pragma unroll
        for (int q0 = 0; q0 < n; q0 += M) {  // (a column's values are four scalar registers)
          double vc[M], wc[M], vr[2][T], wr[2][T];
#pragma unroll
          for (int r = 0; r < T; r++)
            if (i0 + r < LI) {
              vr[0][r] = Vo[OFF + 64 * (i0 + r) + lj];
              wr[0][r] = Wv[OFF + 64 * (i0 + r) + lj];
            }
#pragma unroll
          for (int k = 0; k < M; k++) {
            vc[k] = readlane_f64(vcl, K + q0 + k);
            wc[k] = readlane_f64(wcl, K + q0 + k);
          }
#pragma unroll
          for (int i = i0; i < LI; i++) {
            const int r = (i - i0) % T, b = (i - i0) / T % 2;
            if (r == 0) {
#pragma unroll
              for (int s = 0; s < T; s++)
                if (i + T + s < LI) {
                  vr[1 - b][s] = Vo[OFF + 64 * (i + T + s) + lj];
                  wr[1 - b][s] = Wv[OFF + 64 * (i + T + s) + lj];
                }
              if (T < LI - i0) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int q = 0; q < M; q++)
              if (q0 + q < n) A[i][K + q0 + q] = fma(wr[b][r], vc[q], fma(vr[b][r], wc[q], A[i][K + q0 + q]));
          }
          if (M < n) __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = i0; i < LI; i++)
#pragma unroll
          for (int q = 0; q < n; q++) asm volatile("" : "+v"(A[i][K + q]));  // (nothing of this is put off until behind the barriers)
        if (j + 1 < je) publish_column(kc, j + 2);
        __syncthreads();
        const int leave = *quit;  // (written before the barrier above only)
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(leave)) je = 0;  // (ends the loops)
      }
    });
    if (je == 0) return;  // (the flag is up)
    __syncthreads();
    // ---- the trailing matrix with the last column's update, for the next phase --------------------------------------
    const double* Vo = (je & 1) ? Va : Vb;
#pragma unroll
    for (int k = 0; k < LK; k++)
#pragma unroll
      for (int i = 0; i < LI; i++) {
        const int fr = i * 64 + lane, fc = k * CW + cw;
        if (fr >= je && fc >= je)
          A0[(size_t)(fc + base) * Np + fr + base] = fma(-Wv[OFF + fr], Vo[OFF + fc], fma(-Vo[OFF + fr], Wv[OFF + fc], A[i][k]));
      }
  } else {  // ==== a wavefront of the vectors ==============================================================================
    // This thread's elements: rows F - 1 - tid - 256 u, so that the live ones stay in the low threads.  Elements of rows that are
    // done with (and of no row) go along: the column is zero there.
    auto at = [](int t, int u) { return OT - 1 - t + OT * (E - 1 - u); };
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    double x[E], v[E], wv[E];  // the column below its head; reflector and w of the column before
#pragma unroll
    for (int u = 0; u < E; u++) {
      x[u] = X[at(tid, u)];
      v[u] = wv[u] = 0.0;
    }
    double half = 0.0;
    bool was = false;
    // Reflectors and results leave sixteen columns at a time, a row's by one lane of the last of these wavefronts, while the
    // others form A x: those of column j - 1 when column j is under way.
    auto hand_out = [&](int j, int l) {
      const int jr = j - 1 + base;
      const double* Vo = (j & 1) ? Va : Vb;
      if (w == 3)
#pragma unroll
        for (int s = 0; s < RO; s += 64) {
          const int q = l + s, f = m * RO + q, r = f + base;
          if (q >= RO) break;
          const double y = Vo[OFF + min(f, F - 1)];
          vblk[q * 16 + (jr & 15)] = f >= j ? (float)y : 0.f;
          if ((jr & 15) == 15 && r >= (jr & ~15) && f < F) {
            float4* dst = reinterpret_cast<float4*>(Vc + (size_t)img * Np * Np + ((size_t)(jr >> 4) * Np + r) * 16);
#pragma unroll
            for (int u = 0; u < 4; u++) dst[u] = reinterpret_cast<const float4*>(vblk + q * 16)[u];
          }
        }
      if (w == 2 && m == 0 && (jr & 15) == 15 && l < 16) {
        const int c = (jr & ~15) + l;
        dvec[(size_t)img * Np + c] = dbuf[l];
        evec[(size_t)img * Np + c] = ebuf[l];
        tauv[(size_t)img * Np + c] = tbuf[l];
      }
    };
    for (int j = js; j < je; j++) {
      int tj = tid;
      fresh<true>(tj);
      const int lj = tj & 63;
      double* Vn = (j & 1) ? Vb : Va;        // this column's reflector
      const double* Vo = (j & 1) ? Va : Vb;  // the one before
      const int jr = j + base;
      const unsigned tag = (((j - js) >> 1) & 1) ^ 1, ctag = (((j - js) >> 2) & 1) ^ 1;
      const u64* Yj = Y + (size_t)((j - js) & 1) * F;
      const u64* Cj = Cn + (size_t)((j - js) & 3) * F;
      const bool live = F - 1 - 64 * w > j;  // uniform in the wavefront
      double g[E], tau = 0.0, alpha = 0.0, vo1 = 0.0, wo1 = 0.0;
      // w of the column before: w = tau p - half v with half = (tau/2) (tau p)^T v
      if (was)
#pragma unroll
        for (int u = 0; u < E; u++) {
          wv[u] = fma(-half, v[u], wv[u]);
          Wv[at(tj, u)] = wv[u];
        }
      was = live;
      if (live) {
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int u = 0; u < E; u++) {
          x[u] = at(tj, u) - OFF > j + 1 ? x[u] : 0.0;
          s0 = fma(x[u], x[u], s0);
          s1 = fma(x[u], wv[u], s1);
          s2 = fma(x[u], v[u], s2);
        }
        const double t = sum_lanes(s0, s1, s2, lj);
        if (lj < 4) red[4 * w + lj] = t;
      } else if (lj < 5) {
        red[lj < 4 ? 4 * w + lj : 16 + w] = 0.0;
      }
      if (j > js) hand_out(j, lj);
      __syncthreads();
      if (live) {
        double t = red[lj & 15];  // lane L: value L % 4 of wavefront L / 4
        alpha = X[OFF + j + 1];
        vo1 = Vo[OFF + j + 1];
        wo1 = Wv[OFF + j + 1];
        t += dpp_f64<0x124>(t);  // row_ror:4
        t += dpp_f64<0x128>(t);  // row_ror:8
        const double xx = readlane_f64(t, 0), wx = readlane_f64(t, 1), vx = readlane_f64(t, 2);
        // Householder reflector that maps x[j+1:] onto beta e_1 (every wavefront for itself)
        double beta = alpha, scal = 0.0;
        if (xx > 0.0) {
          const double n2 = fma(alpha, alpha, xx), rb = fast_rsq(n2);
          double nb = n2 * rb;
          nb = fma(0.5 * rb, fma(-nb, nb, n2), nb);            // |beta| = sqrt(n2)
          beta = -copysign(nb, alpha);
          tau = fma(fabs(alpha), rb, 1.0);                     // (beta - alpha) / beta
          scal = copysign(fast_rcp(fabs(alpha) + nb), alpha);  // 1 / (alpha - beta)
        }
        const double sw = fma(scal, wx, wo1), sv = fma(scal, vx, vo1);  // w_o^T v, v_o^T v
        double pc[E], cx[E];  // what the product and the next column lack of the update with the column before
#pragma unroll
        for (int u = 0; u < E; u++) {
          pc[u] = fma(v[u], sw, wv[u] * sv);
          cx[u] = fma(v[u], wo1, wv[u] * vo1);
          const double y = x[u] * scal;
          v[u] = at(tj, u) - OFF == j + 1 ? 1.0 : y;
          Vn[at(tj, u)] = v[u];
        }
        if (tj == 0) {
          dbuf[jr & 15] = X[OFF + j];
          ebuf[jr & 15] = beta;
          tbuf[jr & 15] = (float)tau;
        }
        // ---- p = A v = (the next column) + scal A x -----------------------------------------------------------
        u64 yq[E], cq[E];
        auto ask = [&]() {
#pragma unroll
          for (int u = 0; u < E; u++) {
            const int f = at(tj, u) - OFF;
            const unsigned o = 8u * (unsigned)(f > j ? f : F - 1);
            yq[u] = peek(reinterpret_cast<const u64*>(reinterpret_cast<const char*>(Yj) + o));
            cq[u] = peek(reinterpret_cast<const u64*>(reinterpret_cast<const char*>(Cj) + o));
          }
        };
        // (Not asked earlier: a question that overtakes the answer on its way to memory takes twice as long.)
        ask();
        for (int spin = 0;; spin++) {
          unsigned wrong = 0;
#pragma unroll
          for (int u = 0; u < E; u++) wrong |= ((unsigned)yq[u] ^ tag) | ((unsigned)cq[u] ^ ctag);
          if (!__any(wrong & 1)) break;
          if (tr_give_up(spin, fail + img)) {
            *quit = 1;
            __hip_atomic_store(fail + img, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
          }
          ask();
        }
        double dot = 0.0;
#pragma unroll
        for (int u = 0; u < E; u++) {
          const double col = received(cq[u]);
          const double tp = tau * fma(scal, received(yq[u]), col - pc[u]);
          dot = fma(tp, v[u], dot);  // (v is zero up to row j)
          PV[at(tj, u)] = tp;
          wv[u] = tp;
          g[u] = (col - cx[u]) - tp;
        }
        dot = sum_lanes(dot);
        if (lj == 0) red[16 + w] = dot;
      }
      __syncthreads();
      const int leave = *quit;
      // ---- the next column: x - v w_1 - w -----------------------------------------------------------------------
      if (live) {
        const double pv = (red[16] + red[17]) + (red[18] + red[19]);
        const double c = fma(-tau, pv, PV[OFF + j + 1]);  // (the reflector's first entry is 1: w_1 - half)
#pragma unroll
        for (int u = 0; u < E; u++) {
          x[u] = fma(-v[u], c, g[u]);
          X[at(tj, u)] = x[u];
        }
        half = 0.5 * tau * pv;
      }
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(leave)) je = 0;  // (ends the loop)
    }
    if (je == 0) return;  // (the flag is up)
    hand_out(je, lane);
    if (was)
#pragma unroll
      for (int u = 0; u < E; u++) Wv[at(tid, u)] = fma(-half, v[u], wv[u]);
    __syncthreads();
  }
}

// What lanes of this wavefront have written to LDS before is there for its other lanes after (no instruction: it keeps the compiler
// from moving accesses across).
__device__ __forceinline__ void between_lanes() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---- the last columns -------------------------------------------------------------------------------------------
// Up to 128 rows by one workgroup of four wavefronts, one per SIMD: wavefront w owns the columns 16 k + 4 w + (lane & 3), a lane of
// them the rows 16 i + (lane >> 2).  The vectors' part is done by every wavefront for itself, bit for bit the same, with copies of
// the vectors of its own, so that a column has one barrier: where the products of the others come in.
__global__ __launch_bounds__(256) void tridiag_last_kernel(double* __restrict__ G, int N, int Np, int first, double* __restrict__ dvec,
                                                           double* __restrict__ evec, float* __restrict__ tauv,
                                                           float* __restrict__ Vc, const int32_t* __restrict__ fail) {
  constexpr int F = TR_LAST, L = 8;
  __shared__ double Y[2][F], Cn[2][F];           // products and next column, two columns in turn
  __shared__ double Xs[4][F], Vs[4][F], Ws[4][F];  // column below its head, reflector and w of the column before: one set for each wavefront
  __shared__ __attribute__((aligned(16))) float vblk[F][20];  // (sixteen and room: fewer rows meet in a bank)
  __shared__ double db[32], eb[16];
  __shared__ float tb[16];
  const int img = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (first > 0 && fail[img] != 0) return;  // (the phase before has not been)
  double* A0 = G + (size_t)img * Np * Np;
  const int base = N - F, js = first - base, rg = lane >> 2, c4 = 4 * w + (lane & 3);
  double* X = Xs[w];
  double* V = Vs[w];
  double* W = Ws[w];
  double A[L][L];
#pragma unroll
  for (int k = 0; k < L; k++)
#pragma unroll
    for (int i = 0; i < L; i++) {
      const int r = 16 * i + rg + base, c = 16 * k + c4 + base;
      A[i][k] = r >= first && c >= first ? A0[(size_t)r * Np + c] : 0.0;
    }
  for (int e = tid; e < F * 20; e += 256) (&vblk[0][0])[e] = 0.f;
  for (int f = tid; f < F; f += 256) Y[0][f] = Y[1][f] = Cn[0][f] = Cn[1][f] = 0.0;
  // a lane's rows of the vectors: lane and lane + 64
  double x[2], v[2] = {0.0, 0.0}, wv[2] = {0.0, 0.0};
#pragma unroll
  for (int u = 0; u < 2; u++) {
    const int f = lane + 64 * u;
    const double y = f >= js ? A0[(size_t)first * Np + f + base] : 0.0;
    x[u] = y;
    X[f] = f > js + 1 ? y : 0.0;
    V[f] = W[f] = 0.0;
  }
  auto element = [&](const double* y, int f) { return f < 64 ? readlane_f64(y[0], f) : readlane_f64(y[1], f - 64); };
  double alpha = element(x, min(js + 1, F - 1));
  if (tid == 3 * 64) db[first & 31] = element(x, js);
#pragma unroll
  for (int u = 0; u < 2; u++) x[u] = lane + 64 * u > js + 1 ? x[u] : 0.0;
  __syncthreads();

  int j = js;
  walk_up<0, L>([&](auto kc) __attribute__((always_inline)) {
    constexpr int K = decltype(kc)::value, n = L - K, U0 = K < 4 ? 0 : 1;  // rows below 64 are done with from class 4 on
    for (; j < min(F - 1, 16 * K + 15); j++) {
      const int jr = j + base, par = j & 1;
      int lj = lane;
      fresh<true>(lj);
      const int rj = lj >> 2, cj = 4 * w + (lj & 3);
      // ---- the update with the column before, and A x ------------------------------------------------------------
      double acc[n];
      {
        double xr[n], vr[n], wr[n];
#pragma unroll
        for (int i = 0; i < n; i++) {
          xr[i] = X[16 * (K + i) + rj];
          vr[i] = V[16 * (K + i) + rj];
          wr[i] = W[16 * (K + i) + rj];
        }
#pragma unroll
        for (int q = 0; q < n; q++) {
          const double vc = -V[16 * (K + q) + cj], wc = -W[16 * (K + q) + cj];
#pragma unroll
          for (int i = 0; i < n; i++) {
            double& a = A[K + i][K + q];
            a = fma(wr[i], vc, fma(vr[i], wc, a));
            acc[q] = i == 0 ? a * xr[i] : fma(a, xr[i], acc[q]);
          }
        }
      }
      if (cj == ((j + 1) & 15))  // the next column
#pragma unroll
        for (int i = 0; i < n; i++) Cn[par][16 * (K + i) + rj] = A[K + i][K];
      {
        constexpr int h5 = (n + 1) / 2, h4 = (h5 + 1) / 2;
#pragma unroll
        for (int u = 0; u < h5; u++) acc[u] = trade32(acc[u], u + h5 < n ? acc[u + h5 < n ? u + h5 : 0] : 0.0);
#pragma unroll
        for (int u = 0; u < h4; u++) acc[u] = trade16(acc[u], u + h4 < h5 ? acc[u + h4 < h5 ? u + h4 : 0] : 0.0);
#pragma unroll
        for (int u = 0; u < h4; u++) {
          acc[u] += dpp_f64<0x128>(acc[u]);  // row_ror:8
          acc[u] += dpp_f64<0x124>(acc[u]);  // row_ror:4
          const int p = u + ((lj & 16) ? h4 : 0), q = p + ((lj & 32) ? h5 : 0);
          if ((lj & 12) == 0 && p < h5 && q < n) Y[par][16 * (K + q) + cj] = acc[u];
        }
      }
      // ---- Householder reflector that maps x[j+1:] onto beta e_1 ---------------------------------------------------
      const double xx = sum_lanes(U0 == 0 ? fma(x[0], x[0], x[1] * x[1]) : x[1] * x[1]);
      double beta = alpha, tau = 0.0, scal = 0.0;
      if (__builtin_amdgcn_readfirstlane(xx > 0.0)) {
        const double n2 = fma(alpha, alpha, xx), rb = fast_rsq(n2);
        double nb = n2 * rb;
        nb = fma(0.5 * rb, fma(-nb, nb, n2), nb);            // |beta| = sqrt(n2)
        beta = -copysign(nb, alpha);
        tau = fma(fabs(alpha), rb, 1.0);                     // (beta - alpha) / beta
        scal = copysign(fast_rcp(fabs(alpha) + nb), alpha);  // 1 / (alpha - beta)
      }
      __syncthreads();
      // ---- p = A v = (the next column) + scal A x, w = tau p - half v, the next column x - v w_1 - w -----------------
      double tp[2], col[2], dot = 0.0;
#pragma unroll
      for (int u = U0; u < 2; u++) {
        const int f = lj + 64 * u;
        col[u] = Cn[par][f];
        v[u] = f == j + 1 ? 1.0 : x[u] * scal;
        tp[u] = tau * fma(scal, Y[par][f], col[u]);
        dot = fma(tp[u], v[u], dot);  // (v is zero up to row j)
      }
      const double pv = sum_lanes(dot), half = 0.5 * tau * pv;
      const double c = fma(-tau, pv, readlane_f64(tp[K < 4 ? 0 : 1], (j + 1) & 63));  // (the reflector's first entry is 1: w_1 - half)
#pragma unroll
      for (int u = U0; u < 2; u++) {
        const int f = lj + 64 * u;
        wv[u] = fma(-half, v[u], tp[u]);
        x[u] = fma(-v[u], c, col[u] - tp[u]);
        V[f] = v[u];
        W[f] = wv[u];
      }
      const double d = readlane_f64(x[K < 4 ? 0 : 1], (j + 1) & 63);
      alpha = K < 4 ? element(x, j + 2) : readlane_f64(x[1], (j + 2) & 63);
#pragma unroll
      for (int u = U0; u < 2; u++) {
        const int f = lj + 64 * u;
        x[u] = f > j + 2 ? x[u] : 0.0;
        X[f] = x[u];
      }
      // ---- reflectors and results leave, sixteen columns at a time --------------------------------------------------
      if (w == 3) {
        const int q = jr & 15;
#pragma unroll
        for (int u = U0; u < 2; u++) vblk[lj + 64 * u][q] = (float)v[u];
        if (lj == 0) {
          eb[q] = beta;
          tb[q] = (float)tau;
          db[(jr + 1) & 31] = d;
        }
        between_lanes();
        if (q == 15 || j == F - 2) {
#pragma unroll
          for (int u = 0; u < 2; u++) {
            const int f = lj + 64 * u, r = f + base;
            if (r >= (jr & ~15)) {
              float4* dst = reinterpret_cast<float4*>(Vc + (size_t)img * Np * Np + ((size_t)(jr >> 4) * Np + r) * 16);
              float4* src = reinterpret_cast<float4*>(vblk[f]);
#pragma unroll
              for (int s = 0; s < 4; s++) {
                dst[s] = src[s];
                src[s] = float4{0.f, 0.f, 0.f, 0.f};
              }
            }
          }
          if (lj <= q) {
            const int col0 = (jr & ~15) + lj;
            dvec[(size_t)img * Np + col0] = db[col0 & 31];
            evec[(size_t)img * Np + col0] = eb[lj];
            tauv[(size_t)img * Np + col0] = tb[lj];
          }
        }
      }
      between_lanes();  // (X, V, W to the next column; sixteen results before the next overwrites them)
    }
  });
  if (tid == 3 * 64) {
    dvec[(size_t)img * Np + N - 1] = db[(N - 1) & 31];
    evec[(size_t)img * Np + N - 1] = 0.0;
    tauv[(size_t)img * Np + N - 1] = 0.f;
  }
}

template <class S>
static int launch_shape(const Plan& pl, const TrPhase& ph, double* G, double* dvec, double* evec, float* tauv, float* Vc, u64* sync,
                        size_t stride, u64* arrived, int patience, bool sixteen, int xcds, int32_t* fail, hipStream_t st) {
  if (S::LDS > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(tridiag_columns_kernel<S>),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS) != hipSuccess)
    return TC_ERR_HIP;
  // Captured launches cannot be kept apart.  Up to eight members on one XCD do no harm then (see TrTurn); sixteen are spread
  // over the XCDs like larger groups.
  TrTurn turn(S::P, S::LOCAL, pl.B, sixteen, xcds, st);
  if (turn.rc != TC_OK) return turn.rc;
  const int shift = turn.captured && S::P > 8 ? -1 : turn.first;
  const int grid = (S::LOCAL ? (pl.B + xcds - 1) / xcds * xcds : pl.B) * S::P;
  TC_TIMED(PK_TRIDIAG, 0, st, (tridiag_columns_kernel<S><<<grid, TR_THREADS, S::LDS, st>>>(G, pl.N, pl.Np, pl.B, ph.first, ph.last, dvec, evec, tauv, Vc, sync, stride, arrived, patience, xcds, shift, fail)));
  const int rc = check_launch(), rc2 = turn.done();
  return rc != TC_OK ? rc : rc2;
}

int launch_columns(const Plan& pl, const TrPhase& ph, double* G, double* dvec, double* evec, float* tauv, float* Vc, u64* sync,
                   size_t stride, u64* arrived, int patience, bool sixteen, int xcds, int32_t* fail, hipStream_t st) {
  switch (ph.size) {
    case TR_LAST_SIZE:
      TC_TIMED(PK_TRIDIAG, 0, st, (tridiag_last_kernel<<<pl.B, 256, 0, st>>>(G, pl.N, pl.Np, ph.first, dvec, evec, tauv, Vc, fail)));
      return check_launch();
#define TC_CASE(N_, LI_, LK_, P_, US_) case N_: return launch_shape<TcShape<LI_, LK_, P_>>(pl, ph, G, dvec, evec, tauv, Vc, sync, stride, arrived, patience, sixteen, xcds, fail, st);
    TC_FRAMES(TC_CASE)
#undef TC_CASE
  }
  return TC_ERR_SHAPE;
}

}  // namespace tc
