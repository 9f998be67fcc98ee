// Stage II (Section 3.3.2): cosine similarity between SetB and SetA rows of the metric (Eq. 3-10),
// choice of the merged tokens and their destinations, and the averaging pass that writes the
// compressed token rows in ascending position.
#include <type_traits>

#include "tc_internal.h"

namespace tc {

typedef __attribute__((ext_vector_type(8))) __bf16 bf8;
typedef __attribute__((ext_vector_type(8))) _Float16 h8;
typedef __attribute__((ext_vector_type(16))) float f16v;

// ---- 1 / ||metric row||_2 for the k_prune surviving rows, in score order (float rows) -----------
__global__ __launch_bounds__(256) void rownorm_kernel(const float* __restrict__ metric, const int32_t* __restrict__ order,
                                                      float* __restrict__ rnorm, int N, int D, int kp) {
  const int b = blockIdx.y, lane = threadIdx.x & 63, r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= kp) return;
  const int x = min(max(order[(size_t)b * kp + r], 0), N - 1);
  const float* row = metric + ((size_t)b * N + x) * D;
  float ss = 0.f;
  for (int k = lane * 4; k < D; k += 256) {
    const float4 v = *reinterpret_cast<const float4*>(row + k);
    ss += v.x * v.x; ss += v.y * v.y; ss += v.z * v.z; ss += v.w * v.w;
  }
  ss = wave_sum(ss);
  if (lane == 0) rnorm[(size_t)b * kp + r] = 1.0f / fmaxf(sqrtf(ss), 1e-30f);
}

// ---- Sim[b][j][i] = <z_Bj, z_Ai> / (|z_Bj| |z_Ai|), 16-bit rows (bf16 or half) on the matrix cores ---
// What leaves a tile: the similarities themselves (sim, tc_similarity), or (part) for each of its SetB rows the key of the most
// similar of its SetA rows, part[b][j][tile column]: the merge needs no more, and the matrix is neither written nor read.
typedef unsigned long long u64;

__device__ inline u64 best_key(float v, int a) {
  if (v != v) v = -INFINITY;  // a NaN similarity (a NaN in the metric row) loses against everything
  return order_key(v, a);     // equal similarity: lower visual index
}
__device__ inline u64 key_max(u64 a, u64 b) { return a > b ? a : b; }

template <bool F16>
__device__ inline f16v sim_mma(uint4 a, uint4 b, f16v c) {
  union U { uint4 u; bf8 b; h8 h; };
  U x, y;
  x.u = a;
  y.u = b;
  if constexpr (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(x.h, y.h, c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.b, y.b, c, 0, 0, 0);
}

constexpr int SK = 64;       // K chunk
constexpr int SP = SK + 8;   // padded LDS row (16-bit elements)

// acc[i] += the square of element i of eight 16-bit elements
template <bool F16>
__device__ inline void add_squares(uint4 v, float* acc) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; i++) {
    float lo, hi;
    unpack2<typename std::conditional<F16, f16_t, uint16_t>::type>(w[i], &lo, &hi);
    acc[2 * i] = fmaf(lo, lo, acc[2 * i]);
    acc[2 * i + 1] = fmaf(hi, hi, acc[2 * i + 1]);
  }
}
__device__ inline float sum8f(const float* q) { return ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7])); }
__device__ inline float inv_norm(float ss) { return 1.0f / fmaxf(sqrtf(ss), 1e-30f); }

// 64 x 64 tiles through LDS, two chunks in flight while one is multiplied: for calls with enough tiles.  The row norms are
// formed from the rows on their way through the registers: a launch of their own read all rows once more (64 images of 256
// rows of 4096: 40 + 51 us, now 59).
template <bool F16>
__global__ __launch_bounds__(256) void sim_tile_kernel(const uint16_t* __restrict__ metric, const int32_t* __restrict__ order,
                                                       float* __restrict__ sim, u64* __restrict__ part, int N, int D, int kp,
                                                       int nA, int nB) {
  __shared__ __attribute__((aligned(16))) uint16_t rows[2][64][SP];
  static_assert(sizeof(rows) >= 64 * 65 * 4, "the tile of similarities takes their place");
  __shared__ int ordA[64];
  __shared__ float rn[2][64];
  uint16_t(*Bj)[SP] = rows[0];
  uint16_t(*Ai)[SP] = rows[1];
  const int b = blockIdx.y;
  const int tilesA = (nA + 63) / 64;
  const int tj = blockIdx.x / tilesA, ti = blockIdx.x % tilesA;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wr = wave >> 1, wc = wave & 1;
  const int32_t* ord = order + (size_t)b * kp;
  const int lrow = tid >> 2, piece = tid & 3;  // loader: 64 rows x 4 pieces of 16 elements
  // (rows past the end repeat the last one: what they give is not used)
  const int j_l = min(tj * 64 + lrow, nB - 1), i_l = min(ti * 64 + lrow, nA - 1);
  const uint16_t* srcB = metric + ((size_t)b * N + min(max(ord[nA + j_l], 0), N - 1)) * D + piece * 16;
  const uint16_t* srcA = metric + ((size_t)b * N + min(max(ord[i_l], 0), N - 1)) * D + piece * 16;
  if (tid < 64) ordA[tid] = ord[min(ti * 64 + tid, nA - 1)];
  f16v acc;
#pragma unroll
  for (int i = 0; i < 16; i++) acc[i] = 0.f;
  float qb[16], qa[16];
#pragma unroll
  for (int i = 0; i < 16; i++) qb[i] = qa[i] = 0.f;
  uint4 r[2][4];
  auto load = [&](int k, uint4* q) {  // (D is a multiple of SK; past the end the last chunk again)
    const int kk = min(k, D - SK);
    q[0] = *reinterpret_cast<const uint4*>(srcB + kk);
    q[1] = *reinterpret_cast<const uint4*>(srcB + kk + 8);
    q[2] = *reinterpret_cast<const uint4*>(srcA + kk);
    q[3] = *reinterpret_cast<const uint4*>(srcA + kk + 8);
  };
  auto step = [&](int k0, uint4* q) {
    __syncthreads();
    *reinterpret_cast<uint4*>(&Bj[lrow][piece * 16]) = q[0];
    *reinterpret_cast<uint4*>(&Bj[lrow][piece * 16 + 8]) = q[1];
    *reinterpret_cast<uint4*>(&Ai[lrow][piece * 16]) = q[2];
    *reinterpret_cast<uint4*>(&Ai[lrow][piece * 16 + 8]) = q[3];
    add_squares<F16>(q[0], qb);
    add_squares<F16>(q[1], qb + 8);
    add_squares<F16>(q[2], qa);
    add_squares<F16>(q[3], qa + 8);
    load(k0 + 2 * SK, q);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < SK; kk += 16)
      acc = sim_mma<F16>(*reinterpret_cast<const uint4*>(&Bj[wr * 32 + (lane & 31)][kk + 8 * (lane >> 5)]),
                         *reinterpret_cast<const uint4*>(&Ai[wc * 32 + (lane & 31)][kk + 8 * (lane >> 5)]), acc);
  };
  load(0, r[0]);
  load(SK, r[1]);
  for (int k0 = 0; k0 < D; k0 += 2 * SK) {
    step(k0, r[0]);
    if (k0 + SK < D) step(k0 + SK, r[1]);  // uniform
  }
  {
    float sb = sum8f(qb) + sum8f(qb + 8), sa = sum8f(qa) + sum8f(qa + 8);
    sb += __shfl_xor(sb, 1, 64);
    sa += __shfl_xor(sa, 1, 64);
    sb += __shfl_xor(sb, 2, 64);
    sa += __shfl_xor(sa, 2, 64);
    if (piece == 0) {
      rn[0][lrow] = inv_norm(sb);
      rn[1][lrow] = inv_norm(sa);
    }
  }
  __syncthreads();
  float(*tile)[65] = reinterpret_cast<float(*)[65]>(&rows[0][0][0]);
  const int il = wc * 32 + (lane & 31), i = ti * 64 + il;
  const float rn_i = rn[1][il];
#pragma unroll
  for (int e = 0; e < 16; e++) {
    const int jl = wr * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3), j = tj * 64 + jl;
    const float v = acc[e] * rn[0][jl] * rn_i;
    if (part) tile[jl][il] = v;
    else if (i < nA && j < nB) sim[((size_t)b * nB + j) * nA + i] = v;
  }
  if (!part) return;
  __syncthreads();
  u64 best = 0;
  for (int c = piece; c < min(64, nA - ti * 64); c += 4) best = key_max(best, best_key(tile[lrow][c], ordA[c]));
  best = key_max(best, __shfl_xor(best, 1, 64));
  best = key_max(best, __shfl_xor(best, 2, 64));
  if (piece == 0 && tj * 64 + lrow < nB) part[((size_t)b * nB + tj * 64 + lrow) * tilesA + ti] = best;
}

// 32 x 32 tiles, the contraction split over eight wavefronts that read their rows straight into operand registers (eight
// steps in flight, no barrier before the end) and form the row norms on the way: for calls with few tiles, where the
// 64 x 64 form is a chain of D / 64 chunks on a handful of compute units (one image of 256 survivors: 5 + 43 -> 21 us; 64 images of
// 128: 15 + 51 -> 34 us).
constexpr int SW = 8;
// Where the forms meet: 64 images of 256 survivors (256 tiles of 64 x 64) 59 us in tiles, 102 split; 64 of 128 (64 tiles) 66 in tiles
// with norms of their own, 34 split.
constexpr long long SIM_FEW = 192;
template <bool F16>
__global__ __launch_bounds__(64 * SW) void sim_split_kernel(const uint16_t* __restrict__ metric, const int32_t* __restrict__ order,
                                                            float* __restrict__ sim, u64* __restrict__ part, int N, int D,
                                                            int kp, int nA, int nB) {
  __shared__ float red[SW][1024];
  __shared__ float nrm[2][SW][32];
  __shared__ float tile[32][33];
  __shared__ float rn[2][32];
  const int b = blockIdx.y;
  const int tilesA = (nA + 31) / 32;
  const int tj = blockIdx.x / tilesA, ti = blockIdx.x % tilesA;
  const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, wave = tid >> 6;
  const int32_t* ord = order + (size_t)b * kp;
  const int j_l = min(tj * 32 + l31, nB - 1), i_l = min(ti * 32 + l31, nA - 1);
  const uint16_t* srcB = metric + ((size_t)b * N + min(max(ord[nA + j_l], 0), N - 1)) * D + 8 * (lane >> 5);
  const uint16_t* srcA = metric + ((size_t)b * N + min(max(ord[i_l], 0), N - 1)) * D + 8 * (lane >> 5);
  const int steps = D / 16, s0 = steps * wave / SW, s1 = steps * (wave + 1) / SW;  // (D is a multiple of 64)
  f16v acc;
#pragma unroll
  for (int i = 0; i < 16; i++) acc[i] = 0.f;
  float qb[8], qa[8];
#pragma unroll
  for (int i = 0; i < 8; i++) qb[i] = qa[i] = 0.f;
  for (int s = s0; s < s1; s += 8) {
    uint4 fb[8], fa[8];
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const int k = min(s + u, s1 - 1) * 16;
      fb[u] = *reinterpret_cast<const uint4*>(srcB + k);
      fa[u] = *reinterpret_cast<const uint4*>(srcA + k);
    }
#pragma unroll
    for (int u = 0; u < 8; u++)
      if (s + u < s1) {  // uniform
        acc = sim_mma<F16>(fb[u], fa[u], acc);
        add_squares<F16>(fb[u], qb);
        add_squares<F16>(fa[u], qa);
      }
  }
  auto total = [](const float* q) {
    const float t = sum8f(q);
    return t + __shfl_xor(t, 32, 64);
  };
  const float tb = total(qb), ta = total(qa);
  if (lane < 32) {
    nrm[0][wave][l31] = tb;
    nrm[1][wave][l31] = ta;
  }
#pragma unroll
  for (int r = 0; r < 16; r++) red[wave][r * 64 + lane] = acc[r];
  __syncthreads();
  if (tid < 64) {
    float ss = 0.f;
#pragma unroll
    for (int w = 0; w < SW; w++) ss += nrm[tid >> 5][w][l31];
    rn[tid >> 5][l31] = inv_norm(ss);
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; h++) {
    const int e = tid + 512 * h, r = e >> 6;
    const int jl = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < SW; w++) v += red[w][e];
    v = v * rn[0][jl] * rn[1][l31];
    if (part) tile[jl][l31] = v;
    else if (ti * 32 + l31 < nA && tj * 32 + jl < nB) sim[((size_t)b * nB + tj * 32 + jl) * nA + ti * 32 + l31] = v;
  }
  if (!part) return;
  __syncthreads();
  const int row = tid >> 4;
  u64 best = 0;
  for (int c = tid & 15; c < min(32, nA - ti * 32); c += 16) best = key_max(best, best_key(tile[row][c], ord[ti * 32 + c]));
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) best = key_max(best, __shfl_xor(best, o, 64));
  if ((tid & 15) == 0 && tj * 32 + row < nB) part[((size_t)b * nB + tj * 32 + row) * tilesA + ti] = best;
}

// float rows: plain LDS-tiled FMA (the float32 storage type is a correctness path, not a fast one)
__global__ __launch_bounds__(256) void sim_f32_kernel(const float* __restrict__ metric,
                                                      const int32_t* __restrict__ order,
                                                      const float* __restrict__ rnorm, float* __restrict__ sim,
                                                      u64* __restrict__ part, int N, int D, int kp, int nA, int nB) {
  __shared__ float Bj[16][33];
  __shared__ float Ai[16][33];
  const int b = blockIdx.y;
  const int tilesA = (nA + 15) / 16;
  const int tj = blockIdx.x / tilesA, ti = blockIdx.x % tilesA;
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int32_t* ord = order + (size_t)b * kp;
  const int lrow = tid >> 4, lk = tid & 15;
  const int j_l = tj * 16 + lrow, i_l = ti * 16 + lrow;
  const float* srcB = j_l < nB ? metric + ((size_t)b * N + min(max(ord[nA + j_l], 0), N - 1)) * D : nullptr;
  const float* srcA = i_l < nA ? metric + ((size_t)b * N + min(max(ord[i_l], 0), N - 1)) * D : nullptr;
  double acc = 0.0;
  for (int k0 = 0; k0 < D; k0 += 32) {
    __syncthreads();
    for (int h = 0; h < 2; h++) {
      const int k = k0 + lk + 16 * h;
      Bj[lrow][lk + 16 * h] = (srcB && k < D) ? srcB[k] : 0.f;
      Ai[lrow][lk + 16 * h] = (srcA && k < D) ? srcA[k] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 32; k++) acc += (double)Bj[ty][k] * (double)Ai[tx][k];
  }
  const int j = tj * 16 + ty, i = ti * 16 + tx;
  const bool in = j < nB && i < nA;
  const float v = in ? (float)acc * rnorm[(size_t)b * kp + nA + j] * rnorm[(size_t)b * kp + i] : 0.f;
  if (!part) {
    if (in) sim[((size_t)b * nB + j) * nA + i] = v;
    return;
  }
  u64 best = in ? best_key(v, ord[i]) : 0;
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) best = key_max(best, __shfl_xor(best, o, 64));
  if (tx == 0 && j < nB) part[((size_t)b * nB + j) * tilesA + ti] = best;
}

// ---- per image: most similar SetA token of every SetB token, top-m of SetB, index bookkeeping -----
// LDS: key[nB] (8 bytes) | best[nB] | dst[N]
// One workgroup per image, bound by its chain of steps: the best of a row's tiles, a rank by counting, one scan.
constexpr int AS_THREADS = 1024;
__global__ __launch_bounds__(AS_THREADS) void assign_kernel(const u64* __restrict__ part, const int32_t* __restrict__ order,
                                                            int32_t* __restrict__ kept_idx, int32_t* __restrict__ merge_dst,
                                                            int32_t* __restrict__ mlist, int N, int kp, int kf, int nA,
                                                            int nB, int tilesA) {
  extern __shared__ __attribute__((aligned(16))) unsigned char as_smem[];
  u64* key = reinterpret_cast<u64*>(as_smem);
  int* best = reinterpret_cast<int*>(key + nB);
  int* dst = best + nB;
  __shared__ uint32_t wsum[AS_THREADS / 64];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t* ord = order + (size_t)b * kp;
  const int m = kp - kf;
  for (int x = tid; x < N; x += AS_THREADS) dst[x] = -1;
  for (int j = tid; j < nB; j += AS_THREADS) {
    const u64* p = part + ((size_t)b * nB + j) * tilesA;
    u64 k = 0;
    for (int t = 0; t < tilesA; t++) k = key_max(k, p[t]);
    // the rank among the SetB tokens: the same similarity, equal ones by the token's own index
    key[j] = (k & 0xffffffff00000000ull) | (0x7fffffffu - (uint32_t)ord[nA + j]);
    best[j] = (int)(0x7fffffffu - (uint32_t)k);
  }
  __syncthreads();
  for (int r = tid; r < kp; r += AS_THREADS) {
    const int x = ord[r];
    if ((unsigned)x < (unsigned)N) dst[x] = x;  // entries outside [0,N) violate the contract and are ignored
  }
  __syncthreads();
  // the m SetB tokens with the highest similarity; equal similarity -> lower visual index
  for (int j = tid; j < nB; j += AS_THREADS) {
    const u64 mine = key[j];
    int rank = 0;
#pragma unroll 8
    for (int k = 0; k < nB; k++) rank += key[k] > mine ? 1 : 0;
    const int xj = ord[nA + j];
    if (rank < m && (unsigned)xj < (unsigned)N) dst[xj] = best[j];
  }
  __syncthreads();
  // compact, in ascending position: output rows (dst[x] == x) and merged sources (dst[x] != x, >= 0)
  const int chunk = (N + AS_THREADS - 1) / AS_THREADS;
  const int x0 = min(N, tid * chunk), x1 = min(N, x0 + chunk);
  uint32_t mine = 0;  // both counts in one word (at most MAX_NVIS each)
  for (int x = x0; x < x1; x++) {
    const int d = dst[x];
    mine += d == x ? 1u : d >= 0 ? 0x10000u : 0u;
  }
  uint32_t sum = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(sum, o, 64);
    sum += lane >= o ? v : 0u;
  }
  if (lane == 63) wsum[wave] = sum;
  __syncthreads();
  uint32_t before = sum - mine;
  for (int w = 0; w < wave; w++) before += wsum[w];
  int pk = before & 0xffffu, pm = before >> 16;
  for (int x = x0; x < x1; x++) {
    const int d = dst[x];
    if (d == x) { if (pk < kf) kept_idx[(size_t)b * kf + pk++] = x; }
    else if (d >= 0 && pm < m) { mlist[((size_t)b * (m > 0 ? m : 1) + pm) * 2] = x; mlist[((size_t)b * (m > 0 ? m : 1) + pm) * 2 + 1] = d; pm++; }
  }
  for (int x = tid; x < N; x += AS_THREADS) merge_dst[(size_t)b * N + x] = dst[x];
}

// ---- averaging pass: one workgroup per output row ------------------------------------------------
template <typename TIn>
__global__ __launch_bounds__(256) void average_kernel(const TIn* __restrict__ X, const int32_t* __restrict__ kept_idx,
                                                      const int32_t* __restrict__ mlist, TIn* __restrict__ X_out,
                                                      int N, int hidden, int kf, int m) {
  constexpr int V = 16 / sizeof(TIn);  // elements per 16-byte access
  __shared__ int srcs[MAX_NVIS / 2];   // sources merged into this row, ascending position
  __shared__ int wave_cnt[4];
  const int b = blockIdx.y, r = blockIdx.x, tid = threadIdx.x;
  const int a = kept_idx[(size_t)b * kf + r];
  const int32_t* ml = mlist + (size_t)b * (m > 0 ? m : 1) * 2;
  const TIn* Xb = X + (size_t)b * N * hidden;
  TIn* out = X_out + ((size_t)b * kf + r) * hidden;
  int nsrc = 0;
  for (int base = 0; base < m; base += 256) {  // uniform trip count; order of mlist is kept
    const int e = base + tid;
    const bool hit = e < m && ml[2 * e + 1] == a;
    const unsigned long long mask = __ballot(hit);
    __syncthreads();
    if ((tid & 63) == 0) wave_cnt[tid >> 6] = __popcll(mask);
    __syncthreads();
    int off = nsrc;
    for (int w = 0; w < (tid >> 6); w++) off += wave_cnt[w];
    if (hit) srcs[off + __popcll(mask & ((1ull << (tid & 63)) - 1ull))] = ml[2 * e];
    nsrc += wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3];
  }
  __syncthreads();
  const float fc = (float)(1 + nsrc);
  for (int v0 = tid * V; v0 < hidden; v0 += 256 * V) {
    float acc[V];
    auto add_row = [&](const TIn* row, bool first) {
      const uint4 raw = *reinterpret_cast<const uint4*>(row + v0);
      const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
      if constexpr (sizeof(TIn) == 2) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
          float lo, hi;
          unpack2<TIn>(w[i], &lo, &hi);
          acc[2 * i] = first ? lo : acc[2 * i] + lo;
          acc[2 * i + 1] = first ? hi : acc[2 * i + 1] + hi;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 4; i++) acc[i] = first ? __uint_as_float(w[i]) : acc[i] + __uint_as_float(w[i]);
      }
    };
    add_row(Xb + (size_t)a * hidden, true);
    for (int s = 0; s < nsrc; s++) add_row(Xb + (size_t)srcs[s] * hidden, false);
    uint32_t w[4];
    if constexpr (sizeof(TIn) == 2) {
#pragma unroll
      for (int i = 0; i < 4; i++) w[i] = pack2<TIn>(acc[2 * i] / fc, acc[2 * i + 1] / fc);
    } else {
#pragma unroll
      for (int i = 0; i < 4; i++) w[i] = __float_as_uint(acc[i] / fc);
    }
    *reinterpret_cast<uint4*>(out + v0) = uint4{w[0], w[1], w[2], w[3]};
  }
}

// Eq. 3-10: Sim [B, |B|, |A|] (sim), or the best of every row and tile (part); the number of tiles of a row in *tilesA.
static int run_similarity(const Plan& pl, int dtype, const void* metric, const int32_t* order, float* rnorm, float* sim,
                          u64* part, int* tilesA, hipStream_t st) {
  *tilesA = 0;
  if (pl.nA == 0) return TC_OK;  // a single survivor: Set A is empty, there is nothing to compare
  auto tiles = [&](int t) { return dim3(((pl.nB + t - 1) / t) * ((pl.nA + t - 1) / t), pl.B); };
  if (dtype == TC_F32) {
    *tilesA = (pl.nA + 15) / 16;
    const dim3 gn((pl.kp + 3) / 4, pl.B);
    TC_TIMED(PK_ROWNORM, 0, st, (rownorm_kernel<<<gn, 256, 0, st>>>((const float*)metric, order, rnorm, pl.N, pl.D, pl.kp)));
    TC_TIMED(PK_SIM, 0, st, (sim_f32_kernel<<<tiles(16), 256, 0, st>>>((const float*)metric, order, rnorm, sim, part, pl.N, pl.D, pl.kp, pl.nA, pl.nB)));
    return check_launch();
  }
  const uint16_t* z = (const uint16_t*)metric;
  const dim3 g64 = tiles(64);
  if ((long long)g64.x * pl.B < SIM_FEW) {
    *tilesA = (pl.nA + 31) / 32;
    if (dtype == TC_F16) TC_TIMED(PK_SIM, 0, st, (sim_split_kernel<true><<<tiles(32), 64 * SW, 0, st>>>(z, order, sim, part, pl.N, pl.D, pl.kp, pl.nA, pl.nB)));
    else TC_TIMED(PK_SIM, 0, st, (sim_split_kernel<false><<<tiles(32), 64 * SW, 0, st>>>(z, order, sim, part, pl.N, pl.D, pl.kp, pl.nA, pl.nB)));
    return check_launch();
  }
  *tilesA = (pl.nA + 63) / 64;
  if (dtype == TC_F16) TC_TIMED(PK_SIM, 0, st, (sim_tile_kernel<true><<<g64, 256, 0, st>>>(z, order, sim, part, pl.N, pl.D, pl.kp, pl.nA, pl.nB)));
  else TC_TIMED(PK_SIM, 0, st, (sim_tile_kernel<false><<<g64, 256, 0, st>>>(z, order, sim, part, pl.N, pl.D, pl.kp, pl.nA, pl.nB)));
  return check_launch();
}

int launch_similarity(const Plan& pl, int dtype, const void* metric, const int32_t* order, float* rnorm, float* sim,
                      hipStream_t st) {
  int tilesA;
  return run_similarity(pl, dtype, metric, order, rnorm, sim, nullptr, &tilesA, st);
}

int launch_merge(const Plan& pl, int dtype, const void* X, const void* metric, const int32_t* order, void* X_out,
                 int32_t* kept_idx, int32_t* merge_dst, float* rnorm, void* part, int32_t* mlist, hipStream_t st) {
  int tilesA;
  const int rc = run_similarity(pl, dtype, metric, order, rnorm, nullptr, static_cast<u64*>(part), &tilesA, st);
  if (rc != TC_OK) return rc;
  const size_t lds = ((size_t)pl.N + 3 * (size_t)pl.nB) * 4;
  TC_TIMED(PK_ASSIGN, 0, st, (assign_kernel<<<pl.B, AS_THREADS, lds, st>>>(static_cast<const u64*>(part), order, kept_idx, merge_dst, mlist, pl.N, pl.kp, pl.kf, pl.nA, pl.nB, tilesA)));
  const dim3 ga(pl.kf, pl.B);
  if (dtype == TC_F16)
    TC_TIMED(PK_AVERAGE, 0, st, (average_kernel<f16_t><<<ga, 256, 0, st>>>((const f16_t*)X, kept_idx, mlist, (f16_t*)X_out, pl.N, pl.hidden, pl.kf, pl.m)));
  else if (dtype == TC_BF16)
    TC_TIMED(PK_AVERAGE, 0, st, (average_kernel<uint16_t><<<ga, 256, 0, st>>>((const uint16_t*)X, kept_idx, mlist, (uint16_t*)X_out, pl.N, pl.hidden,
                                                pl.kf, pl.m)));
  else
    TC_TIMED(PK_AVERAGE, 0, st, (average_kernel<float><<<ga, 256, 0, st>>>((const float*)X, kept_idx, mlist, (float*)X_out, pl.N, pl.hidden, pl.kf,
                                             pl.m)));
  return check_launch();
}

}  // namespace tc
