// Gram matrix G[b] = O[b] O[b]^T (the route to the SVD of Section 3.3.1: O = U Sigma V^T gives
// O O^T = U Sigma^2 U^T).  Products and sums are formed in float64 on the fp64 matrix cores so that
// small singular values are not drowned by the rounding of the large ones; G is stored in the
// eigensolver's type, zero padded to Np x Np.
#include "tc_internal.h"

namespace tc {

typedef __attribute__((ext_vector_type(4))) double d4;

constexpr int GK = 32;   // K chunk staged in LDS
constexpr int GLD = 66;  // panel leading dimension: panel[k][row]; 66 keeps the four contraction rows a wavefront reads at once in different banks

// Eight consecutive stored elements of a row, still in the storage type (converted on the way into LDS).
template <typename TIn> struct Raw8;
template <> struct Raw8<uint16_t> { uint4 v; };
template <> struct Raw8<f16_t> { uint4 v; };
template <> struct Raw8<float> { float4 a, b; };

template <typename TIn>
__device__ inline Raw8<TIn> fetch8(const TIn* src) {
  Raw8<TIn> r;
  if constexpr (sizeof(TIn) == 2) {
    r.v = *reinterpret_cast<const uint4*>(src);
  } else {
    r.a = *reinterpret_cast<const float4*>(src);
    r.b = *reinterpret_cast<const float4*>(src + 4);
  }
  return r;
}
template <typename TIn>
__device__ inline Raw8<TIn> zero8() {
  Raw8<TIn> r;
  if constexpr (sizeof(TIn) == 2) r.v = uint4{0, 0, 0, 0};
  else { r.a = float4{0, 0, 0, 0}; r.b = float4{0, 0, 0, 0}; }
  return r;
}
template <typename TIn>
__device__ inline void widen8(const Raw8<TIn>& r, double* dst) {
  if constexpr (sizeof(TIn) == 2) {
    const uint32_t w[4] = {r.v.x, r.v.y, r.v.z, r.v.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
      float lo, hi;
      unpack2<TIn>(w[i], &lo, &hi);
      dst[2 * i] = (double)lo;
      dst[2 * i + 1] = (double)hi;
    }
  } else {
    dst[0] = r.a.x; dst[1] = r.a.y; dst[2] = r.a.z; dst[3] = r.a.w;
    dst[4] = r.b.x; dst[5] = r.b.y; dst[6] = r.b.z; dst[7] = r.b.w;
  }
}

// One workgroup: a 64x64 tile (ti >= tj) of G for one image, mirrored into (tj, ti).  Wavefront w
// owns quadrant (w / 2, w % 2).  The products run on v_mfma_f64_4x4x4 (four independent 4x4x4 blocks
// per instruction), which sustains half as much again as the 16x16x4 form on this chip; a plain
// product with a long contraction can feed it: lane l = p + 4 q + 16 k holds A[p][k] of block q
// (here the same for all four blocks), B[k][p] of block q, and gets D[k][p] of block q, so with
//   A = rows 8 p + r of the quadrant (r = 0..7: eight products share one 16-byte-aligned run of LDS),
//   B = columns 2 (4 q + p) + s    (s = 0, 1: both in one 16-byte read),
// sixteen products per four contraction indices take five 16-byte LDS reads, and a lane ends with
// rows 8 k + r, columns 2 (4 q + p) + s: 16-byte pairs along the row for the tile, runs of eight
// along the column for its mirror.  The next 32 columns of O are fetched into registers meanwhile.
// In a tile on the diagonal the upper right quadrant is the mirror of the lower left one, bit for bit: its wavefront only
// loads and leaves the matrix cores of its SIMD to the other workgroups (64 images of 576 x 4096: 1.83 -> 1.76 ms).
// A tile takes one workgroup, and its contraction is a chain of D / 32 chunks (one image of 576 x 4096: 0.169 ms on 45 of the 256
// compute units, 0.069 with three workgroups per tile and the sum).
// Where the tiles of a call are few, `splits` workgroups share a tile: each contracts its part of D and leaves its sums,
// gram_sum_kernel adds them in order.  A float64 G keeps the first part in the place of the tile, rows of 64 as they come;
// the others (all of them for a float32 G) go to `part` [image][tile][split][8][256] (pairs, a lane's rows r).
template <typename TOut>
__host__ __device__ constexpr int parts_in_g() { return sizeof(TOut) == sizeof(double) ? 1 : 0; }

// the place of element 2 (256 r + tid) of the first part: four wavefronts, eight rows of the tile at a time
template <typename TOut>
__device__ inline TOut* place_in_g(TOut* Gb, int Np, int ti, int tj, int r, int tid) {
  return Gb + (size_t)(ti * 64 + 8 * r + (tid >> 5)) * Np + tj * 64 + ((2 * tid) & 63);
}

template <typename TOut>
__device__ inline void store_tile(const double (*acc)[2], TOut* __restrict__ Gb, int Np, int ti, int tj, int tid) {
  typedef __attribute__((ext_vector_type(2))) TOut o2;
  const int lane = tid & 63, wave = tid >> 6;
  const int p4 = lane & 3, blk = (lane >> 2) & 3, kq = lane >> 4;
  // the lane holds rows 8 kq + r, columns 2 (4 blk + p4) + s of its quadrant
  if (ti == tj && wave == 1) return;
  const int r0 = ti * 64 + (wave >> 1) * 32 + 8 * kq, c0 = tj * 64 + (wave & 1) * 32 + 2 * (4 * blk + p4);
#pragma unroll
  for (int r = 0; r < 8; r++)
    *reinterpret_cast<o2*>(&Gb[(size_t)(r0 + r) * Np + c0]) = o2{(TOut)acc[r][0], (TOut)acc[r][1]};
  if (ti != tj || wave == 2) {
#pragma unroll
    for (int sc = 0; sc < 2; sc++)
#pragma unroll
      for (int r = 0; r < 8; r += 2)
        *reinterpret_cast<o2*>(&Gb[(size_t)(c0 + sc) * Np + r0 + r]) = o2{(TOut)acc[r][sc], (TOut)acc[r + 1][sc]};
  }
}

template <typename TIn, typename TOut>
__global__ __launch_bounds__(256) void gram_kernel(const TIn* __restrict__ O, TOut* __restrict__ G, int N, int D,
                                                   int Np, int B, int splits, double* __restrict__ part) {
  typedef __attribute__((ext_vector_type(2))) double d2;
  __shared__ __attribute__((aligned(16))) double As[GK][GLD];
  __shared__ __attribute__((aligned(16))) double Bs[GK][GLD];
  const int ntile = Np / 64;
  int b, t;
  if (!group_on_xcd(blockIdx.x, ntile * (ntile + 1) / 2 * splits, B, &b, &t)) return;
  const int split = t % splits;
  t /= splits;
  double* mine = part + (((size_t)b * (ntile * (ntile + 1) / 2) + t) * (splits - parts_in_g<TOut>()) + split - parts_in_g<TOut>()) * 4096;
  int ti = 0;  // decode the lower-triangular tile index
  while (t >= ti + 1) { t -= ti + 1; ti++; }
  const int tj = t;
  const TIn* Ob = O + (size_t)b * N * D;
  TOut* Gb = G + (size_t)b * Np * Np;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int lrow = tid & 63, kc = tid >> 6;  // loader: row within the panel, which 8-wide k chunk
  const int p4 = lane & 3, blk = (lane >> 2) & 3, kq = lane >> 4;
  double acc[8][2];
#pragma unroll
  for (int r = 0; r < 8; r++) acc[r][0] = acc[r][1] = 0.0;
  const int rowA = ti * 64 + lrow, rowB = tj * 64 + lrow;
  const bool diag = ti == tj;
  const int nchunk = D / GK;  // (D is a multiple of 64)
  const int kbeg = (int)((long long)nchunk * split / splits) * GK, kend = (int)((long long)nchunk * (split + 1) / splits) * GK;
  const TIn* srcA = Ob + (size_t)rowA * D + kbeg + kc * 8;
  const TIn* srcB = Ob + (size_t)rowB * D + kbeg + kc * 8;
  Raw8<TIn> ra = rowA < N ? fetch8<TIn>(srcA) : zero8<TIn>();
  Raw8<TIn> rb = (!diag && rowB < N) ? fetch8<TIn>(srcB) : zero8<TIn>();
  for (int k0 = 0; k0 < kend - kbeg; k0 += GK) {
    double va[8], vb[8];
    widen8<TIn>(ra, va);
    if (!diag) widen8<TIn>(rb, vb);
    __syncthreads();  // previous chunk fully consumed
#pragma unroll
    for (int i = 0; i < 8; i++) {
      As[kc * 8 + i][lrow] = va[i];
      if (!diag) Bs[kc * 8 + i][lrow] = vb[i];
    }
    __syncthreads();
    if (k0 + GK < kend - kbeg) {  // in flight during the products
      if (rowA < N) ra = fetch8<TIn>(srcA + k0 + GK);
      if (!diag && rowB < N) rb = fetch8<TIn>(srcB + k0 + GK);
    }
    if (diag && wave == 1) continue;  // the mirror of wavefront 2's quadrant
    const double(*Bp)[GLD] = diag ? As : Bs;
#pragma unroll
    for (int kk = 0; kk < GK; kk += 4) {
      const double* arow = &As[kk + kq][wr * 32 + 8 * p4];
      const d2 a01 = *reinterpret_cast<const d2*>(arow), a23 = *reinterpret_cast<const d2*>(arow + 2);
      const d2 a45 = *reinterpret_cast<const d2*>(arow + 4), a67 = *reinterpret_cast<const d2*>(arow + 6);
      const d2 bb = *reinterpret_cast<const d2*>(&Bp[kk + kq][wc * 32 + 2 * (4 * blk + p4)]);
      const double a[8] = {a01.x, a01.y, a23.x, a23.y, a45.x, a45.y, a67.x, a67.y};
#pragma unroll
      for (int r = 0; r < 8; r++) {
        acc[r][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[r], bb.x, acc[r][0], 0, 0, 0);
        acc[r][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[r], bb.y, acc[r][1], 0, 0, 0);
      }
    }
  }
  if (splits > 1) {
    if (split < parts_in_g<TOut>()) {
#pragma unroll
      for (int r = 0; r < 8; r++) *reinterpret_cast<d2*>(place_in_g(Gb, Np, ti, tj, r, tid)) = d2{acc[r][0], acc[r][1]};
      return;
    }
#pragma unroll
    for (int r = 0; r < 8; r++) *reinterpret_cast<d2*>(mine + ((size_t)r * 256 + tid) * 2) = d2{acc[r][0], acc[r][1]};
    return;
  }
  store_tile<TOut>(acc, Gb, Np, ti, tj, tid);
}

template <typename TOut>
__global__ __launch_bounds__(256) void gram_sum_kernel(const double* __restrict__ part, TOut* __restrict__ G, int Np, int splits) {
  typedef __attribute__((ext_vector_type(2))) double d2;
  const int tid = threadIdx.x, b = blockIdx.y;
  int t = blockIdx.x, ti = 0;
  const double* p = part + ((size_t)b * gridDim.x + t) * (splits - parts_in_g<TOut>()) * 4096 + 2 * tid;
  TOut* Gb = G + (size_t)b * Np * Np;
  while (t >= ti + 1) { t -= ti + 1; ti++; }
  double acc[8][2];
#pragma unroll
  for (int r = 0; r < 8; r++) acc[r][0] = acc[r][1] = 0.0;
  if (parts_in_g<TOut>()) {
#pragma unroll
    for (int r = 0; r < 8; r++) {
      const d2 v = *reinterpret_cast<const d2*>(place_in_g(Gb, Np, ti, t, r, tid));
      acc[r][0] = v.x;
      acc[r][1] = v.y;
    }
  }
  for (int s = 0; s < splits - parts_in_g<TOut>(); s++) {
#pragma unroll
    for (int r = 0; r < 8; r++) {
      const d2 v = *reinterpret_cast<const d2*>(p + (size_t)s * 4096 + r * 512);
      acc[r][0] += v.x;
      acc[r][1] += v.y;
    }
  }
  __syncthreads();  // the first part has been read by everyone
  store_tile<TOut>(acc, Gb, Np, ti, t, tid);
}

// Workgroups per tile: as many as keep the launch within three per compute unit, with at least eight chunks each and no more
// than 3 MiB of parts per image: a workspace stays in proportion to the batch (one image of 576 x 4096 needs 14 MB; eight
// workgroups per tile would add 7 to save another 0.012 ms of 2.5).  By the size of the whole call: the order of a sum
// must not depend on stream groups.
static size_t part_bytes(const Plan& pl, int splits) {  // of one image
  const size_t nt = pl.Np / 64, parts = splits - (pl.tsize == 8 ? parts_in_g<double>() : parts_in_g<float>());
  return splits > 1 ? nt * (nt + 1) / 2 * parts * 4096 * 8 : 0;
}
int gram_splits(const Plan& pl) {
  const int nt = pl.Np / 64;
  const long long tiles = (long long)nt * (nt + 1) / 2 * pl.batch_call;
  int s = 1;
  while (s < 8 && tiles * (s + 1) <= 768 && pl.D / GK >= 8 * (s + 1) && part_bytes(pl, s + 1) <= (3u << 20)) s++;
  return s;
}
size_t gram_part_bytes(const Plan& pl) { return part_bytes(pl, gram_splits(pl)); }
// What a plan sets aside for the parts of all its images.  The parts themselves get fewer where another tile or image takes
// away a workgroup per tile; a workspace must not, since a smaller call has to fit it: an image has at most 3 MiB and at most as
// many parts as D allows, a call at most a part for each of its 768 workgroups.
size_t gram_reserve_bytes(const Plan& pl) {
  const int most = pl.D / GK / 8 < 8 ? pl.D / GK / 8 : 8;
  const size_t image = part_bytes(pl, most), lim = (size_t)3 << 20, call = (size_t)768 * 4096 * 8;
  const size_t all = (image < lim ? image : lim) * pl.B;
  return all < call ? all : call;
}

template <typename TIn, typename TOut>
static void run_gram(const Plan& pl, const void* O, void* G, double* part, hipStream_t st) {
  const int nt = pl.Np / 64, tiles = nt * (nt + 1) / 2, splits = gram_splits(pl);
  TC_TIMED(PK_GRAM, 0, st, (gram_kernel<TIn, TOut><<<grid_for_groups(tiles * splits, pl.B), 256, 0, st>>>((const TIn*)O, (TOut*)G, pl.N, pl.D, pl.Np, pl.B, splits, part)));
  if (splits > 1) TC_TIMED(PK_GRAM, 1, st, (gram_sum_kernel<TOut><<<dim3(tiles, pl.B), 256, 0, st>>>(part, (TOut*)G, pl.Np, splits)));
}

int launch_gram(const Plan& pl, int dtype, int eig_dtype, const void* O, void* G, double* part, hipStream_t st) {
  const bool f64 = eig_dtype == TC_EIG_F64;
  if (dtype == TC_BF16) f64 ? run_gram<uint16_t, double>(pl, O, G, part, st) : run_gram<uint16_t, float>(pl, O, G, part, st);
  else if (dtype == TC_F16) f64 ? run_gram<f16_t, double>(pl, O, G, part, st) : run_gram<f16_t, float>(pl, O, G, part, st);
  else f64 ? run_gram<float, double>(pl, O, G, part, st) : run_gram<float, float>(pl, O, G, part, st);
  return check_launch();
}

}  // namespace tc
