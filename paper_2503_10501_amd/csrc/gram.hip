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

// What the digits of 16-bit rows (below) leave out of an image: single values, and rows that are formed anew, which take as long
// as D / 128 values.  With much of it gram_kernel forms the image, and the digits' products are not begun.  The line is where
// adding what is left (gram_rows_kernel) takes six tenths of what the products save; it is not proportional to D, since a value
// left also costs a row of G.  us: 64 images of 576 x 4096 (1070 saved), 36 values an image 64, 576 322, 1152 490, 1536 618; 4 rows
// anew 89, 18 256, 24 313; 8 of 2880 x 4096 (3100), 2880 values 1142, 7680 1768; 20 rows 213, 120 1169; 128 of 576 x 1024 (470),
// 36 values 99, 144 256, 384 511; 18 rows 193, 24 237.
struct Left { int values, anew; };
__device__ inline bool too_much(Left l, int N, int D) {
  return l.values + l.anew * (D / 128.f) > fmaxf((float)N * (D - 768) / 1280.f, N / 8.f);
}
// Of an image, from its blocks of eight rows (rows anew in the upper half of a word); every wavefront asks for itself.
__device__ inline Left image_left(const int32_t* __restrict__ blocks, int Np) {
  int n = 0;
  for (int i = threadIdx.x & 63; i < Np / 8; i += 64) n += blocks[i];
  n = wave_sum(n);
  return {n & 0xffff, n >> 16};  // (at most 32768 values)
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
                                                   int Np, int B, int splits, double* __restrict__ part,
                                                   const int32_t* __restrict__ left_over) {
  typedef __attribute__((ext_vector_type(2))) double d2;
  __shared__ __attribute__((aligned(16))) double As[GK][GLD];
  __shared__ __attribute__((aligned(16))) double Bs[GK][GLD];
  const int ntile = Np / 64;
  int b, t;
  if (!group_on_xcd(blockIdx.x, ntile * (ntile + 1) / 2 * splits, B, &b, &t)) return;
  if (left_over && !too_much(image_left(left_over + (size_t)b * (Np / 8), Np), N, D)) return;  // the digits have formed this image's products
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

// ---- 16-bit rows: the products in whole numbers, exact -------------------------------------------------------------
// The float64 matrix cores bound the kernel above (74 % busy); the 8-bit integer ones do sixty times the operations.  A row of
// 16-bit values, scaled by a power of two that brings its largest to 31 bits, is a row of whole numbers unless one of its
// values lies below about 2^-23 of the largest (bf16, eight bits of significand; in Gaussian rows one value in two million) or
// 2^-20 (half, eleven bits; none where the largest is below 128, since the unit of the type is 2^-24).  Four signed digits to the base
// 256 each, sixteen digit products per product, summed in 32 bits by the weight of the digits (seven sums; D <= 16384 keeps
// them below 2^31), joined in 64 bits and rounded once: no sum of float64 products is closer.  Values that are
// not whole numbers are added in float64, rows with more than a few, an infinity or NaN are formed in float64
// (gram_rows_kernel), an image with many of either by gram_kernel.
// The digits lie in memory as the matrix instruction takes them: [32 rows][32 columns of O][digit][lane][16], lane l holds row
// l % 32, columns 16 (l / 32) ..; a fragment is 1 KB in one piece, and copies to LDS and reads from it have no bank conflicts.
typedef __attribute__((ext_vector_type(4))) int i4;
typedef __attribute__((ext_vector_type(16))) int i16v;

__device__ inline uint32_t bits16(uint16_t v) { return v; }
__device__ inline uint32_t bits16(f16_t v) { return v.bits; }
template <typename TIn> __device__ inline float widen1(uint32_t bits) {
  float lo, hi;
  unpack2<TIn>(bits, &lo, &hi);
  return lo;
}

// Per row: the exponent of its scale and how many of its values are no whole numbers (their columns are listed and they count
// as zero in the digits); ROW_WHOLE where they are more, or one is not finite.
constexpr int ROW_LIST = 8, ROW_WHOLE = 15;
__device__ inline int row_scale(int info) { return info >> 4; }
__device__ inline int row_left(int info) { return info & 15; }

// x 2^s, if it is a whole number (a value that vanishes in the scaling is none)
__device__ inline bool whole(float x, int s, int* q) {
  const float v = ldexpf(x, s);
  *q = (int)v;
  return (float)*q == v && (*q != 0 || x == 0.f);
}
// the bits of the power of two 2^e in storage type TIn; 0x8000 (above every value) or 0 where that has none
template <typename TIn> __device__ inline uint32_t least_bits(int e) {
  constexpr bool half = __is_same(TIn, f16_t);
  constexpr int LOW = half ? -24 : -133, NORMAL = half ? -14 : -126, HIGH = half ? 15 : 127, BITS = half ? 10 : 7;
  if (e > HIGH) return 0x8000u;
  if (e < LOW) return 0;
  return e < NORMAL ? 1u << (e - LOW) : (uint32_t)(e - NORMAL + 1) << BITS;
}

// One workgroup: eight rows, read once and kept in registers until their largest value is known and what they leave is listed;
// eight that are formed anew need no digits.  Bound by memory: 2 bytes an element in, 4 out (64 images of 576 x 4096: 32 rows a
// workgroup, read twice, took 222 us; one image 23).
template <typename TIn, int ITER>  // ITER: runs of 16 columns per thread, D <= 2048 ITER
__global__ __launch_bounds__(1024) void gram_slice_kernel(const TIn* __restrict__ O, char* __restrict__ P, int32_t* __restrict__ rowinfo,
                                                          uint16_t* __restrict__ left, int32_t* __restrict__ left_over, int N, int D, int Np) {
  typedef __attribute__((ext_vector_type(2))) unsigned short us2;
  constexpr uint32_t INF = __is_same(TIn, f16_t) ? 0x7c00u : 0x7f80u;
  __shared__ uint32_t most[16][8];
  __shared__ int cnt[8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = blockIdx.y;
  const int r = tid & 7, row = blockIdx.x * 8 + r;
  const TIn* src = O + ((size_t)b * N + min(row, N - 1)) * D;
  const int runs = row < N ? D / 16 : 0;
  uint4 in[ITER][2];
#pragma unroll
  for (int i = 0; i < ITER; i++) {
    const int c = (tid >> 3) + 128 * i;
    in[i][0] = in[i][1] = uint4{0, 0, 0, 0};
    if (c < runs) {
      in[i][0] = *reinterpret_cast<const uint4*>(src + c * 16);
      in[i][1] = *reinterpret_cast<const uint4*>(src + c * 16 + 8);
    }
  }
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < ITER; i++) {
    const uint32_t w[8] = {in[i][0].x, in[i][0].y, in[i][0].z, in[i][0].w, in[i][1].x, in[i][1].y, in[i][1].z, in[i][1].w};
#pragma unroll
    for (int k = 0; k < 8; k++) m = max(m, max(w[k] & 0x7fffu, (w[k] >> 16) & 0x7fffu));
  }
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
  if (lane < 8) most[wave][lane] = m;
  if (tid < 8) cnt[tid] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; k++) m = max(m, most[k][r]);
  int s = 0;
  if (m != 0 && m < INF) {
    int ex;
    const float mant = frexpf(widen1<TIn>(m), &ex);  // [0.5, 1): at most 11 bits, so that 2^31 of it is a whole number
    s = (int)ldexpf(mant, 31) > 0x7f7f7f7f ? 30 - ex : 31 - ex;  // 0x7f7f7f7f: the largest number of four signed digits
  }
  const bool finite = m < INF;
  uint16_t* list = left + ((size_t)b * Np + row) * ROW_LIST;
  // x 2^s of a value from here on is a whole number, whatever its last bits; the few smaller ones are looked at
  constexpr int BITS = __is_same(TIn, f16_t) ? 10 : 7;  // of the stored significand
  const uint32_t sure = least_bits<TIn>(BITS - s);
  us2 least = {0xffff, 0xffff};
#pragma unroll
  for (int i = 0; i < ITER; i++) {
    const uint32_t w[8] = {in[i][0].x, in[i][0].y, in[i][0].z, in[i][0].w, in[i][1].x, in[i][1].y, in[i][1].z, in[i][1].w};
#pragma unroll
    for (int k = 0; k < 8; k++)  // (a zero becomes the largest)
      least = __builtin_elementwise_min(least, __builtin_bit_cast(us2, w[k] & 0x7fff7fffu) - us2{1, 1});
  }
  if (finite && min((uint32_t)least.x, (uint32_t)least.y) + 1 < sure) {
#pragma unroll
    for (int i = 0; i < ITER; i++) {
      const uint32_t w[8] = {in[i][0].x, in[i][0].y, in[i][0].z, in[i][0].w, in[i][1].x, in[i][1].y, in[i][1].z, in[i][1].w};
      uint32_t off = 0;
#pragma unroll
      for (int k = 0; k < 8; k++) {
        float lo, hi;
        unpack2<TIn>(w[k], &lo, &hi);
        int q;
        off |= (whole(lo, s, &q) ? 0u : 1u) << (2 * k) | (whole(hi, s, &q) ? 0u : 2u) << (2 * k);
      }
      while (off) {
        const int k = __ffs(off) - 1, at = atomicAdd(&cnt[r], 1);
        off &= off - 1;
        if (at >= ROW_LIST) break;  // the row is formed anew
        list[at] = (uint16_t)(((tid >> 3) + 128 * i) * 16 + k);
      }
    }
  }
  __syncthreads();
  const int n = cnt[r];
  const bool anew = !finite || n > ROW_LIST;
  if (tid < 8) {  // (row is the thread's own)
    if (n > 1 && n <= ROW_LIST)  // ascending, so that sums over the list have one order
      for (int i = 1; i < n; i++) {
        const uint16_t v = list[i];
        int k = i;
        for (; k > 0 && list[k - 1] > v; k--) list[k] = list[k - 1];
        list[k] = v;
      }
    rowinfo[(size_t)b * Np + row] = s * 16 + (anew ? ROW_WHOLE : n);
    int over = anew ? 1 << 16 : n;
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) over += __shfl_xor(over, o, 64);
    if (tid == 0) left_over[(size_t)b * (Np / 8) + blockIdx.x] = over;
  }
  int n_anew = 0;
#pragma unroll
  for (int k = 0; k < 8; k++) n_anew += __shfl(anew ? 1 : 0, k, 64);
  if (n_anew == 8) return;  // (lines of 128 bytes, filled by the eight rows together: written in part they take longer)
  char* dst = P + ((size_t)b * (Np / 32) + row / 32) * (D / 32) * 4096 + (row & 31) * 16;
#pragma unroll
  for (int i = 0; i < ITER; i++) {
    const int c = (tid >> 3) + 128 * i;
    if (c >= D / 16) break;
    const uint32_t w[8] = {in[i][0].x, in[i][0].y, in[i][0].z, in[i][0].w, in[i][1].x, in[i][1].y, in[i][1].z, in[i][1].w};
    i4 out[4];
#pragma unroll
    for (int g = 0; g < 4; g++) {  // four columns: their 16 digits, turned
      uint32_t t[4];
#pragma unroll
      for (int k = 0; k < 4; k++) {
        float lo, hi;
        unpack2<TIn>(w[2 * g + k / 2], &lo, &hi);
        int q;
        if (!whole(k & 1 ? hi : lo, s, &q)) q = 0;
        t[k] = ((uint32_t)q + 0x00808080u) ^ 0x00808080u;
      }
      const uint32_t a01 = __builtin_amdgcn_perm(t[1], t[0], 0x05010400u), b01 = __builtin_amdgcn_perm(t[1], t[0], 0x07030602u);
      const uint32_t a23 = __builtin_amdgcn_perm(t[3], t[2], 0x05010400u), b23 = __builtin_amdgcn_perm(t[3], t[2], 0x07030602u);
      out[0][g] = (int)__builtin_amdgcn_perm(a23, a01, 0x05040100u);
      out[1][g] = (int)__builtin_amdgcn_perm(a23, a01, 0x07060302u);
      out[2][g] = (int)__builtin_amdgcn_perm(b23, b01, 0x05040100u);
      out[3][g] = (int)__builtin_amdgcn_perm(b23, b01, 0x07060302u);
    }
#pragma unroll
    for (int d = 0; d < 4; d++) *reinterpret_cast<i4*>(dst + (size_t)(c >> 1) * 4096 + d * 1024 + (c & 1) * 512) = out[d];
  }
}

// One workgroup: a 64x64 tile (ti >= tj), mirrored; a wavefront one quadrant, its seven sums in registers.  A chunk of 64
// columns comes to LDS without passing through registers, goes from there to registers as a whole, and the next chunk's copy
// runs while the matrix cores work on it; two workgroups share a compute unit.  64 images of 576 x 4096: 0.555 ms, 2.8 P operations/s
// (three workgroups, with half of a chunk in registers at a time: 0.562; 8 images of 2880 1.64 and 1.74 ms).
__global__ __launch_bounds__(256, 2) void gram_slices_kernel(const char* __restrict__ P, const int32_t* __restrict__ rowinfo,
                                                             const int32_t* __restrict__ left_over, double* __restrict__ G, int N, int KB,
                                                             int Np, int B) {
  __shared__ __attribute__((aligned(16))) char L[32768];  // [row blocks of A, of B][2 blocks of 32 columns][digit][1 KB]
  const int ntile = Np / 64;
  int b, t;
  if (!group_on_xcd(blockIdx.x, ntile * (ntile + 1) / 2, B, &b, &t)) return;
  if (too_much(image_left(left_over + (size_t)b * (Np / 8), Np), N, KB * 32)) return;
  int ti = 0;
  while (t >= ti + 1) { t -= ti + 1; ti++; }
  const int tj = t;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  const bool diag = ti == tj, idle = diag && wave == 1;  // (the mirror of wavefront 2's quadrant)
  const int rb = (wave < 2 ? 2 * ti : 2 * tj) + (wave & 1);  // the row block this wavefront copies
  const char* src = P + ((size_t)b * (Np / 32) + rb) * KB * 4096 + lane * 16;
  auto copy = [&](int kb) {
    if (diag && wave >= 2) return;
#pragma unroll
    for (int i = 0; i < 8; i++)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + (size_t)kb * 4096 + i * 1024),
                                       (__attribute__((address_space(3))) void*)(L + wave * 8192 + i * 1024), 16, 0, 0);
  };
  i16v acc[7];
#pragma unroll
  for (int c = 0; c < 7; c++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[c][r] = 0;
  const char* la = L + wr * 8192 + lane * 16;
  const char* lb = L + (diag ? wc : 2 + wc) * 8192 + lane * 16;
  copy(0);
  for (int kb = 0; kb < KB; kb += 2) {  // (D is a multiple of 64)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's copies have landed ...
    __syncthreads();                                  // ... and everyone's
    i4 fa[2][4], fb[2][4];
    if (!idle) {
#pragma unroll
      for (int h = 0; h < 2; h++)
#pragma unroll
        for (int d = 0; d < 4; d++) {
          fa[h][d] = *reinterpret_cast<const i4*>(la + h * 4096 + d * 1024);
          fb[h][d] = *reinterpret_cast<const i4*>(lb + h * 4096 + d * 1024);
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();  // the chunk is in registers: its place is free
    if (kb + 2 < KB) copy(kb + 2);
    if (idle) continue;
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int x = 0; x < 4; x++)
#pragma unroll
        for (int y = 0; y < 4; y++)
          acc[x + y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[h][x], fb[h][y], acc[x + y], 0, 0, 0);
  }
  if (idle) return;
  double* Gb = G + (size_t)b * Np * Np;
  const int32_t* info = rowinfo + (size_t)b * Np;
  const int r0 = ti * 64 + wr * 32 + 4 * (lane >> 5), col = tj * 64 + wc * 32 + (lane & 31);
  const int sc = row_scale(info[col]);
#pragma unroll
  for (int g = 0; g < 4; g++) {  // four rows side by side
    d4 v;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int r = 4 * g + k, row = r0 + 8 * g + k;
      const long long hi = ((long long)acc[6][r] << 16) + ((long long)acc[5][r] << 8) + acc[4][r];
      const long long lo = ((long long)acc[3][r] << 24) + ((long long)acc[2][r] << 16) + ((long long)acc[1][r] << 8) + acc[0][r];
      // hi below 2^44, lo below 2^53 (2^39.003 a column at most; only from 16352 columns on it could pass): one rounding
      const double x = fma((double)hi, 4294967296.0, (double)lo);
      v[k] = ldexp(x, -(sc + row_scale(info[row])));
      Gb[(size_t)row * Np + col] = v[k];
    }
    if (!diag || wave == 2) *reinterpret_cast<d4*>(&Gb[(size_t)col * Np + r0 + 8 * g]) = v;
  }
}

// What the digits leave out, in float64: of rows with a few values left the products of those, rows with more anew.  64 columns
// of an image are shared by sixteen wavefronts that do not wait for one another: each takes every sixteenth of the rows with values
// left, and four columns of the others, four of these at a time.  An entry of G and its mirror have one writer: of two rows with
// values left the first.  The products of a value left read a column of O, 64 lines: an image stays on one XCD, and the loads of
// a row are issued together.  (One workgroup for the 64 columns, a value's loads one after the other, the rows anew one by one:
// 576 values 412 us, 1152 715, 18 rows 860, by the figures at too_much.)
template <typename TIn>
__global__ __launch_bounds__(256, 4) void gram_rows_kernel(const TIn* __restrict__ O, const int32_t* __restrict__ rowinfo,
                                                        const uint16_t* __restrict__ left, double* __restrict__ G,
                                                        const int32_t* __restrict__ left_over, int N, int D, int Np, int B) {
  int b, t;
  if (!group_on_xcd(blockIdx.x, Np / 64 * 4, B, &b, &t)) return;
  const int lane = threadIdx.x & 63, col0 = t / 4 * 64, wave = __builtin_amdgcn_readfirstlane(t % 4 * 4 + (threadIdx.x >> 6));
  const Left image = image_left(left_over + (size_t)b * (Np / 8), Np);
  if ((image.values | image.anew) == 0 || too_much(image, N, D)) return;
  const int32_t* info = rowinfo + (size_t)b * Np;
  const uint16_t* lists = left + (size_t)b * Np * ROW_LIST;
  const TIn* Ob = O + (size_t)b * N * D;
  double* Gb = G + (size_t)b * Np * Np;
  auto bits = [&](int row, int k) { return bits16(Ob[(size_t)row * D + k]); };
  auto of = [](const uint32_t* list, int i) { return (list[i / 2] >> (16 * (i & 1))) & 0xffff; };

  if (image.values > 0) {
    const int col = col0 + lane, cn = col < N ? row_left(info[col]) : ROW_WHOLE;
    const bool listed = cn > 0 && cn != ROW_WHOLE;
    int most = 0;  // values of a column's own list
    uint32_t lc[4] = {0, 0, 0, 0}, oc[ROW_LIST];
#pragma unroll
    for (int i = 0; i < ROW_LIST; i++) {
      if (__ballot(listed && cn > i)) most = i + 1;
      oc[i] = 0;
    }
    if (listed) {
      const uint4 v = *reinterpret_cast<const uint4*>(lists + (size_t)col * ROW_LIST);
      lc[0] = v.x; lc[1] = v.y; lc[2] = v.z; lc[3] = v.w;
#pragma unroll
      for (int i = 0; i < ROW_LIST; i++)
        if (i < cn) oc[i] = bits(col, of(lc, i));
    }
    for (int r0 = wave; r0 < N; r0 += 1024) {
      const int mine = r0 + 16 * lane, rl = mine < N ? row_left(info[mine]) : 0;
      for (unsigned long long rows = __ballot(rl > 0 && rl != ROW_WHOLE); rows; rows &= rows - 1) {
        const int at = __ffsll(rows) - 1, row = r0 + 16 * at, rn = __builtin_amdgcn_readlane(rl, at);
        if (cn == ROW_WHOLE || (listed && col < row)) continue;  // formed anew, or the other row's entry
        const uint4 v = *reinterpret_cast<const uint4*>(lists + (size_t)row * ROW_LIST);
        const uint32_t lr[4] = {v.x, v.y, v.z, v.w};
        const double g = Gb[(size_t)row * Np + col];
        uint32_t x[ROW_LIST], y[ROW_LIST], z[ROW_LIST];
        double add = 0.0;
#pragma unroll
        for (int i = 0; i < ROW_LIST; i++) {  // (rn and most are the same in every lane)
          if (i < rn) {
            x[i] = bits(row, of(lr, i));
            y[i] = bits(col, of(lr, i));
          }
          if (i < most) z[i] = i < cn ? bits(row, of(lc, i)) : 0;
        }
#pragma unroll
        for (int i = 0; i < ROW_LIST; i++)
          if (i < rn) add = fma((double)widen1<TIn>(x[i]), (double)widen1<TIn>(y[i]), add);
#pragma unroll
        for (int i = 0; i < ROW_LIST; i++)
          if (i < most) {  // of the column's own those that the row's list does not hold
            bool both = i >= cn;
#pragma unroll
            for (int j = 0; j < ROW_LIST; j++) both |= j < rn && of(lr, j) == of(lc, i);
            if (!both) add = fma((double)widen1<TIn>(z[i]), (double)widen1<TIn>(oc[i]), add);
          }
        Gb[(size_t)row * Np + col] = g + add;
        if (row != col) Gb[(size_t)col * Np + row] = g + add;
      }
    }
  }

  if (image.anew == 0) return;
  const int c0 = col0 + wave * 4;
  unsigned long long rows = 0;
  for (int r0 = -64;;) {
    int row[4] = {0, 0, 0, 0}, n = 0;
    while (n < 4) {
      while (!rows && r0 + 64 < N) {
        r0 += 64;
        rows = __ballot(r0 + lane < N && row_left(info[r0 + lane]) == ROW_WHOLE);
      }
      if (!rows) break;
#pragma unroll
      for (int i = 0; i < 4; i++) if (i == n) row[i] = r0 + __ffsll(rows) - 1;
      rows &= rows - 1;
      n++;
    }
    if (n == 0) return;
    double sum[4][4];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int c = 0; c < 4; c++) sum[i][c] = 0.0;
    for (int k = lane * 8; k < D; k += 512) {
      uint32_t x[4][4], y[4][4];
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const uint4 v = fetch8<TIn>(Ob + (size_t)(i < n ? row[i] : row[0]) * D + k).v;
        x[i][0] = v.x; x[i][1] = v.y; x[i][2] = v.z; x[i][3] = v.w;
      }
#pragma unroll
      for (int c = 0; c < 4; c++) {
        const uint4 v = fetch8<TIn>(Ob + (size_t)min(c0 + c, N - 1) * D + k).v;
        y[c][0] = v.x; y[c][1] = v.y; y[c][2] = v.z; y[c][3] = v.w;
      }
#pragma unroll
      for (int u = 0; u < 4; u++) {
        float lo[4], hi[4];
#pragma unroll
        for (int c = 0; c < 4; c++) unpack2<TIn>(y[c][u], &lo[c], &hi[c]);
#pragma unroll
        for (int i = 0; i < 4; i++) {
          if (i >= n) break;
          float xl, xh;
          unpack2<TIn>(x[i][u], &xl, &xh);
#pragma unroll
          for (int c = 0; c < 4; c++) {
            sum[i][c] = fma((double)xl, (double)lo[c], sum[i][c]);
            sum[i][c] = fma((double)xh, (double)hi[c], sum[i][c]);
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int c = 0; c < 4; c++) {
        const double v = wave_sum_dpp(sum[i][c]);
        if (lane == 0 && i < n && c0 + c < N) {  // (of two such rows both write the same value)
          Gb[(size_t)row[i] * Np + c0 + c] = v;
          Gb[(size_t)(c0 + c) * Np + row[i]] = v;
        }
      }
  }
}

// Digits for 16-bit rows of calls with work for the chip.  A tile is a chain of D / 64 chunks (0.85 us each) by one workgroup, where
// gram_kernel shares a small call's tiles, and an image of one tile has a fourth of it idle in gram_kernel but not here.  All
// launches of the step, float64 and digits, us: D = 4096, 64 images of 64 tokens 47 and 79, 256 of them 144 and 164; 27 of 128
// (81 tiles) 66 and 87, 48 (144) 98 and 89; 10 of 256 (100) 79 and 91; where the parts leave three workgroups or fewer to a tile, one
// image of 576 (45) 65 and 77, two (90) 111 and 79; one of 2880 717 and 275; D = 1024, 64 of 128 (192) 40 and 40, 20 of 256 (200)
// 49 and 41.  By the size of the whole call, as for the parts.  A float32 matrix (TC_EIG_F32) keeps gram_kernel: the values that are
// added apart would find the digits' part already rounded to float32, and round it again.
constexpr int FEWEST_TILES = 80, MANY_TILES = 128;  // (the latter where gram_kernel shares a tile among more than three)
constexpr long long LEAST_WORK = 200000;
int gram_splits(const Plan& pl);
static long long call_tiles(const Plan& pl) {
  const long long nt = pl.Np / 64;
  return nt * (nt + 1) / 2 * pl.batch_call;
}
static bool may_use_slices(const Plan& pl) {
  return pl.esize == 2 && pl.tsize == 8 && pl.D <= 16384 && pl.Np > 64 && call_tiles(pl) >= FEWEST_TILES && call_tiles(pl) * pl.D >= LEAST_WORK;
}
static bool use_slices(const Plan& pl) {
  return may_use_slices(pl) && call_tiles(pl) >= (gram_splits(pl) > 3 ? MANY_TILES : FEWEST_TILES);
}
// Room for the digits of the images that a turn takes, 4 bytes an element; the images of a call beyond that go in turns.
constexpr size_t TURN_BYTES = (size_t)1 << 30;
static size_t slice_bytes(const Plan& pl) { return (size_t)pl.Np * pl.D * 4; }
static int turn_images(const Plan& pl) { return slice_bytes(pl) < TURN_BYTES ? (int)(TURN_BYTES / slice_bytes(pl)) : 1; }
// A workspace also serves calls of fewer tokens and images, so it has this room where one of them may take this way (with fewer
// tiles none does): up to a turn.
void gram_slice_reserve(const Plan& pl, size_t* digits, size_t* rows) {
  const size_t all = slice_bytes(pl) * pl.B, most = slice_bytes(pl) > TURN_BYTES ? slice_bytes(pl) : TURN_BYTES;
  *digits = may_use_slices(pl) ? (all < most ? all : most) : 0;
  *rows = may_use_slices(pl) ? (size_t)pl.B * pl.Np : 0;
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
static size_t gram_part_bytes(const Plan& pl) { return part_bytes(pl, gram_splits(pl)); }
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
static void run_gram(const Plan& pl, const void* O, void* G, void* ws, int img0, hipStream_t st) {
  const int nt = pl.Np / 64, tiles = nt * (nt + 1) / 2, splits = gram_splits(pl);
  if constexpr (sizeof(TIn) == 2 && sizeof(TOut) == 8) {
    if (use_slices(pl)) {
      char* P = at<char>(ws, pl.off_gslice);  // (stream groups form their matrices one after the other)
      int32_t* info = at<int32_t>(ws, pl.off_grow) + (size_t)img0 * pl.Np;
      uint16_t* left = at<uint16_t>(ws, pl.off_gleft) + (size_t)img0 * pl.Np * ROW_LIST;
      int32_t* left_over = at<int32_t>(ws, pl.off_gover) + (size_t)img0 * (pl.Np / 8);
      const auto slice = pl.D <= 2048 ? gram_slice_kernel<TIn, 1> : pl.D <= 4096 ? gram_slice_kernel<TIn, 2> : (pl.D <= 8192 ? gram_slice_kernel<TIn, 4> : gram_slice_kernel<TIn, 8>);
      const int turns = (pl.B + turn_images(pl) - 1) / turn_images(pl);
      for (int k = 0; k < turns; k++) {
        const int first = (int)((long long)pl.B * k / turns), n = (int)((long long)pl.B * (k + 1) / turns) - first;
        const TIn* Ok = (const TIn*)O + (size_t)first * pl.N * pl.D;
        double* Gk = (double*)G + (size_t)first * pl.Np * pl.Np;
        int32_t* ik = info + (size_t)first * pl.Np;
        int32_t* ok = left_over + (size_t)first * (pl.Np / 8);
        TC_TIMED(PK_GRAM, 2, st, (slice<<<dim3(pl.Np / 8, n), 1024, 0, st>>>(Ok, P, ik, left + (size_t)first * pl.Np * ROW_LIST, ok, pl.N, pl.D, pl.Np)));
        TC_TIMED(PK_GRAM, 0, st, (gram_slices_kernel<<<grid_for_groups(tiles, n), 256, 0, st>>>(P, ik, ok, Gk, pl.N, pl.D / 32, pl.Np, n)));
      }
      TC_TIMED(PK_GRAM, 3, st, (gram_rows_kernel<TIn><<<grid_for_groups(nt * 4, pl.B), 256, 0, st>>>((const TIn*)O, info, left, (double*)G, left_over, pl.N, pl.D, pl.Np, pl.B)));
      TC_TIMED(PK_GRAM, 1, st, (gram_kernel<TIn, TOut><<<grid_for_groups(tiles, pl.B), 256, 0, st>>>((const TIn*)O, (TOut*)G, pl.N, pl.D, pl.Np, pl.B, 1, nullptr, left_over)));
      return;
    }
  }
  double* part = at<double>(ws, pl.off_gpart) + img0 * (gram_part_bytes(pl) / 8);
  TC_TIMED(PK_GRAM, 0, st, (gram_kernel<TIn, TOut><<<grid_for_groups(tiles * splits, pl.B), 256, 0, st>>>((const TIn*)O, (TOut*)G, pl.N, pl.D, pl.Np, pl.B, splits, part, nullptr)));
  if (splits > 1) TC_TIMED(PK_GRAM, 1, st, (gram_sum_kernel<TOut><<<dim3(tiles, pl.B), 256, 0, st>>>(part, (TOut*)G, pl.Np, splits)));
}

// O and G of the images img0 .. img0 + pl.B - 1 of the call; the scratch is the call's.
int launch_gram(const Plan& pl, int dtype, int eig_dtype, const void* O, void* G, void* ws, int img0, hipStream_t st) {
  const bool f64 = eig_dtype == TC_EIG_F64;
  if (dtype == TC_BF16) f64 ? run_gram<uint16_t, double>(pl, O, G, ws, img0, st) : run_gram<uint16_t, float>(pl, O, G, ws, img0, st);
  else if (dtype == TC_F16) f64 ? run_gram<f16_t, double>(pl, O, G, ws, img0, st) : run_gram<f16_t, float>(pl, O, G, ws, img0, st);
  else f64 ? run_gram<float, double>(pl, O, G, ws, img0, st) : run_gram<float, float>(pl, O, G, ws, img0, st);
  return check_launch();
}

}  // namespace tc

// For the tests, no part of the interface: the Gram step of a call on rows O by itself, G [B, Np, Np]; `digits` (host): whether
// the call takes the digits.  Without O nothing is launched.
extern "C" __attribute__((visibility("default"))) int tc_gram_matrix(const tc_params* p, const void* O, void* G, void* ws, size_t ws_bytes,
                                                                     void* stream, int* digits) {
  tc::Plan pl;
  int rc = tc::make_plan(p, &pl);
  if (rc != TC_OK) return rc;
  *digits = tc::use_slices(pl) ? 1 : 0;
  if (!O) return TC_OK;
  if ((rc = tc::check_ws(pl, ws, ws_bytes)) != TC_OK) return rc;
  return tc::launch_gram(pl, p->dtype, p->eig_dtype, O, G, ws, 0, (hipStream_t)stream);
}
