// Common to the kernels of the reduction to tridiagonal form (tridiag.hip, tridiag_columns.hip): exchange between workgroups,
// waits, scalars, order of the launches.
#pragma once
#include <utility>

#include "tc_internal.h"
#include "tridiag_frames.h"

namespace tc {

typedef unsigned long long u64;

// The turn of a launch with groups of P, each on one XCD (local) or spread over them, in a call that has groups of sixteen or not
// (tridiag.hip): taken before the launch, over with done(), which is called after it in any case.
struct TrTurn {
  int rc, first = 0;      // status; number of the first XCD
  bool captured, apart;   // the stream is being captured; the launch is kept apart from others
  TrTurn(int P, bool local, int images, bool sixteen, int xcds, hipStream_t st);
  int done();
 private:
  int unit(int i) const { return TR_PLACES * ((first + i / places) % xcds) + from + i % places; }
  int count = 0, places = 1, from = 0, event = 0, dev = 0, xcds;
  hipStream_t st;
};

constexpr int TD_SPIN = 1 << 22;  // polls before a wait is given up (seconds; a wait in good order is a microsecond)

// The lowest bit makes room for the tag by rounding to nearest even, and a reader clears the tag: zero arrives as zero.
__device__ __forceinline__ u64 tagged(double v, unsigned tag) {
  const u64 y = (u64)__double_as_longlong(v);
  return ((y + ((y >> 1) & 1)) & ~1ull) | tag;
}
__device__ __forceinline__ void publish(u64* p, double v, unsigned tag) {
  __hip_atomic_store(p, tagged(v, tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double received(u64 y) { return __longlong_as_double((long long)(y & ~1ull)); }
__device__ __forceinline__ u64 peek(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True when a wait has to end: it has lasted for TD_SPIN polls, or another workgroup of the image has given up.
__device__ __forceinline__ bool tr_give_up(int spin, const int32_t* fail) {
  return spin >= TD_SPIN ||
         ((spin & 1023) == 1023 && __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0);
}

// The members of a group count themselves in.  True when the group is not complete after `patience` polls (at once where that
// is negative): the first member to find that out sets the top bit, which nobody does once the count is whole, so all
// members decide alike, those too that get their compute unit later.
__device__ __forceinline__ bool tr_stranded(u64* arrived, u64 P, int patience, u64 counter = ~(1ull << 63), u64* all = nullptr) {
  constexpr u64 off = 1ull << 63;
  if (patience < 0) return true;
  for (int spin = 0;; spin++) {
    u64 n = peek(arrived);
    if (n & off) return true;
    if ((n & counter) >= P) {
      if (all) *all = n;
      return false;
    }
    if (spin >= patience &&
        __hip_atomic_compare_exchange_strong(arrived, &n, n | off, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return true;
  }
}

// f(a), f(a + 1), ... f(n - 1) with the index as a constant.
template <int a, int n, typename F>
__device__ __forceinline__ void walk_up(F f) {
  [&]<int... i>(std::integer_sequence<int, i...>) { (f(std::integral_constant<int, a + i>{}), ...); }(std::make_integer_sequence<int, n - a>{});
}

__device__ __forceinline__ double sum8(const double* r) {
  return ((r[0] + r[1]) + (r[2] + r[3])) + ((r[4] + r[5]) + (r[6] + r[7]));
}

// 1 / x and 1 / sqrt(x) to the last bit or so: hardware estimate and Newton steps (a library division is 73 cycles of
// dependent instructions, a square root 105, and a column waits for two of them)
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ double fast_rsq(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// The index as a value that the compiler knows nothing about.
template <bool on>
__device__ __forceinline__ void fresh(int& x) { if (on) asm volatile("" : "+v"(x)); }

}  // namespace tc
