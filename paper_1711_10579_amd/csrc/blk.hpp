// 2x2 blocks of the Jacobian (row-major [a b; c d]) and their arithmetic,
// shared by the factor and Krylov kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace pfd {

// Pointers into device (global) memory.  Memory reached through the
// instance descriptors is otherwise accessed through generic pointers, whose
// loads the compiler issues as flat loads; flat loads are also counted by the
// LDS wait counter, so every LDS wait or barrier would wait for them too.
#define PF_AS1 __attribute__((address_space(1)))
template <typename T>
__device__ inline PF_AS1 T* gp(T* p) {
  return (PF_AS1 T*)p;
}
template <typename T>
__device__ inline const PF_AS1 T* gp(const T* p) {
  return (const PF_AS1 T*)p;
}

// work item i of a list of (instance, index) pairs, through a global pointer
__device__ inline int2 ld_item(const int2* work, int i) {
  const auto wp = (const PF_AS1 int*)work;
  return make_int2(wp[2 * i], wp[2 * i + 1]);
}

// Bound of an in-launch wait in ticks of the device's constant real-time
// counter (100 MHz): about one second.
constexpr unsigned long long kWaitTicks = 100000000ull;
__device__ inline unsigned long long rt_now() { return __builtin_amdgcn_s_memrealtime(); }
// s_waitcnt vmcnt(0): every vector memory access of the wave, stores
// included, has completed
__device__ inline void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Device-coherent accesses for data handed between work-groups inside a
// launch: relaxed atomics at agent scope (stores write through, loads bypass
// the caches that are not coherent across the device), issued as global
// (not generic) accesses so that they are counted by the vector-memory wait
// counter alone and LDS waits do not wait for them.  p points to device
// memory.
template <typename T>
__device__ inline T ld_dev(const T* p) {
  return __hip_atomic_load((const PF_AS1 T*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline void st_dev(T* p, T v) {
  __hip_atomic_store((PF_AS1 T*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Work-groups of a launch are handed to the device's eight XCDs (each with
// its own L2) in turn.  xcd_block(b, G) renumbers block b of a grid of G so
// that each XCD takes one contiguous range of the renumbered blocks: data
// that neighbouring blocks share is then fetched into one L2, not eight.
// A permutation of [0, G).
__device__ inline int xcd_block(int b, int G) {
  constexpr int kXcd = 8;
  const int c = G / kXcd, rem = G % kXcd;
  const int x = b % kXcd, k = b / kXcd;
  return x < rem ? x * (c + 1) + k : rem * (c + 1) + (x - rem) * c + k;
}

// four ints as a native vector (loadable through any address space)
typedef int i4v __attribute__((ext_vector_type(4)));

template <typename T>
struct Blk {
  T a, b, c, d;  // [[a b] [c d]]
};

template <typename T, typename Ptr>
__device__ inline Blk<T> ld_blk_as(Ptr p, int64_t id) {
  const auto q = p + 4 * id;
  Blk<T> r;
  r.a = q[0];
  r.b = q[1];
  r.c = q[2];
  r.d = q[3];
  return r;
}

template <typename T>
__device__ inline Blk<T> ld_blk(const PF_AS1 T* p, int64_t id) {
  return ld_blk_as<T>(p, id);
}

template <typename T>
__device__ inline void st_blk(PF_AS1 T* p, int64_t id, const Blk<T>& v) {
  PF_AS1 T* q = p + 4 * id;
  q[0] = v.a;
  q[1] = v.b;
  q[2] = v.c;
  q[3] = v.d;
}

template <typename T>
__device__ inline Blk<T> ld_blk(const T* p, int64_t id) {
  const T* q = p + 4 * id;
  Blk<T> r;
  r.a = q[0];
  r.b = q[1];
  r.c = q[2];
  r.d = q[3];
  return r;
}

template <typename T>
__device__ inline void st_blk(T* p, int64_t id, const Blk<T>& v) {
  T* q = p + 4 * id;
  q[0] = v.a;
  q[1] = v.b;
  q[2] = v.c;
  q[3] = v.d;
}

template <typename T>
__device__ inline Blk<double> blk_f64(const Blk<T>& v) {
  return {(double)v.a, (double)v.b, (double)v.c, (double)v.d};
}

// The block operations name their fused multiply-adds: a column is formed by
// different kernels alone and in a batch, and left to the compiler each could
// fuse another product of a sum (results must agree to the bit).

// a - (x y + z w)
template <typename T>
__device__ inline T sub2(T a, T x, T y, T z, T w) {
  return fma(-x, y, fma(-z, w, a));
}

// acc -= X * Y
template <typename T>
__device__ inline void blk_msub(Blk<T>& acc, const Blk<T>& X, const Blk<T>& Y) {
  acc.a = sub2(acc.a, X.a, Y.a, X.b, Y.c);
  acc.b = sub2(acc.b, X.a, Y.b, X.b, Y.d);
  acc.c = sub2(acc.c, X.c, Y.a, X.d, Y.c);
  acc.d = sub2(acc.d, X.c, Y.b, X.d, Y.d);
}

// the determinant of a 2x2 block
template <typename T>
__device__ inline T blk_det(const Blk<T>& m) {
  return fma(m.a, m.d, -(m.b * m.c));
}

template <typename T>
__device__ inline Blk<T> blk_mul(const Blk<T>& X, const Blk<T>& Y) {
  Blk<T> r;
  r.a = fma(X.a, Y.a, X.b * Y.c);
  r.b = fma(X.a, Y.b, X.b * Y.d);
  r.c = fma(X.c, Y.a, X.d * Y.c);
  r.d = fma(X.c, Y.b, X.d * Y.d);
  return r;
}

// inverse of a 2x2 block (determinant in FP64); false when it is zero or
// not finite
template <typename T>
__device__ inline bool blk_inv(const Blk<T>& m, Blk<T>* out) {
  const double det = (double)m.a * (double)m.d - (double)m.b * (double)m.c;
  if (!(det != 0.0) || !isfinite(det)) return false;
  const double id = 1.0 / det;
  out->a = (T)((double)m.d * id);
  out->b = (T)(-(double)m.b * id);
  out->c = (T)(-(double)m.c * id);
  out->d = (T)((double)m.a * id);
  return true;
}

// The values a, b of this lane's group of OFF lanes and of the one beside it
// (lane ^ OFF), in either order, once all lanes of a group hold the same value
// (a butterfly taken from the smallest offset up): within rows of 16 lanes a
// mirror reaches the other group's lanes as well as an xor does, so these are
// data-parallel moves (a few cycles) and lane swaps, not LDS permutes (some
// 130 cycles a step)
template <int OFF>
__device__ inline int lane_other(int x) {
  if constexpr (OFF == 1) return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xf, 0xf, true);   // quad (1,0,3,2)
  if constexpr (OFF == 2) return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xf, 0xf, true);   // quad (2,3,0,1)
  if constexpr (OFF == 4) return __builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, true);  // half row mirrored
  return __builtin_amdgcn_mov_dpp(x, 0x140, 0xf, 0xf, true);                          // row mirrored
}
template <int OFF>
__device__ inline void lane_pair(int v, int& a, int& b) {
  if constexpr (OFF <= 8) {
    a = v;
    b = lane_other<OFF>(v);
  } else {
    const auto r = OFF == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false)
                             : __builtin_amdgcn_permlane32_swap(v, v, false, false);
    a = r[0];
    b = r[1];
  }
}
template <int OFF>
__device__ inline void lane_pair(float v, float& a, float& b) {
  int x, y;
  lane_pair<OFF>(__builtin_bit_cast(int, v), x, y);
  a = __builtin_bit_cast(float, x);
  b = __builtin_bit_cast(float, y);
}
template <int OFF>
__device__ inline void lane_pair(double v, double& a, double& b) {
  const int2 u = __builtin_bit_cast(int2, v);
  int2 x, y;
  lane_pair<OFF>(u.x, x.x, y.x);
  lane_pair<OFF>(u.y, x.y, y.y);
  a = __builtin_bit_cast(double, x);
  b = __builtin_bit_cast(double, y);
}
template <int OFF, typename T>
__device__ inline T lane_add(T v) {
  T a, b;
  lane_pair<OFF>(v, a, b);
  return a + b;
}
// sum over the G lanes of a group (G a power of two, groups aligned to G), in
// every lane of it
template <int G, typename T>
__device__ inline T group_add(T v) {
  if constexpr (G > 1) v = lane_add<1>(v);
  if constexpr (G > 2) v = lane_add<2>(v);
  if constexpr (G > 4) v = lane_add<4>(v);
  if constexpr (G > 8) v = lane_add<8>(v);
  if constexpr (G > 16) v = lane_add<16>(v);
  if constexpr (G > 32) v = lane_add<32>(v);
  return v;
}
template <int OFF, typename T>
__device__ inline Blk<T> blk_lane_add(const Blk<T>& v) {
  return {lane_add<OFF>(v.a), lane_add<OFF>(v.b), lane_add<OFF>(v.c), lane_add<OFF>(v.d)};
}

// the same of a block, G known only when the kernel runs (uniform)
template <typename T>
__device__ inline Blk<T> group_sum_rt(Blk<T> v, int G) {
  if (G > 1) v = blk_lane_add<1>(v);
  if (G > 2) v = blk_lane_add<2>(v);
  if (G > 4) v = blk_lane_add<4>(v);
  if (G > 8) v = blk_lane_add<8>(v);
  if (G > 16) v = blk_lane_add<16>(v);
  if (G > 32) v = blk_lane_add<32>(v);
  return v;
}
template <typename T, int G>
__device__ inline Blk<T> group_sum(const Blk<T>& v) {
  return group_sum_rt(v, G);
}

// Marker of a solution entry not yet computed: a signalling NaN with a fixed
// payload.  Arithmetic never produces a signalling NaN (its NaN results are
// quiet) and the inputs are finite, so a stored solution value never has
// these bits.
template <typename T>
struct Unsolved;
template <>
struct Unsolved<double> {
  typedef unsigned long long U;
  static constexpr U bits = 0x7FF4DEADBEEFCAFEull;
};
template <>
struct Unsolved<float> {
  typedef unsigned int U;
  static constexpr U bits = 0x7FA5DEADu;
};
template <typename T>
__device__ inline bool unsolved(T v) {
  return __builtin_bit_cast(typename Unsolved<T>::U, v) == Unsolved<T>::bits;
}
template <typename T>
__device__ inline T unsolved_value() {
  return __builtin_bit_cast(T, Unsolved<T>::bits);
}

}  // namespace pfd
