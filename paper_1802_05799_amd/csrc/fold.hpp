// The whole ring of a stretch of elements in one wavefront, the messages in registers.
//
// An element's ring never involves another element, so a lane can run all 2(N-1) steps of
// its elements by itself: the partial sum that rank c+s would send in adding step s is the
// lane's accumulator, rank c+s+1's own value is added to it, and the replacing steps store
// the finished value to every rank.  Same order of additions and same roundings as the
// per-step kernels, so the same bits, for 2N elements moved instead of 5N-6.
//
// Bound: HBM, N read and N write streams at once.  What the shape has to get right is how
// much is in flight.  Measured on MI355X (N buffers, in place, binary32):
//   256-thread blocks, full occupancy, 4 loads in flight per lane   4.9 TB/s (N=8), 4.9 (N=32)
//   one wavefront per block, the loads in whole bursts              5.85 (N=8), 5.2 (N=16, 32)
//   the same with 6 (N=8), 4 (N=16) or 2 (N=32) wavefronts per CU   6.36, 6.22, 6.0
// (one stream in place: 6.55).  More in flight only spreads the accesses to an HBM page
// apart in time: some 24 to 40 KiB of loads per CU is best, and the stores, which wait for
// nothing, follow at once.  A wavefront that goes on to a second tile loses 10-20%: loads and
// stores share one in-order counter, so its next loads wait behind its own stores.  Hence one
// wavefront per block, one 16-byte vector per lane and rank, its loads in whole bursts, the
// stores, and the end; an LDS reservation no one uses holds the wavefronts per CU down.
#pragma once

#include <algorithm>

#include "ring_math.hpp"

namespace hvdx {
namespace {

constexpr int kFoldLanes = 64;

// 16-byte vectors that need only their elements' alignment.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef _Float16 f16x8u __attribute__((ext_vector_type(8), aligned(2)));

// Tensors of type TT, sums in type TB: a lane's vector, the same without its alignment, the
// accumulator, and the conversions (binary32 tensors summed in binary16 are rounded where
// first read and widened exactly where stored).
template <typename TT, typename TB>
struct FoldTypes;
template <>
struct FoldTypes<float, float> {
  using vec = f32x4;
  using uvec = f32x4u;
  using acc = f32x4;
  static constexpr int V = 4;
  __device__ static acc in(vec v) { return v; }
  __device__ static vec out(acc v) { return v; }
};
template <>
struct FoldTypes<_Float16, _Float16> {
  using vec = f16x8;
  using uvec = f16x8u;
  using acc = f16x8;
  static constexpr int V = 8;
  __device__ static acc in(vec v) { return v; }
  __device__ static vec out(acc v) { return v; }
};
template <>
struct FoldTypes<float, _Float16> {
  using vec = f32x4;
  using uvec = f32x4u;
  using acc = f16x4;
  static constexpr int V = 4;
  __device__ static acc in(vec v) {
    acc h;
#pragma unroll
    for (int k = 0; k < 4; ++k) h[k] = (_Float16)v[k];
    return h;
  }
  __device__ static vec out(acc h) {
    vec v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (float)h[k];
    return v;
  }
};

// The AVERAGE divide of a finished sum (mode: one DivMode for the whole launch).
__device__ __forceinline__ float finish_one(float s, const RingArgs& a, int mode) {
  return mode == DIV_NONE ? s : mode == DIV_POW2 ? finish<DIV_POW2>(s, a) : finish<DIV_TRUE>(s, a);
}
__device__ __forceinline__ _Float16 finish_one(_Float16 s, const RingArgs& a, int mode) {
  return mode == DIV_NONE ? s : mode == DIV_POW2 ? finish16<DIV_POW2>(s, a) : finish16<DIV_TRUE>(s, a);
}
template <int V, typename A>
__device__ __forceinline__ A finish_vec(A s, const RingArgs& a, int mode) {
  if (mode == DIV_POW2) {
#pragma unroll
    for (int k = 0; k < V; ++k) s[k] = finish_one(s[k], a, DIV_POW2);
  } else if (mode == DIV_TRUE) {
#pragma unroll
    for (int k = 0; k < V; ++k) s[k] = finish_one(s[k], a, DIV_TRUE);
  }
  return s;
}

// The same number, which the compiler cannot tell: a burst's loads and its additions test it
// separately, and joining the two tests would copy the code for every length.
__device__ __forceinline__ int same_count(int v) {
  asm("" : "+s"(v));
  return v;
}

// A pointer every lane has alike, read where this stands: the compiler would otherwise read
// each behind the test of its own load, one memory round trip after the other.
template <typename T>
__device__ __forceinline__ T* uniform_here(T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<T*>((uint64_t)hi << 32 | lo);
}

template <bool CACHED, typename P>
__device__ __forceinline__ auto fold_load(P p) {
  if constexpr (CACHED) return *p;
  else return __builtin_nontemporal_load(p);
}

// One vector per lane.  ptr(k) is the address of the stretch's first element on the k-th
// rank of its ring (rank c+k mod N).  The last burst reads, but does not use, up to ptr(n+B-2):
// with the ring's ranks from rank c on, entry c+n+B-2 <= 2n+B-3 of a list of 2n; MT is
// FoldTypes::vec or, unaligned, ::uvec.
template <typename TT, typename TB, bool CACHED, int B, typename MT, typename Ptr>
__device__ __forceinline__ void fold_vectors(const Ptr& ptr, const RingArgs& a, int mode) {
  static_assert(B - 2 <= kFoldPad, "a list of 2n rank pointers is followed by kFoldPad more");
  using F = FoldTypes<TT, TB>;
  using vec = typename F::vec;
  const unsigned off = threadIdx.x * 16u;  // unsigned: a scalar base and a 32-bit offset per access
  typename F::acc s = (typename F::acc)((TB)-0.0f);  // x + -0 = x for every x
  auto at = [&](TT* p) { return (Global<MT>)((Global<char>)p + off); };
  const int n = a.n;
  int k0 = 0;
#pragma unroll 1
  for (; k0 + B <= n; k0 += B) {  // whole bursts, no test between the loads
    vec x[B];
#pragma unroll
    for (int j = 0; j < B; ++j) x[j] = fold_load<CACHED>(at(ptr(k0 + j)));
    __builtin_amdgcn_sched_barrier(0);  // no addition, and so no wait, before the last load is out
#pragma unroll
    for (int j = 0; j < B; ++j) s = F::in(x[j]) + s;
  }
  if (k0 < n) {  // the rest in one more
    vec x[B];
    TT* p[B];
    const int left = n - k0, adds = same_count(left);
#pragma unroll
    for (int j = 0; j < B; ++j) p[j] = uniform_here(ptr(k0 + j));
#pragma unroll
    for (int j = 0; j < B; ++j)
      if (j < left) x[j] = fold_load<CACHED>(at(p[j]));
#pragma unroll
    for (int j = 0; j < B; ++j)
      if (j < adds) s = F::in(x[j]) + s;
  }
  const MT o = F::out(finish_vec<F::V>(s, a, mode));
#pragma unroll 4
  for (int k = 0; k < n; ++k) __builtin_nontemporal_store(o, at(ptr(k)));
}

// The same for one element per lane: the elements past a stretch's last whole vector.  Loads
// past the last rank repeat its own.
template <typename TT, typename TB, typename Ptr>
__device__ __forceinline__ void fold_element(const Ptr& ptr, const RingArgs& a, int mode, int e) {
  constexpr int B = 8;
  const int n = a.n;
  TB s = (TB)-0.0f;
#pragma unroll 1
  for (int k0 = 0; k0 < n; k0 += B) {
    TT x[B];
#pragma unroll
    for (int j = 0; j < B; ++j) x[j] = ((Global<TT>)ptr(k0 + j < n ? k0 + j : n - 1))[e];
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const TB sum = (TB)x[j] + s;
      s = k0 + j < n ? sum : s;
    }
  }
  const TT o = (TT)finish_one(s, a, mode);
#pragma unroll 1
  for (int k = 0; k < n; ++k) ((Global<TT>)ptr(k))[e] = o;
}

// Both at once, for a stretch with whole vectors (vecs >= 1, from element `head` on) and single
// elements (rest >= 1: the `head` before the vectors, then those past them): one after the other
// the second's loads would wait behind the first's stores (with that, and what precedes the first
// 16-byte boundary in a wavefront of its own, Inception-V3's tensors reduced one by one on 16 ranks
// 565 us, 510 so).  Lanes past the last vector or element
// load that one too, and store nothing.
template <typename TT, typename TB, bool CACHED, int B, typename MT, typename Ptr>
__device__ __forceinline__ void fold_edges(const Ptr& ptr, const RingArgs& a, int mode, int head, int vecs, int rest) {
  using F = FoldTypes<TT, TB>;
  const int n = a.n, lane = threadIdx.x;
  const int i = lane < rest ? lane : rest - 1;
  const unsigned voff = head * (unsigned)sizeof(TT) + (lane < vecs ? lane : vecs - 1) * 16u;
  const unsigned eoff = (i < head ? i : vecs * F::V + i) * (unsigned)sizeof(TT);
  auto vector = [&](TT* p) { return (Global<MT>)((Global<char>)p + voff); };
  auto element = [&](TT* p) { return (Global<TT>)((Global<char>)p + eoff); };
  typename F::acc s = (typename F::acc)((TB)-0.0f);
  TB t = (TB)-0.0f;
#pragma unroll 1
  for (int k0 = 0; k0 < n; k0 += B) {
    typename F::vec x[B];
    TT y[B];
#pragma unroll
    for (int j = 0; j < B; ++j) {
      TT* p = ptr(k0 + j < n ? k0 + j : n - 1);
      x[j] = fold_load<CACHED>(vector(p));
      y[j] = *element(p);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < B; ++j)
      if (k0 + j < n) {
        s = F::in(x[j]) + s;
        t = (TB)y[j] + t;
      }
  }
  const MT o = F::out(finish_vec<F::V>(s, a, mode));
  const TT u = (TT)finish_one(t, a, mode);
  if (lane < vecs) {
#pragma unroll 4
    for (int k = 0; k < n; ++k) __builtin_nontemporal_store(o, vector(ptr(k)));
  }
  if (lane < rest) {
#pragma unroll 4
    for (int k = 0; k < n; ++k) *element(ptr(k)) = u;
  }
}

// A wavefront's stretch of m (1 .. 64*V) elements; aligned: its element `head` (< V) lies on a
// 16-byte boundary of every rank (head is 0 if not).
template <typename TT, typename TB, bool CACHED, int B, typename Ptr>
__device__ __forceinline__ void fold_stretch(const Ptr& ptr, const RingArgs& a, int mode, int m, bool aligned,
                                             int head) {
  using F = FoldTypes<TT, TB>;
  const int lane = threadIdx.x;
  if (head > m) head = m;
  const int vecs = (m - head) / F::V, rest = m - vecs * F::V;
  if (vecs && rest) {
    if (aligned) fold_edges<TT, TB, CACHED, B, typename F::vec>(ptr, a, mode, head, vecs, rest);
    else fold_edges<TT, TB, CACHED, B, typename F::uvec>(ptr, a, mode, head, vecs, rest);
  } else if (lane < vecs) {
    if (aligned) fold_vectors<TT, TB, CACHED, B, typename F::vec>(ptr, a, mode);
    else fold_vectors<TT, TB, CACHED, B, typename F::uvec>(ptr, a, mode);
  } else if (lane < rest) {
    fold_element<TT, TB>(ptr, a, mode, lane);
  }
}

// Wavefronts per SIMD that the registers of a burst have to leave room for.
constexpr int fold_waves(int burst) { return burst <= 8 ? 4 : 3; }

// Host side: the loads of a burst for n ranks (one instantiation each), and the wavefronts per CU
// that go with it, as Inception-V3's binary32 tensors measure them (TB/s; a:b is bursts of a with
// b wavefronts).  Every burst but the last should be a whole one of up to 16: a shorter one tests
// before each load, and more registers than that leave too few wavefronts to small launches.
//   7 ranks  7:6 6.44, 4:10 6.39          16  8:4 6.25, 16:3 6.11, 4:6 6.19, 16:8 5.77
//   8        4:6 6.37, 8:5 6.26, 8:8 6.20 24  12:3 6.09, 8:3 6.06, 16:2 5.59
//   12       6:5 6.32, 12:3 6.25          40  10:3 5.81, 8:3 5.77, 16:2 5.52
//   13       7:5 6.21, 13:3 6.28          64  16:2 5.64, 8:3 5.63, 16:4 5.46 (rounded to binary16)
// So: all ranks below 8; halves up to 24 ranks; then the longest of 16 to 10 that divides n, else
// near-equal ones of up to 12 (33 ranks: 11:3 5.90, 16:2 5.39).
inline int fold_burst(int n) {
  if (n < 8) return n < 2 ? 2 : n;
  if (n <= 24) return (n + 1) / 2;
  for (int b = 16; b >= 10; --b)
    if (n % b == 0) return b;
  const int bursts = (n + 11) / 12;
  return (n + bursts - 1) / bursts;
}

// LDS bytes per block that hold the wavefronts per CU down: all ranks' loads in one burst like some
// 36 loads in flight per CU (3 ranks 12 wavefronts 6.41, 16 6.32; 4: 10 6.38, 16 6.29; 6: 6 6.49,
// 10 6.34), several bursts some 28, in at most 6 wavefronts (VGG-16 on 32 ranks 16:2 5.90, 16:3
// 5.46, 16:6 5.31).  2 ranks like all there is (6.39; 6.24 with 16).
inline unsigned fold_lds(int n, int burst) {
  if (burst < 3) return 0;
  const int waves = burst == n ? (36 + burst - 1) / burst : std::min(6, (28 + burst - 1) / burst);
  return (160u << 10) / waves / 512 * 512 - 512;
}

}  // namespace
}  // namespace hvdx
