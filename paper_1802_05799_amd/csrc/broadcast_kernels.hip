// Broadcast chain step: in step s the link from rank root+k to rank root+k+1
// carries chunk s-k (paper sections 4 and 5: variables broadcast from one process
// to all).  Block row y is link k; every link whose chunk index is in range copies
// that chunk's bytes with 16-byte vectors, the short last unit byte by byte.
#include "ring_math.hpp"

namespace hvdx {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kUnits = 2;  // 16-byte units per lane per pass

template <bool VEC_OK>
__global__ __launch_bounds__(kBlock) void bcast_step_kernel(RankPtrs bufs, BcastArgs a) {
  const int k = blockIdx.y;
  const int64_t j = (int64_t)a.step - k;
  if (j < 0 || j >= a.n) return;
  const int src = (a.root + k) % a.n;
  const int dst = (src + 1) % a.n;
  const int64_t u0 = j * a.q + (j < a.rem ? j : a.rem);
  const int64_t units = a.q + (j < a.rem ? 1 : 0);
  const int64_t lo = u0 * 16 < a.nbytes ? u0 * 16 : a.nbytes;
  const int64_t hi = (u0 + units) * 16 < a.nbytes ? (u0 + units) * 16 : a.nbytes;
  const unsigned char* __restrict__ s = static_cast<const unsigned char*>(bufs.p[src]);
  unsigned char* __restrict__ d = static_cast<unsigned char*>(bufs.p[dst]);
  const int64_t full = VEC_OK ? (hi - lo) / 16 : 0;  // whole units in the chunk
  const int64_t gtid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t gthreads = (int64_t)gridDim.x * kBlock;
  const u32x4* __restrict__ s4 = reinterpret_cast<const u32x4*>(s + lo);
  u32x4* __restrict__ d4 = reinterpret_cast<u32x4*>(d + lo);
  for (int64_t base = (int64_t)blockIdx.x * kBlock * kUnits + threadIdx.x; base < full;
       base += gthreads * kUnits) {
    u32x4 v[kUnits];
#pragma unroll
    for (int u = 0; u < kUnits; ++u)
      if (base + u * kBlock < full) v[u] = __builtin_nontemporal_load(s4 + base + u * kBlock);
#pragma unroll
    for (int u = 0; u < kUnits; ++u)
      if (base + u * kBlock < full) __builtin_nontemporal_store(v[u], d4 + base + u * kBlock);
  }
  for (int64_t e = lo + full * 16 + gtid; e < hi; e += gthreads) d[e] = s[e];
}

// The whole chain in one launch: a wavefront takes one stretch of the buffer from the root and
// hands it to every other rank, the links' messages in registers: N bytes moved per byte where
// the chain's steps move 2(N-1).  The stretches are cut at multiples of their size of the first
// receiver's addresses, so that each is whole cache lines; a unit that would begin before the
// buffer or end after it is moved as the buffer's first or last 16 bytes (the bytes its
// neighbour moves too are the same).
typedef unsigned int u32x4u __attribute__((ext_vector_type(4), aligned(1)));

template <int U>
__global__ __launch_bounds__(64) void bcast_kernel(RankPtrs bufs, BcastArgs a, int shift) {
  constexpr int V = 16, R = 8;
  const int64_t p0 = ((int64_t)blockIdx.y * kBcastRow + blockIdx.x) * (64 * U * V) - shift;
  const int others = a.n - 1;
  const auto src = (Global<unsigned char>)bufs.p[a.root];
  auto dst = [&](int i) {  // in chain order
    const int r = a.root + 1 + (i < others ? i : others - 1);
    return (Global<unsigned char>)bufs.p[r < a.n ? r : r - a.n];
  };
  if (a.nbytes < V) {  // one block
    const int e = threadIdx.x;
    if (p0 > 0 || e >= a.nbytes) return;
    const unsigned char x = src[e];
    for (int i = 0; i < others; ++i) dst(i)[e] = x;
    return;
  }
  u32x4 x[U];
  int64_t e[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    e[u] = p0 + (int64_t)(u * 64 + threadIdx.x) * V;
    if (e[u] >= a.nbytes || e[u] <= -V) e[u] = -1;  // outside
    else e[u] = e[u] < 0 ? 0 : e[u] + V > a.nbytes ? a.nbytes - V : e[u];
    if (e[u] >= 0) x[u] = __builtin_nontemporal_load((Global<u32x4u>)(src + e[u]));
  }
  for (int i0 = 0; i0 < others; i0 += R) {
    Global<unsigned char> d[R];
#pragma unroll
    for (int i = 0; i < R; ++i) d[i] = dst(i0 + i);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (i0 + i >= others) break;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (e[u] >= 0) __builtin_nontemporal_store((u32x4u)x[u], (Global<u32x4u>)(d[i] + e[u]));
    }
  }
}

template <int U>
void bcast_launch(const RankPtrs& bufs, const BcastArgs& a, unsigned lds, hipStream_t stream) {
  const int64_t tile = 64 * U * 16;
  const int shift = a.nbytes < 16 ? 0 : (int)(reinterpret_cast<uintptr_t>(bufs.p[(a.root + 1) % a.n]) % tile);
  const int64_t blocks = (a.nbytes + shift + tile - 1) / tile;
  const int64_t bx = blocks < kBcastRow ? blocks : kBcastRow;
  HVDX_LAUNCH(bcast_kernel<U>, dim3((unsigned)bx, (unsigned)((blocks + bx - 1) / bx)), dim3(64), lds, stream, bufs, a,
              shift);
}

}  // namespace

hipError_t launch_bcast(const RankPtrs& bufs, const BcastArgs& a, hipStream_t stream) {
  const BcastShape s = bcast_shape(a.n, a.nbytes);
  if (s.units == 4) bcast_launch<4>(bufs, a, s.lds, stream);
  else if (s.units == 2) bcast_launch<2>(bufs, a, s.lds, stream);
  else bcast_launch<1>(bufs, a, s.lds, stream);
  return hipGetLastError();
}

hipError_t launch_bcast_step(const RankPtrs& bufs, const BcastArgs& a, bool vector_ok, hipStream_t stream) {
  const int64_t longest = a.q + (a.rem ? 1 : 0);
  int64_t bx = (longest + (int64_t)kBlock * kUnits - 1) / ((int64_t)kBlock * kUnits);
  if (bx < 1) bx = 1;
  if (bx > (1 << 20)) bx = 1 << 20;
  const dim3 grid((unsigned)bx, (unsigned)(a.n - 1));
  if (vector_ok)
    HVDX_LAUNCH((bcast_step_kernel<true>), grid, dim3(kBlock), 0, stream, bufs, a);
  else
    HVDX_LAUNCH((bcast_step_kernel<false>), grid, dim3(kBlock), 0, stream, bufs, a);
  return hipGetLastError();
}

}  // namespace hvdx
