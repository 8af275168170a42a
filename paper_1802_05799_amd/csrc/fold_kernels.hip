// The whole ring in one launch, over flat rank buffers (fold_flat_kernel) or over the
// tensors of a table (fold_table_kernel).  fold.hpp has the wavefront's work and why it
// has this shape.

#include <type_traits>

#include "fold.hpp"

namespace hvdx {
namespace {

// ---- flat rank buffers ---------------------------------------------------------------
//
// Block row y is chunk y, whose stretches are the chunk's pieces of the buffer's grid of
// 64*V elements, so that every whole stretch is 1 KiB aligned when the buffers are.  The
// rank pointers are listed twice over, so that a ring's ranks from any first rank on are one
// run of them (scalar loads, several per instruction).

// Loads are non-temporal: nothing read is read again, and a launch on data that no cache holds is
// 5 to 15% faster so.  Cached ones keep data that fits the Infinity Cache in it from one call on
// the same buffers to the next; on buffers another kernel has just written the two are alike (us,
// non-temporal and cached, 128 MiB in all: on 2 ranks repeated 42.3 and 32.8, from memory 43.2 and
// 49.2, just written 44.0 and 42.3; on 8 ranks 47.3 and 37.3, 49.0 and 51.9, 42.6 and 42.6).  So a
// caller can ask for them (`cached`): hvdx_fold_allreduce and the ring of 2 ranks, which were one
// launch with cached loads before all rings were, and would lose on repeated calls.  Up to a
// little over the cache's 256 MiB (2 ranks, 272 MiB: 88.1 and 74.9, 304: 98.1 and 103.5).
constexpr int64_t kCachedBytes = 272ll << 20;

struct RingPtrs {
  void* p[2 * HVDX_MAX_RANKS + kFoldPad];
};

template <typename TT, typename TB, bool CACHED, int B>
__global__ __launch_bounds__(kFoldLanes, fold_waves(B)) void fold_flat_kernel(RingPtrs bufs, RingArgs a, int mode, bool aligned) {
  constexpr int64_t S = kFoldLanes * FoldTypes<TT, TB>::V;
  const int c = blockIdx.y;
  const Chunk ch = chunk_of(c, a);
  const int64_t end = ch.start + ch.len;
  for (int64_t g = ch.start / S + blockIdx.x; g * S < end; g += gridDim.x) {
    const int64_t e0 = g * S > ch.start ? g * S : ch.start;
    const int64_t e1 = (g + 1) * S < end ? (g + 1) * S : end;
    auto ptr = [&](int k) { return static_cast<TT*>(bufs.p[c + k]) + e0; };
    const bool al = aligned && e0 % FoldTypes<TT, TB>::V == 0;
    fold_stretch<TT, TB, CACHED, B>(ptr, a, mode, (int)(e1 - e0), al, 0);
  }
}

// ---- the tensors of a table -------------------------------------------------------------
//
// One block per stretch of a tile of the table, which lists every
// tensor's ranks twice over, too.  The table is read as constant memory: read as plain
// memory, a store's pointer is a vector load behind the store before it, and a wavefront's N
// stores go out one round trip apart (ResNet-50 on 8 ranks 265 us, 256 so; Inception-V3 on 16 510,
// 486; VGG-16 on 32 6.20 ms, 5.98, in both the bursts and the wavefronts that suit it best).

constexpr int64_t kFoldRow = 1 << 22;  // blocks in a row of the grid, when there are more than one row

template <typename TT, typename TB, int B>
__global__ __launch_bounds__(kFoldLanes, fold_waves(B)) void fold_table_kernel(FoldTable t, RingArgs a, int mode) {
  constexpr int S = kFoldLanes * FoldTypes<TT, TB>::V;
  const int64_t b = (int64_t)blockIdx.y * kFoldRow + blockIdx.x;
  const bool wide = t.stretches != 1;
  if (b >= t.ntiles * t.stretches) return;
  typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
  const i32x4 w = constant(reinterpret_cast<const i32x4*>(t.tiles))[wide ? b / kFoldWide : b];  // a FoldTile in one load
  const uint32_t bits = (uint32_t)w[3];
  const auto p = constant(t.ptrs) + (int64_t)w[2] * 2 * a.n + (bits >> 16 & 0xff);
  const int part = wide ? (int)(b % kFoldWide) * S : 0;
  const int left = (int)(bits & 0xffff) - part;
  if (left <= 0) return;
  const int64_t li = ((int64_t)w[1] << 32 | (uint32_t)w[0]) + part;
  auto ptr = [&](int k) { return static_cast<TT*>(p[k]) + li; };
  fold_stretch<TT, TB, false, B>(ptr, a, mode, left < S ? left : S, bits >> 24 & 1, (int)(bits >> 28));
}

// Whether to hold the wavefronts per CU down (fold_lds).  Not in a launch so short that filling the
// chip is what counts (TB/s held and not: 8 ranks of 1M binary32 elements 4.69, 4.96; of 3M 5.46,
// 5.44; of 6M 5.87, 5.45; 16 ranks of 0.3M 3.65, 4.06; of 1.5M 5.31, 5.13; 32 of 1.5M 5.36, 5.02; 4
// of 3M 5.19, 5.30).  And not where more than 1/8 of the blocks have little to move (short tensors,
// each cut into N chunks; Inception-V3's tensors reduced one by one on 16 ranks have 4% more blocks
// than whole stretches: 510 us held, 552 not; with 21% more it was 605 and 580).
bool fold_holds(int64_t blocks, int64_t count, int nranks, int tensor_dtype) {
  const int64_t bytes = count * (tensor_dtype == HVDX_FLOAT16 ? 2 : 4);
  const int64_t filled = bytes / (kFoldLanes * 16);
  return bytes > (96ll << 20) / nranks && blocks <= filled + filled / 8;
}

// Calls f(TT{}, TB{}, integral_constant<burst>) for the launch's types and burst.
template <typename TT, typename TB, typename F>
void with_burst(int burst, const F& f) {
  switch (burst) {
#define HVDX_BURST(B) \
  case B: return f(TT{}, TB{}, std::integral_constant<int, B>{});
    HVDX_BURST(2) HVDX_BURST(3) HVDX_BURST(4) HVDX_BURST(5) HVDX_BURST(6) HVDX_BURST(7) HVDX_BURST(8) HVDX_BURST(9)
    HVDX_BURST(10) HVDX_BURST(11) HVDX_BURST(12) HVDX_BURST(13) HVDX_BURST(14) HVDX_BURST(15)
#undef HVDX_BURST
    default: return f(TT{}, TB{}, std::integral_constant<int, 16>{});
  }
}
template <typename F>
void with_types(int tensor_dtype, int buf_dtype, int burst, const F& f) {
  if (tensor_dtype == HVDX_FLOAT16) with_burst<_Float16, _Float16>(burst, f);
  else if (buf_dtype == HVDX_FLOAT16) with_burst<float, _Float16>(burst, f);
  else with_burst<float, float>(burst, f);
}

}  // namespace

hipError_t launch_fold_flat(const RankPtrs& bufs, const RingArgs& a, int tensor_dtype, int buf_dtype, int divmode,
                            bool aligned, bool cached, hipStream_t stream) {
  if (a.n == 1 && tensor_dtype == buf_dtype) return hipSuccess;  // the buffer is its own sum
  const int64_t span = kFoldLanes * (tensor_dtype == HVDX_FLOAT16 ? 8 : 4);
  int64_t bx = (a.q + (a.rem ? 1 : 0)) / span + 2;  // a chunk may begin and end inside a stretch
  if (bx > (1 << 22)) bx = 1 << 22;
  const dim3 grid((unsigned)bx, (unsigned)a.n);
  const int burst = fold_burst(a.n);
  const unsigned lds = fold_holds(bx * a.n, a.q * a.n + a.rem, a.n, tensor_dtype) ? fold_lds(a.n, burst) : 0;
  RingPtrs ptrs{};  // the pad is read, if not used
  for (int r = 0; r < a.n; ++r) ptrs.p[r] = ptrs.p[a.n + r] = bufs.p[r];
  const int64_t bytes = (a.q * a.n + a.rem) * a.n * (tensor_dtype == HVDX_FLOAT16 ? 2 : 4);
  cached = cached && bytes <= kCachedBytes;
  with_types(tensor_dtype, buf_dtype, burst, [&](auto tt, auto tb, auto b) {
    if (cached)
      HVDX_LAUNCH((fold_flat_kernel<decltype(tt), decltype(tb), true, b.value>), grid, dim3(kFoldLanes), lds, stream,
                  ptrs, a, divmode, aligned);
    else
      HVDX_LAUNCH((fold_flat_kernel<decltype(tt), decltype(tb), false, b.value>), grid, dim3(kFoldLanes), lds, stream,
                  ptrs, a, divmode, aligned);
  });
  return hipGetLastError();
}

hipError_t launch_fold_table(const FoldTable& t, const RingArgs& a, int64_t count, int tensor_dtype, int buf_dtype,
                             int divmode, hipStream_t stream) {
  const int64_t blocks = t.ntiles * t.stretches;
  const int64_t bx = blocks < kFoldRow ? blocks : kFoldRow;
  const dim3 grid((unsigned)bx, (unsigned)((blocks + bx - 1) / bx));
  const int burst = fold_burst(a.n);
  const unsigned lds = fold_holds(blocks, count, a.n, tensor_dtype) ? fold_lds(a.n, burst) : 0;
  with_types(tensor_dtype, buf_dtype, burst, [&](auto tt, auto tb, auto b) {
    HVDX_LAUNCH((fold_table_kernel<decltype(tt), decltype(tb), b.value>), grid, dim3(kFoldLanes), lds, stream, t, a,
                divmode);
  });
  return hipGetLastError();
}

}  // namespace hvdx
