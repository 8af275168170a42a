// The whole ring in one launch, over flat rank buffers (fold_flat_kernel) or over the
// tensors of a table (fold_table_kernel).  fold.hpp has the wavefront's work and why it
// has this shape.

#include "fold.hpp"

namespace hvdx {
namespace {

// ---- flat rank buffers ---------------------------------------------------------------
//
// Block row y is chunk y, whose stretches are the chunk's pieces of the buffer's grid of
// 64*V elements, so that every whole stretch is 1 KiB aligned when the buffers are.  The
// rank pointers are listed twice over, so that a ring's ranks from any first rank on are one
// run of them (scalar loads, several per instruction).

struct RingPtrs {
  void* p[2 * HVDX_MAX_RANKS];
};

template <typename TT, typename TB, int DIV, int B>
__global__ __launch_bounds__(kFoldLanes, fold_waves(B)) void fold_flat_kernel(RingPtrs bufs, RingArgs a, bool aligned) {
  constexpr int64_t S = kFoldLanes * FoldTypes<TT, TB>::V;
  const int c = blockIdx.y;
  const Chunk ch = chunk_of(c, a);
  const int64_t end = ch.start + ch.len;
  for (int64_t g = ch.start / S + blockIdx.x; g * S < end; g += gridDim.x) {
    const int64_t e0 = g * S > ch.start ? g * S : ch.start;
    const int64_t e1 = (g + 1) * S < end ? (g + 1) * S : end;
    auto ptr = [&](int k) { return static_cast<TT*>(bufs.p[c + k]) + e0; };
    const bool al = aligned && e0 % FoldTypes<TT, TB>::V == 0;
    fold_stretch<TT, TB, DIV, B>(ptr, a, (int)(e1 - e0), al);
  }
}

// ---- the tensors of a table -------------------------------------------------------------
//
// kFoldParts blocks per tile of the table, one per 64*V elements of it; the table lists
// every tensor's ranks twice over, too.

constexpr int64_t kFoldRow = 1 << 22;  // blocks in a row of the grid, when there are more than one row

template <typename TT, typename TB, int DIV, int B>
__global__ __launch_bounds__(kFoldLanes, fold_waves(B)) void fold_table_kernel(FoldTable t, RingArgs a) {
  constexpr int S = kFoldLanes * FoldTypes<TT, TB>::V;
  const int64_t b = (int64_t)blockIdx.y * kFoldRow + blockIdx.x;
  if (b >= t.ntiles * kFoldParts) return;
  typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
  const i32x4 w = reinterpret_cast<const i32x4*>(t.tiles)[b / kFoldParts];  // a FoldTile in one load
  const uint32_t bits = (uint32_t)w[3];
  const int part = (int)(b % kFoldParts) * S;
  const int left = (int)(bits & 0xffff) - part;
  if (left <= 0) return;
  void* const* p = t.ptrs + (int64_t)w[2] * 2 * a.n + (bits >> 16 & 0xff);
  const int64_t li = ((int64_t)w[1] << 32 | (uint32_t)w[0]) + part;
  auto ptr = [&](int k) { return static_cast<TT*>(p[k]) + li; };
  fold_stretch<TT, TB, DIV, B>(ptr, a, left < S ? left : S, bits >> 24);
}

// Blocks at or below which the wavefronts per CU are left alone: with no more than that the
// chip is not full, and what counts is that every block is resident at once.
constexpr int64_t kFoldFewBlocks = 256 * 16;

#define HVDX_FOLD_BURST(F, TT, TB, DIV) \
  if (burst == 8) F(TT, TB, DIV, 8); else if (burst == 16) F(TT, TB, DIV, 16); else F(TT, TB, DIV, 32)
#define HVDX_FOLD_DIV(F, TT, TB) \
  if (divmode == DIV_NONE) { HVDX_FOLD_BURST(F, TT, TB, DIV_NONE); } \
  else if (divmode == DIV_POW2) { HVDX_FOLD_BURST(F, TT, TB, DIV_POW2); } \
  else { HVDX_FOLD_BURST(F, TT, TB, DIV_TRUE); }
#define HVDX_FOLD_ALL(F) \
  if (tensor_dtype == HVDX_FLOAT16) { HVDX_FOLD_DIV(F, _Float16, _Float16) } \
  else if (buf_dtype == HVDX_FLOAT16) { HVDX_FOLD_DIV(F, float, _Float16) } \
  else { HVDX_FOLD_DIV(F, float, float) }

}  // namespace

hipError_t launch_fold_flat(const RankPtrs& bufs, const RingArgs& a, int tensor_dtype, int buf_dtype, int divmode,
                            bool aligned, hipStream_t stream) {
  if (a.n == 1 && tensor_dtype == buf_dtype) return hipSuccess;  // the buffer is its own sum
  const int64_t span = kFoldLanes * (tensor_dtype == HVDX_FLOAT16 ? 8 : 4);
  int64_t bx = (a.q + (a.rem ? 1 : 0)) / span + 2;  // a chunk may begin and end inside a stretch
  if (bx > (1 << 22)) bx = 1 << 22;
  const dim3 grid((unsigned)bx, (unsigned)a.n);
  const int burst = fold_burst(a.n);
  const unsigned lds = bx * a.n <= kFoldFewBlocks ? 0 : fold_lds(a.n);
  RingPtrs ptrs;
  for (int r = 0; r < a.n; ++r) ptrs.p[r] = ptrs.p[a.n + r] = bufs.p[r];
#define HVDX_FLAT(TT, TB, DIV, B) \
  HVDX_LAUNCH((fold_flat_kernel<TT, TB, DIV, B>), grid, dim3(kFoldLanes), lds, stream, ptrs, a, aligned)
  HVDX_FOLD_ALL(HVDX_FLAT)
#undef HVDX_FLAT
  return hipGetLastError();
}

hipError_t launch_fold_table(const FoldTable& t, const RingArgs& a, int tensor_dtype, int buf_dtype, int divmode,
                             hipStream_t stream) {
  const int64_t blocks = t.ntiles * kFoldParts;
  const int64_t bx = blocks < kFoldRow ? blocks : kFoldRow;
  const dim3 grid((unsigned)bx, (unsigned)((blocks + bx - 1) / bx));
  const int burst = fold_burst(a.n);
  const unsigned lds = blocks <= kFoldFewBlocks ? 0 : fold_lds(a.n);
#define HVDX_TABLE(TT, TB, DIV, B) \
  HVDX_LAUNCH((fold_table_kernel<TT, TB, DIV, B>), grid, dim3(kFoldLanes), lds, stream, t, a)
  HVDX_FOLD_ALL(HVDX_TABLE)
#undef HVDX_TABLE
  return hipGetLastError();
}

}  // namespace hvdx
