// Internal declarations shared by the library's translation units (not installed).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "hvdx.h"

namespace hvdx {

// Events that a timeline record hands to this thread's next kernel launch, which then
// runs through hipExtLaunchKernel: the dispatch itself stamps them with the kernel's
// start and end, with no extra commands in the stream.  Empty when nothing waits.
struct LaunchEvents {
  hipEvent_t start = nullptr, stop = nullptr;
};
LaunchEvents& pending_launch_events();

// Every rank's base pointer travels in the kernel arguments (1 KiB).
struct RankPtrs {
  void* p[HVDX_MAX_RANKS];
};

// Ring partition and step, identical for every block of one launch.
struct RingArgs {
  int n;          // ranks
  int step;       // 0 .. n-2
  int64_t q;      // count / n
  int64_t rem;    // count % n
  float nf;       // (float) n
  float inv;      // 1 / n, used only when n is a power of two
  int64_t wire_stride;  // elements per rank in the fp16 wire workspace
};

// The same step of two rings (two fusion buffers of one call) in one launch.
struct RingPair {
  RankPtrs bufs[2];
  RingArgs a[2];  // same n and step, each ring its own count
};

// The fused copy-in or copy-out of two fusion buffers in one launch.
struct CopyPair {
  void* const* t[2];  // DEVICE tables of tensor pointers, rank-major
  const int64_t* numel[2];
  const int64_t* offset[2];
  int ntensors[2];
  RankPtrs bufs[2];
  int64_t count[2], q[2], rem[2];  // buffer elements and their ring partition
};

// The fused copies of one or two fusion buffers driven by tile tables (hvdx_copy_tile):
// blocks [0, x0) take bucket 0's tiles, the rest bucket 1's.  A tile is at most
// kTileLanes * tile_vectors(...) vectors of tile_vec_elems(...) elements: the host cuts
// the tables and the kernels move them with the same constants.
constexpr int kTileLanes = 256;
#ifndef HVDX_TILE_U32
#define HVDX_TILE_U32 1  // binary32 tensors and buffers
#endif
#ifndef HVDX_TILE_U16  // binary32 tensors, binary16 buffers: one vector per lane.  Two make the copies of
#define HVDX_TILE_U16 1  // the paper's mode 3 points faster; the ring on the tensors is 1% faster with one
#endif
#ifndef HVDX_TILE_UH
#define HVDX_TILE_UH 1  // binary16 tensors and buffers
#endif
inline int tile_vec_elems(int tensor_dtype, int buf_dtype) {
  return tensor_dtype == HVDX_FLOAT32 || buf_dtype == HVDX_FLOAT32 ? 4 : 8;
}
inline int tile_vectors(int tensor_dtype, int buf_dtype) {
  if (tensor_dtype == HVDX_FLOAT32 && buf_dtype == HVDX_FLOAT32) return HVDX_TILE_U32;
  if (tensor_dtype == HVDX_FLOAT32) return HVDX_TILE_U16;
  return HVDX_TILE_UH;
}
struct TiledCopy {
  CopyPair m;  // tensors and buffers of the buckets (the partition fields are not used)
  const hvdx_copy_tile* tiles[2];
  int64_t x0;
};

// How the last adding step finishes an AVERAGE.
enum DivMode { DIV_NONE = 0, DIV_POW2 = 1, DIV_TRUE = 2 };

constexpr int kBlock = 256;

// Launchers (ring_kernels.hip).  Arguments are already validated; return a hipError_t.
hipError_t launch_rs_step(const RankPtrs& bufs, const RingArgs& a, int dtype, int divmode, bool vector_ok,
                          hipStream_t stream);
hipError_t launch_ag_step(const RankPtrs& bufs, const RingArgs& a, int dtype, bool vector_ok, hipStream_t stream);
hipError_t launch_rs_step_c16(const RankPtrs& x, void* wire, const RingArgs& a, int divmode, bool vector_ok,
                              hipStream_t stream);
hipError_t launch_ag_step_c16(const RankPtrs& x, void* wire, const RingArgs& a, bool vector_ok, hipStream_t stream);
hipError_t launch_roundtrip_c16(void* x, int64_t count, hipStream_t stream);
// Adding step N-2 and replacing step 0 in one launch.
hipError_t launch_rs_ag_step(const RankPtrs& bufs, const RingArgs& a, int dtype, int divmode, bool vector_ok,
                             hipStream_t stream);
hipError_t launch_rs_ag_step_c16(const RankPtrs& x, void* wire, const RingArgs& a, int divmode, bool vector_ok,
                                 hipStream_t stream);
// One step of two rings at once (binary32 or binary16 buffers, both 16-byte aligned):
// an adding step, adding step N-2 fused with replacing step 0, a replacing step.
hipError_t launch_rs_step_pair(const RingPair& m, int dtype, int divmode, hipStream_t stream);
hipError_t launch_rs_ag_step_pair(const RingPair& m, int dtype, int divmode, hipStream_t stream);
hipError_t launch_ag_step_pair(const RingPair& m, int dtype, hipStream_t stream);
// The copy-in fused with adding step 0 (no sender storing its own sent chunk), and
// replacing step N-2 fused with the copy-out, for two fusion buffers at once.
hipError_t launch_pack_pair(const CopyPair& m, int src_dtype, int buf_dtype, int nranks, hipStream_t stream);
hipError_t launch_unpack_pair(const CopyPair& m, int buf_dtype, int dst_dtype, int nranks, hipStream_t stream);
// The same two fused copies driven by tile tables, for one or two buckets: `blocks` tiles in
// all, each block one tile and one rank.
hipError_t launch_pack_tiles(const TiledCopy& k, int src_dtype, int buf_dtype, int nranks, int64_t blocks,
                             hipStream_t stream);
hipError_t launch_unpack_tiles(const TiledCopy& k, int buf_dtype, int dst_dtype, int nranks, int64_t blocks,
                               hipStream_t stream);
// The ring on the tensors of one to kRingBuckets fusion buffers, every launch serving
// all of them: the launch's tiles [end[i-1], end[i]) are bucket i's (from tiles[i]),
// bucket i's tensor pointer table is the DEVICE table t[i] (rank-major, ntensors[i] per
// rank), and its rank r fusion buffer is bufs[i * nranks + r].
constexpr int kRingBuckets = 4;
constexpr int kRingBufPtrs = 256;  // nbuckets * nranks at most
struct TiledRing {
  const hvdx_copy_tile* tiles[kRingBuckets];
  int64_t end[kRingBuckets];
  void* const* t[kRingBuckets];
  int64_t ntensors[kRingBuckets];
  int nbuckets;
  int nranks;
  void* bufs[kRingBufPtrs];
};

// Replacing steps that deliver into the tensors, over the copy-out's tiles: adding step
// N-2 with replacing step 0 (own_in_tensors: the owner's value from its tensors), and
// replacing step s between the tensors.
hipError_t launch_rs_ag_tiles(const TiledRing& k, const RingArgs& a, int tensor_dtype, int buf_dtype, int divmode,
                              bool own_in_tensors, hipStream_t stream);
hipError_t launch_ag_tiles(const TiledRing& k, int tensor_dtype, int buf_dtype, int step, hipStream_t stream);
// Adding step s (0 .. N-3) reading every receiver's own values from its tensors (and at
// s = 0 the sender's too), over the copy-in's tiles.
hipError_t launch_add_tiles(const TiledRing& k, int tensor_dtype, int buf_dtype, int step, hipStream_t stream);
// A small fusion buffer's copy-in, ring and copy-out in one launch.
hipError_t launch_small_cycle(const void* const* tensors, const int64_t* numel, const int64_t* offset, int ntensors,
                              int tensor_dtype, const RingArgs& a, int64_t count, int buf_dtype, int divmode,
                              hipStream_t stream);

// The whole ring in one launch (fold_kernels.hip): each lane runs every step for its elements,
// the messages in registers.  Over flat rank buffers (a holds their partition), with cached loads
// where asked for and the buffers fit the Infinity Cache:
hipError_t launch_fold_flat(const RankPtrs& bufs, const RingArgs& a, int tensor_dtype, int buf_dtype, int divmode,
                            bool aligned, bool cached, hipStream_t stream);
// ... and over the tensors of a table, where a tile is at most 64 16-byte vectors of one tensor in one
// ring chunk, a wavefront's stretch, or kFoldWide times that.  Wide tiles leave blocks with nothing
// to do at each piece's end, and need a tile of its own for what precedes a piece's first 16-byte
// boundary; narrow ones are four times the table, which wavefronts on different XCDs each fetch from
// memory.  So narrow where pieces are shorter than 64 stretches on average (us wide and narrow:
// Inception-V3's tensors one by one on 16 ranks, 20 stretches to a piece, 565 and 510; in fusion
// buffers, over 100, 486 and 491; ResNet-50 on 8 ranks 256 and 257).
constexpr int kFoldWide = 4;
inline int fold_stretches(int64_t stretches, int64_t pieces) { return stretches < 64 * pieces ? 1 : kFoldWide; }
struct alignas(16) FoldTile {
  int64_t li;      // the tile's first element in its tensor
  int32_t tensor;
  uint32_t bits;   // elements, the ring's first rank << 16, on every rank 16-byte aligned << 24 from
                   // its first so many << 28 elements on
};
constexpr int kFoldPad = 16;  // pointers a burst may read past the last tensor's
constexpr int64_t fold_pointers(int64_t ntensors, int nranks) { return ntensors * 2 * nranks + kFoldPad; }
struct FoldTable {
  void* const* ptrs;  // DEVICE [ntensors][2 * nranks]: each tensor's ranks, twice over, then kFoldPad zeros
  const FoldTile* tiles;  // DEVICE
  int64_t ntiles;
  int stretches;  // of a tile: 1 or kFoldWide
};
hipError_t launch_fold_table(const FoldTable& t, const RingArgs& a, int64_t count, int tensor_dtype, int buf_dtype,
                             int divmode, hipStream_t stream);  // count: elements the tiles hold, about

// Broadcast chain step (broadcast_kernels.hip).
struct BcastArgs {
  int n, root, step;
  int64_t nbytes;
  int64_t q, rem;  // 16-byte units per chunk: q, the first rem chunks one more
};
hipError_t launch_bcast_step(const RankPtrs& bufs, const BcastArgs& a, bool vector_ok, hipStream_t stream);
// The whole broadcast in one launch (broadcast_kernels.hip, fusion_kernels.hip for many tensors):
// 16-byte units per lane, and an LDS reservation that holds the wavefronts per CU down.  Few
// ranks leave a wavefront little to store for what it has to find first (ResNet-50 to 2 ranks 66 us
// with one unit, 44 with two, 39 with four; small lists gain nothing: 1.2 MB to 3 ranks 6.0, 6.1
// and 6.9 us); many ranks are many streams at once, which like little in flight (VGG-16 to 32
// ranks 3.41 ms with two units, 3.43 with one, 3.19 with one and 12 wavefronts per CU; ResNet-50 to
// 8 ranks 151 us with two, 145 with two and 16).
struct BcastShape {
  int units;
  unsigned lds;
};
inline BcastShape bcast_shape(int nranks, int64_t bytes) {
  if (nranks > 16) return {1, (160u << 10) / 12 / 512 * 512 - 512};
  if (nranks <= 4 && bytes >= (32 << 20)) return {4, 0};
  return {2, nranks <= 4 ? 0u : (160u << 10) / 16 / 512 * 512 - 512};
}
constexpr int64_t kBcastRow = 1 << 22;  // blocks in a row of the grid, when there are more than one row
hipError_t launch_bcast(const RankPtrs& bufs, const BcastArgs& a, hipStream_t stream);  // a.step, q, rem not used

// One chain step of a broadcast of many tensors (fusion_kernels.hip): the chain runs over
// a virtual byte space in which tensor t occupies [voff[t], voff[t] + nbytes[t]).
struct BcastTensorsArgs {
  const void* const* ptrs;  // DEVICE table of tensor pointers, rank-major [n * ntensors]
  const int64_t* nbytes;    // DEVICE [ntensors]
  const int64_t* voff;      // DEVICE [ntensors], ascending multiples of 16, disjoint extents
  int ntensors;
  int n, root, step;
  int64_t total;            // bytes of the virtual space
  int64_t q, rem;           // 16-byte units per chunk: q, the first rem chunks one more
};
hipError_t launch_bcast_tensors_step(const BcastTensorsArgs& a, hipStream_t stream);
// The whole broadcast in one launch (a.step is not used); data: the tensors' bytes, about, which
// decide the launch's shape (the space may be far longer than they are).
hipError_t launch_bcast_tensors(const BcastTensorsArgs& a, int64_t data, hipStream_t stream);

// Launchers (fusion_kernels.hip).  With `ring` (nranks >= 3), the copy-in also does
// the ring's adding step 0 (and with `skip_sender` leaves out each chunk's sender's
// own copy, which the fused cycle never reads) and the copy-out its replacing step N-2.
hipError_t launch_pack(const void* const* srcs, const int64_t* numel, const int64_t* offset, int ntensors,
                       int src_dtype, const RankPtrs& bufs, int64_t count, int buf_dtype, int nranks, bool ring,
                       bool skip_sender, hipStream_t stream);
hipError_t launch_unpack(const RankPtrs& bufs, int64_t count, int buf_dtype, void* const* dsts,
                         const int64_t* numel, const int64_t* offset, int ntensors, int dst_dtype, int nranks,
                         bool ring, hipStream_t stream);

}  // namespace hvdx

// Every kernel launch of the library goes through this.
#define HVDX_LAUNCH(kernel, grid, block, shmem, stream, ...)                                                \
  do {                                                                                                      \
    ::hvdx::LaunchEvents& hvdx_ev_ = ::hvdx::pending_launch_events();                                       \
    if (hvdx_ev_.start) {                                                                                   \
      const ::hvdx::LaunchEvents hvdx_take_ = hvdx_ev_;                                                     \
      hvdx_ev_ = ::hvdx::LaunchEvents{};                                                                    \
      hipExtLaunchKernelGGL(kernel, grid, block, shmem, stream, hvdx_take_.start, hvdx_take_.stop, 0,       \
                            __VA_ARGS__);                                                                   \
    } else {                                                                                                \
      hipLaunchKernelGGL(kernel, grid, block, shmem, stream, __VA_ARGS__);                                  \
    }                                                                                                       \
  } while (0)
