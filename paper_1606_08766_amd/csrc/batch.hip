// Gather / scatter kernels that pack many small sort requests into one
// segmented sort (used by the sort server): one launch copies every
// request's keys into the packed input, one launch copies every request's
// sorted keys and permutation back.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "engine.hpp"
#include "internal.hpp"

namespace rs {

// An entry's keys are copied in pieces of kPiece by kPieces workgroups, each
// thread with kPieceItems loads in flight at a time.  An entry per workgroup,
// a key per thread in turn, left most of the chip idle and each workgroup
// waiting for one load after the other (24 requests of 2^8 to 2^22 keys: 208 us
// for the copies in, 276 for those back; now 38 and 30, 5 to 20 a launch).
constexpr int kBatchThreads = 256, kPieceItems = 16, kPieces = 8;
constexpr uint32_t kPiece = kBatchThreads * kPieceItems;

// copy(j0, c): the stretch [j0, j0 + c) of an entry, 0 < c <= kPiece.
template <typename F>
__device__ __forceinline__ void for_pieces(const BatchEntry* tab, uint32_t count, F&& copy) {
  for (uint32_t q = blockIdx.x; q < count * kPieces; q += gridDim.x) {
    const BatchEntry& e = tab[q / kPieces];
    for (uint64_t j0 = (uint64_t)(q % kPieces) * kPiece; j0 < e.n; j0 += (uint64_t)kPieces * kPiece)
      copy(e, j0, (uint32_t)min((uint64_t)kPiece, e.n - j0));
  }
}

// Stretch of c keys from s into v; thread t's i-th is key i * kBatchThreads + t.
template <typename T>
__device__ __forceinline__ void piece_load(const T* s, uint32_t c, T (&v)[kPieceItems]) {
#pragma unroll
  for (int i = 0; i < kPieceItems; i++) v[i] = at32(s, min((uint32_t)(i * kBatchThreads) + threadIdx.x, c - 1u));
}
template <typename T>
__device__ __forceinline__ void piece_store(T* d, uint32_t c, const T (&v)[kPieceItems]) {
#pragma unroll
  for (int i = 0; i < kPieceItems; i++) {
    const uint32_t j = (uint32_t)(i * kBatchThreads) + threadIdx.x;
    if (j < c) at32(d, j) = v[i];
  }
}

template <typename T>
__global__ __launch_bounds__(kBatchThreads) void k_batch_in(const BatchEntry* tab, uint32_t count, T* packed) {
  for_pieces(tab, count, [&](const BatchEntry& e, uint64_t j0, uint32_t c) {
    T v[kPieceItems];
    piece_load((const T*)e.src + j0, c, v);
    piece_store(packed + e.off + j0, c, v);
  });
}

template <typename T>
__global__ __launch_bounds__(kBatchThreads) void k_batch_out(const BatchEntry* tab, uint32_t count, const T* keys,
                                                             const uint32_t* perm) {
  for_pieces(tab, count, [&](const BatchEntry& e, uint64_t j0, uint32_t c) {
    T v[kPieceItems];
    uint32_t p[kPieceItems];
    piece_load(keys + e.off + j0, c, v);
    if (e.dst_perm) piece_load(perm + e.off + j0, c, p);
    piece_store((T*)e.dst_keys + j0, c, v);
    if (e.dst_perm) piece_store(e.dst_perm + j0, c, p);
  });
}

static uint32_t batch_grid(uint32_t count) {
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((uint64_t)count * kPieces, (uint64_t)num_cu_cached() * 8));
}

int enqueue_batch_in(const BatchEntry* tab_dev, uint32_t count, uint32_t key_bytes, void* packed, hipStream_t st) {
  const uint32_t g = batch_grid(count);
  if (key_bytes == 8)
    RS_LAUNCH(k_batch_in<uint64_t>, g, kBatchThreads, st, tab_dev, count, (uint64_t*)packed);
  else
    RS_LAUNCH(k_batch_in<uint32_t>, g, kBatchThreads, st, tab_dev, count, (uint32_t*)packed);
  return 0;
}

int enqueue_batch_out(const BatchEntry* tab_dev, uint32_t count, uint32_t key_bytes, const void* keys,
                      const uint32_t* perm, hipStream_t st) {
  const uint32_t g = batch_grid(count);
  if (key_bytes == 8)
    RS_LAUNCH(k_batch_out<uint64_t>, g, kBatchThreads, st, tab_dev, count, (const uint64_t*)keys, perm);
  else
    RS_LAUNCH(k_batch_out<uint32_t>, g, kBatchThreads, st, tab_dev, count, (const uint32_t*)keys, perm);
  return 0;
}

}  // namespace rs
