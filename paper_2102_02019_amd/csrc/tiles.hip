// Node tiles and their halos for the LDS-staged gather kernels.
//
// Nodes are cut into tiles of kTileNodes consecutive nodes (Morton order makes
// a tile a compact patch). The halo of a tile is the sorted set of distinct
// neighbour indices of its rows. The stage and filter kernels load the halo's
// field values into LDS once per tile and then read every neighbour value
// from LDS through a 16-bit position in the halo, which also halves the
// per-edge index stream (2 instead of 4 bytes).
//
// One workgroup builds one tile: the row entries are inserted into an LDS
// hash set, each distinct index is ranked by counting the smaller ones (its
// position in the sorted halo), and every entry reads its position from the
// set. The list is short (K = 90: 260 of at most 1024 slots), so counting, four
// indices per broadcast read and no barriers, replaces a bitonic sort of all
// 1024 slots (55 barriers) and the binary search of every entry: 234 -> 94 us at
// 262,144 nodes, 61 -> 35 us at 40,000 with mixed orders.
#include <climits>

#include "common.hpp"

namespace labfm {
namespace {

constexpr int kTileNodes = LABFM_TILE_NODES;
constexpr int kHaloMax = LABFM_TILE_HALO_MAX;
constexpr int kHashCap = 2 * kHaloMax;  // load factor <= 1/2
constexpr int kThreads = 256;
constexpr int kEmpty = -1;

__device__ __forceinline__ unsigned hash_slot(int j) {
  return (static_cast<unsigned>(j) * 2654435761u) >> (32 - 11);  // kHashCap = 2^11
}
static_assert(kHashCap == 2048, "hash_slot assumes 2^11 slots");

__global__ void __launch_bounds__(kThreads)
build_tiles_kernel(const int* __restrict__ row_ptr, const int* __restrict__ col, int n,
                   int* __restrict__ halo_count, int* __restrict__ halo_idx,
                   unsigned short* __restrict__ lcol, int* __restrict__ max_halo,
                   int* __restrict__ overflow) {
  __shared__ int table[kHashCap];
  __shared__ unsigned short rank_at[kHashCap];  // position of the index in each slot
  __shared__ unsigned short slot_of[kHaloMax];
  __shared__ alignas(16) int list[kHaloMax];
  __shared__ int s_count;
  const int t = blockIdx.x;
  const int tid = threadIdx.x;
  const int t0 = t * kTileNodes;
  const int t1 = min(n, t0 + kTileNodes);
  const int e0 = row_ptr[t0], e1 = row_ptr[t1];
  for (int k = tid; k < kHashCap; k += kThreads) table[k] = kEmpty;
  for (int k = tid; k < kHaloMax; k += kThreads) list[k] = INT_MAX;
  if (tid == 0) s_count = 0;
  __syncthreads();
  // insert every neighbour index (linear probing; duplicates stop at their
  // slot, most of them at the plain read)
  for (int e = e0 + tid; e < e1; e += kThreads) {
    const int j = col[e];
    unsigned sl = hash_slot(j);
    for (int probe = 0; probe < kHashCap; ++probe) {
      int prev = table[sl];
      if (prev == kEmpty) prev = atomicCAS(&table[sl], kEmpty, j);
      if (prev == kEmpty) {
        const int pos = atomicAdd(&s_count, 1);
        if (pos < kHaloMax) {
          list[pos] = j;
          slot_of[pos] = static_cast<unsigned short>(sl);
        }
        break;
      }
      if (prev == j) break;
      sl = (sl + 1) & (kHashCap - 1);
    }
  }
  __syncthreads();
  const int count = s_count;
  if (count > kHaloMax) {
    if (tid == 0) {
      atomicMax(overflow, 1);
      halo_count[t] = 0;
    }
    return;
  }
  for (int k = tid; k < count; k += kThreads) {
    const int j = list[k];
    int rank = 0;
    for (int i = 0; i < count; i += 4) {  // slots past the count hold INT_MAX
      const int4 o = *reinterpret_cast<const int4*>(list + i);
      rank += (o.x < j) + (o.y < j) + (o.z < j) + (o.w < j);
    }
    halo_idx[static_cast<long long>(t) * kHaloMax + rank] = j;
    rank_at[slot_of[k]] = static_cast<unsigned short>(rank);
  }
  if (tid == 0) {
    halo_count[t] = count;
    // (the plain read may be old, which only costs an atomic; one per tile on
    // the same address takes 10 ns each)
    if (count > *max_halo) atomicMax(max_halo, count);
  }
  __syncthreads();
  // position of every entry in the sorted halo
  for (int e = e0 + tid; e < e1; e += kThreads) {
    const int j = col[e];
    unsigned sl = hash_slot(j);
    while (table[sl] != j) sl = (sl + 1) & (kHashCap - 1);  // it was inserted above
    lcol[e] = rank_at[sl];
  }
}

}  // namespace
}  // namespace labfm

using namespace labfm;

extern "C" int32_t labfm_tile_count(int32_t n) {
  return n > 0 ? (n + kTileNodes - 1) / kTileNodes : 0;
}

extern "C" size_t labfm_tiles_workspace_bytes(void) { return 256; }

extern "C" int labfm_build_tiles(const int32_t* row_ptr, const int32_t* col, int32_t n,
                                 int64_t nnz, int32_t* halo_count, int32_t* halo_idx,
                                 uint16_t* lcol, int32_t* max_halo_out, void* workspace,
                                 size_t workspace_bytes, void* stream_) {
  clear_error();
  LABFM_REQUIRE(n > 0 && row_ptr && halo_count && halo_idx && max_halo_out,
                "build_tiles: bad arguments");
  LABFM_REQUIRE(nnz >= 0 && (nnz == 0 || (col && lcol)), "build_tiles: bad CSR arguments");
  LABFM_WORKSPACE(workspace, workspace_bytes, labfm_tiles_workspace_bytes(), "build_tiles");
  hipStream_t st = as_stream(stream_);
  const int ntiles = labfm_tile_count(n);
  int* d = static_cast<int*>(workspace);
  hipError_t e = hipMemsetAsync(d, 0, 2 * sizeof(int), st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(build_tiles_kernel, dim3(ntiles), dim3(kThreads), 0, st, row_ptr, col, n,
                       halo_count, halo_idx, lcol, d, d + 1);
    e = hipGetLastError();
  }
  int h[2] = {0, 0};
  if (e == hipSuccess) e = hipMemcpyAsync(h, d, 2 * sizeof(int), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  LABFM_HIP(e);
  *max_halo_out = h[0];
  if (h[1]) {
    set_error("build_tiles: a tile's halo exceeds %d nodes", kHaloMax);
    return LABFM_ERR_CAPACITY;
  }
  return LABFM_OK;
}
