// Stencil search: N_i = { j != i : |r_ji| <= 2 h_i } (stencil definition of
// the paper's LABFM section), as CSR with ascending j per row.
//
// Nodes are binned into a uniform cell grid whose cells are at least
// 2 max(h) wide, so every neighbour of a node lies in the 3x3 block of cells
// around it. A counting sort lists each cell's nodes in ascending order (a
// scatter in any order, then each node's rank among its cell's). A workgroup
// takes a run of nodes in cell order; for each cell of the run it brings the
// candidates of the 3x3 block into LDS once, and its wavefronts test 64
// candidates at a time for one node after another. The count pass sizes the
// rows, a scan turns the counts into row offsets, and the fill pass, whose
// candidates are merged into ascending order in LDS, writes the accepted ones
// of each 64 at the row's next positions. The distance test rounds every
// product and sum separately (no fused multiply-add), so the lists are
// reproducible bit for bit by any IEEE-754 double implementation of the same
// test.
//
// Before, one thread per node walked the candidates one by one, the fill as a
// 9-way merge: a serial chain of some 260 dependent gathers. The passes are
// bound by the issue of their instructions (the merge's binary searches and
// the tests of 260 candidates for 90 neighbours). 262,144 nodes, K = 90: count
// 225 -> 109 us, fill 468 -> 171 us; 65,536 nodes, K = 60: 79 -> 37 and
// 222 -> 49 us; the binning and sorting, 23 launches of 115 us together at
// 262,144 nodes, is now 8 launches of 40 us.
// Where h varies the blocks hold more candidates than fit (768) and are taken in
// parts, a cell of more than 64 nodes by several workgroups, each for itself:
// whole calls of the 1.0M-node graded set 23.0 -> 3.4 ms; of 262,144 nodes with
// one of ten times the others' h (29,000 candidates a block) 75 -> 18 ms.
#include <algorithm>
#include <climits>
#include <cmath>
#include <rocprim/device/device_scan.hpp>

#include "common.hpp"

namespace labfm {
namespace {

struct Grid {
  int ncx, ncy;
  double wx, wy;  // cell widths
  double Lx, Ly;
  int px, py;     // periodic flags
};

__device__ __forceinline__ int cell_coord(double p, double w, int nc) {
  int c = static_cast<int>(floor(p / w));
  return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

// Candidate cell coordinates along one axis (at most 3, all distinct).
__device__ __forceinline__ int axis_candidates(int c, int nc, int periodic, int* out) {
  int k = 0;
  if (periodic) {
    if (nc >= 3) {
      out[k++] = (c + nc - 1) % nc;
      out[k++] = c;
      out[k++] = (c + 1) % nc;
    } else {
      for (int a = 0; a < nc; ++a) out[k++] = a;
    }
  } else {
    for (int a = c - 1; a <= c + 1; ++a)
      if (a >= 0 && a < nc) out[k++] = a;
  }
  return k;
}

// |r_ji| <= 2 h_i with separately rounded products and sum (contraction into
// an FMA is switched off here).
__device__ __forceinline__ bool within(double xi, double yi, double xj, double yj, double r2,
                                       const Grid& g) {
#pragma clang fp contract(off)
  const double dx = wrap_axis(xj - xi, g.Lx, g.px);
  const double dy = wrap_axis(yj - yi, g.Ly, g.py);
  const double d2 = dx * dx + dy * dy;
  return d2 <= r2;
}

// The same where no pair is nearer through the boundary.
__device__ __forceinline__ bool within_plain(double xi, double yi, double xj, double yj,
                                             double r2) {
#pragma clang fp contract(off)
  const double dx = xj - xi;
  const double dy = yj - yi;
  const double d2 = dx * dx + dy * dy;
  return d2 <= r2;
}

// Head of the workspace: the two results that the host reads, and the grid
// for labfm_fill_neighbours.
struct Head {
  unsigned long long hmax_bits;  // max(h) over the positive h, as a bit pattern
  unsigned long long total;      // CSR entries
  Grid grid;
};
static_assert(sizeof(Head) <= 256, "the head's part of the workspace");

constexpr int kT = 256;         // threads of every kernel here
constexpr int kWaves = kT / 64;
constexpr int kCap = 768;       // candidates in LDS at a time
constexpr int kSets = 6;        // candidates per lane in registers
constexpr int kRunMax = 64;     // most nodes per workgroup of the search, and
                                // most of a cell that is not cut between two
constexpr int kNodesMax = 2 * kRunMax;
constexpr int kLists = 9;       // cells of a block

// max over h, NaN and negative values ignored, from 0: positive doubles order
// as their bit patterns
__global__ void __launch_bounds__(kT)
hmax_kernel(const double* __restrict__ h, int n, Head* __restrict__ head) {
  double m = 0.0;
  __shared__ double sh[kWaves];
  for (int i = blockIdx.x * kT + threadIdx.x; i < n; i += gridDim.x * kT) m = fmax(m, h[i]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWaves; ++w) m = fmax(m, sh[w]);
    atomicMax(&head->hmax_bits, static_cast<unsigned long long>(__double_as_longlong(m)));
  }
}

__global__ void __launch_bounds__(kT)
clear_kernel(int* __restrict__ p, int count) {
  for (int i = blockIdx.x * kT + threadIdx.x; i < count; i += gridDim.x * kT) p[i] = 0;
}

// Cell of every node and its arrival number in the cell (any order): one
// atomic per distinct cell of a wavefront (nodes near in space are near in
// memory, so a wavefront's lie in a few cells; an atomic per node took 26 us
// at 262,144 nodes).
__global__ void __launch_bounds__(kT)
bin_kernel(const double* __restrict__ x, const double* __restrict__ y, int n, Grid g,
           Head* __restrict__ head, int* __restrict__ cell_of, int* __restrict__ cell_count,
           int* __restrict__ arrival) {
  const int i = blockIdx.x * kT + threadIdx.x;
  if (i == 0) head->grid = g;
  if (i >= n) return;
  const int cx = cell_coord(x[i], g.wx, g.ncx);
  const int cy = cell_coord(y[i], g.wy, g.ncy);
  const int c = cy * g.ncx + cx;
  cell_of[i] = c;
  const unsigned long long below = (1ull << (threadIdx.x & 63)) - 1ull;
  bool done = false;
  int number = 0;
  while (!done) {  // the lanes left take the first one's cell
    if (c == __builtin_amdgcn_readfirstlane(c)) {
      const unsigned long long same = __builtin_amdgcn_ballot_w64(true);
      int start = 0;
      if ((same & below) == 0) start = atomicAdd(&cell_count[c], __builtin_popcountll(same));
      number = __builtin_amdgcn_readfirstlane(start) + __builtin_popcountll(same & below);
      done = true;
    }
  }
  arrival[i] = number;
}

__global__ void __launch_bounds__(kT)
scatter_kernel(const int* __restrict__ cell_of, const int* __restrict__ cell_start,
               const int* __restrict__ arrival, int n, int* __restrict__ unsorted) {
  const int i = blockIdx.x * kT + threadIdx.x;
  if (i < n) unsorted[cell_start[cell_of[i]] + arrival[i]] = i;
}

// Each node to its cell's start plus the number of smaller indices there.
__global__ void __launch_bounds__(kT)
rank_kernel(const int* __restrict__ cell_of, const int* __restrict__ cell_start,
            const int* __restrict__ unsorted, int n, int* __restrict__ cell_nodes) {
  const int i = blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  const int c = cell_of[i];
  const int b = cell_start[c], e = cell_start[c + 1];
  int r = 0;
  for (int k = b; k < e; ++k) r += unsorted[k] < i ? 1 : 0;
  cell_nodes[b + r] = i;
}

// A workgroup's nodes, and the candidates of one cell's block as up to kLists
// ascending lists in cell_nodes with the part of them that is in LDS.
template <bool kFill>
struct SearchSmem {
  int node[kNodesMax], cell[kNodesMax];
  double nx[kNodesMax], ny[kNodesMax], nr2[kNodesMax];
  int first[kNodesMax], room[kNodesMax];  // fill: each row's first place and length
  int seen[kNodesMax];                // accepted so far
  int from[kLists];                   // next candidate of each list
  int left[kLists];                   // candidates of each list not yet taken
  int off[kLists + 1];                // this part: first position of each list's
  int raw[kFill ? kCap : 1];          // fill: the part, list after list
  int idx[kCap];
  double x[kCap], y[kCap];
  unsigned long long sum;             // count: the rows' lengths added up
};

// Candidates not above v among `most` of a list from `from` on.
__device__ __forceinline__ int up_to(const int* __restrict__ cell_nodes, int from, int most, int v) {
  int lo = 0, hi = most;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (cell_nodes[from + mid] <= v) {
      lo = mid + 1;
    } else {
      hi = mid;
    }
  }
  return lo;
}

// One workgroup searches nodes cell_nodes[run blockIdx.x ...], `run` of them,
// except that a cell of at most kRunMax nodes goes whole to the workgroup that
// its first node falls to: its candidates are brought in (and merged) once.
// Count: the rows' lengths and their sum. Fill: the rows, ascending.
template <bool kFill>
__global__ void __launch_bounds__(kT)
search_kernel(const double* __restrict__ x, const double* __restrict__ y,
              const double* __restrict__ h, int n, int run, Head* __restrict__ head,
              const int* __restrict__ cell_of, const int* __restrict__ cell_start,
              const int* __restrict__ cell_nodes, int* __restrict__ counts,
              const int* __restrict__ row_ptr, int* __restrict__ col) {
  __shared__ SearchSmem<kFill> sm;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const Grid g = head->grid;
  int k0 = blockIdx.x * run, k1 = min(n, k0 + run);
  {
    const int ca = cell_of[cell_nodes[k0]], cb = cell_of[cell_nodes[k1 - 1]];
    const int a0 = cell_start[ca], a1 = cell_start[ca + 1];
    const int b0 = cell_start[cb], b1 = cell_start[cb + 1];
    if (a0 < k0 && a1 - a0 <= kRunMax) k0 = a1;  // the workgroup before has it
    if (b1 - b0 <= kRunMax) k1 = b1;
  }
  const int nodes = k1 - k0;  // none if one such cell held the whole run
  if (!kFill && blockIdx.x == 0 && tid == 0) counts[n] = 0;
  if (nodes <= 0) return;
  if (tid < nodes) {
    const int i = cell_nodes[k0 + tid];
    sm.node[tid] = i;
    sm.cell[tid] = cell_of[i];
    sm.nx[tid] = x[i];
    sm.ny[tid] = y[i];
    const double r = 2.0 * h[i];
    sm.nr2[tid] = r * r;  // a lone product: rounded once
    sm.seen[tid] = 0;
    if (kFill) {
      sm.first[tid] = row_ptr[i];
      sm.room[tid] = row_ptr[i + 1] - row_ptr[i];
    }
  }
  if (tid == 0) sm.sum = 0;
  __syncthreads();
  int kb = 0;
  while (kb < nodes) {
    // the run's nodes of one cell: kb .. ke
    const int cell = sm.cell[kb];
    const int ke = min(nodes, cell_start[cell + 1] - k0);
    const int cx = cell % g.ncx, cy = cell / g.ncx;
    // no candidate of a block clear of the box's outermost cells is nearer
    // through the boundary
    const bool wrapped = !(cx >= 2 && cx < g.ncx - 2 && cy >= 2 && cy < g.ncy - 2);
    int xs[3], ys[3];
    const int nx = axis_candidates(cx, g.ncx, g.px, xs);
    const int ny = axis_candidates(cy, g.ncy, g.py, ys);
    const int lists = nx * ny;
    if (tid < lists) {
      const int xa = tid % nx, ya = tid / nx;
      const int c = (ya == 0 ? ys[0] : (ya == 1 ? ys[1] : ys[2])) * g.ncx +
                    (xa == 0 ? xs[0] : (xa == 1 ? xs[1] : xs[2]));
      sm.from[tid] = cell_start[c];
      sm.left[tid] = cell_start[c + 1] - cell_start[c];
    } else if (tid < kLists) {
      sm.from[tid] = 0;
      sm.left[tid] = 0;
    }
    __syncthreads();
    while (true) {
      // the next part: every candidate left if they fit, else (fill) all up
      // to a value chosen so that they fit, which keeps the parts ascending
      int all = 0, before = 0;
#pragma unroll
      for (int r = 0; r < kLists; ++r) {
        const int l = sm.left[r];
        all += l;
        before += r < tid ? l : 0;
      }
      if (all == 0) break;
      if (all <= kCap) {
        if (tid <= kLists) sm.off[tid] = before;
      } else if (tid == 0) {
        int take[kLists];
        if (kFill) {
          // the first `most` of each list bound a value; at kCap / kLists
          // their candidates up to it always fit
          for (int most = kCap;; most = max(most / 2, kCap / kLists)) {
            int v = INT_MAX, part = 0;
            for (int r = 0; r < kLists; ++r)
              if (sm.left[r] > most) v = min(v, cell_nodes[sm.from[r] + most - 1]);
            for (int r = 0; r < kLists; ++r) {
              take[r] = up_to(cell_nodes, sm.from[r], min(sm.left[r], most), v);
              part += take[r];
            }
            if (part <= kCap) break;
          }
        } else {
          int room = kCap;
          for (int r = 0; r < kLists; ++r) {
            take[r] = min(room, sm.left[r]);
            room -= take[r];
          }
        }
        int o = 0;
        for (int r = 0; r < kLists; ++r) {
          sm.off[r] = o;
          o += take[r];
        }
        sm.off[kLists] = o;
      }
      __syncthreads();
      int off[kLists + 1];
#pragma unroll
      for (int r = 0; r <= kLists; ++r) off[r] = sm.off[r];
      const int part = off[kLists];
      for (int t = tid; t < part; t += kT) {
        int r = 0;
#pragma unroll
        for (int q = 1; q < kLists; ++q) r += t >= off[q] ? 1 : 0;
        const int j = cell_nodes[sm.from[r] + t - sm.off[r]];
        if (kFill) {
          sm.raw[t] = j;
        } else {
          sm.idx[t] = j;
          sm.x[t] = x[j];
          sm.y[t] = y[j];
        }
      }
      __syncthreads();
      if (kFill) {
        // a candidate's place: the number of smaller ones in every list, by
        // binary searches side by side
        int longest = 0;
#pragma unroll
        for (int r = 0; r < kLists; ++r) longest = max(longest, off[r + 1] - off[r]);
        const int top = 1 << (31 - __builtin_clz(longest));
        for (int t = tid; t < part; t += kT) {
          const int j = sm.raw[t];
          const double xj = x[j], yj = y[j];
          int at[kLists];
#pragma unroll
          for (int r = 0; r < kLists; ++r) at[r] = off[r];
          for (int step = top; step > 0; step >>= 1) {
#pragma unroll
            for (int r = 0; r < kLists; ++r) {
              const int to = at[r] + step;
              const bool in = to <= off[r + 1];
              const int v = sm.raw[in ? to - 1 : 0];
              at[r] = (in && v < j) ? to : at[r];
            }
          }
          int place = 0;
#pragma unroll
          for (int r = 0; r < kLists; ++r) place += at[r] - off[r];
          sm.idx[place] = j;
          sm.x[place] = xj;
          sm.y[place] = yj;
        }
        __syncthreads();
      }
      // kSets candidates per lane in registers, tested for one node after
      // another
      for (int base = 0; base < part; base += 64 * kSets) {
        int j[kSets];
        double xj[kSets], yj[kSets];
#pragma unroll
        for (int s = 0; s < kSets; ++s) {
          const int t = base + 64 * s + lane;
          const bool in = t < part;
          j[s] = in ? sm.idx[t] : -1;
          xj[s] = in ? sm.x[t] : NAN;  // never within
          yj[s] = in ? sm.y[t] : NAN;
        }
        for (int k = kb + wave; k < ke; k += kWaves) {
          const int i = sm.node[k];
          const double xi = sm.nx[k], yi = sm.ny[k], r2 = sm.nr2[k];
          int seen = sm.seen[k];
          int* row = kFill ? col + __builtin_amdgcn_readfirstlane(sm.first[k]) : nullptr;
          const unsigned room = kFill ? sm.room[k] : 0;
#pragma unroll
          for (int s = 0; s < kSets; ++s) {
            if (base + 64 * s < part) {
              const bool ok = j[s] != i && (wrapped ? within(xi, yi, xj[s], yj[s], r2, g)
                                                    : within_plain(xi, yi, xj[s], yj[s], r2));
              const unsigned long long hit = __builtin_amdgcn_ballot_w64(ok);
              if (kFill && ok) {
                const unsigned o = __builtin_amdgcn_mbcnt_hi(
                    static_cast<unsigned>(hit >> 32),
                    __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(hit), seen));
                if (o < room) row[o] = j[s];
              }
              seen += __builtin_popcountll(hit);
            }
          }
          if (lane == 0) sm.seen[k] = seen;
        }
      }
      if (tid < kLists) {
        const int taken = sm.off[tid + 1] - sm.off[tid];
        sm.from[tid] += taken;
        sm.left[tid] -= taken;
      }
      __syncthreads();
    }
    kb = ke;
    __syncthreads();
  }
  if (!kFill) {
    if (tid < nodes) {
      counts[sm.node[tid]] = sm.seen[tid];
      atomicAdd(&sm.sum, static_cast<unsigned long long>(sm.seen[tid]));
    }
    __syncthreads();
    if (tid == 0 && sm.sum != 0) atomicAdd(&head->total, sm.sum);
  }
}

// Nodes per workgroup: 64, fewer where that would leave compute units idle.
int run_of(int n) { return n >= 65536 ? kRunMax : (n >= 16384 ? 32 : 16); }

// Sizes of the search's workspace for n nodes: the cell table has at most
// 4n + 65 entries (see the cell-count cap below), and one temporary storage
// area serves both scans.
size_t neighbours_temp_bytes(int32_t n) {
  const size_t nscan = 4 * static_cast<size_t>(n) + 65;
  size_t tb_scan = 0;
  hipStream_t st{};
  (void)rocprim::exclusive_scan(nullptr, tb_scan, static_cast<const int*>(nullptr),
                                static_cast<int*>(nullptr), 0, nscan, rocprim::plus<int>(), st);
  return align256(tb_scan);
}

// the per-node and per-cell integer arrays (cell table at its cap)
size_t neighbours_table_bytes(int32_t n) {
  const size_t ncell_max = 4 * static_cast<size_t>(n) + 64;
  return align256(sizeof(int) * (static_cast<size_t>(n) * 4 + 1 + 2 * (ncell_max + 1)));
}

// The workspace's parts. Their places depend on n alone.
struct Tables {
  Head* head;
  void* temp;
  size_t temp_bytes;
  int* cell_of;     // n
  int* cell_nodes;  // n
  int* counts;      // n + 1 (the last stays 0); the arrival numbers before
  int* unsorted;    // n
  int* cell_count;  // ncell + 1 (the last stays 0)
  int* cell_start;  // ncell + 1
  Tables(void* workspace, int32_t n) {
    const size_t ncell_max = 4 * static_cast<size_t>(n) + 64;
    char* base = static_cast<char*>(workspace);
    head = reinterpret_cast<Head*>(base);
    temp = base + 256;
    temp_bytes = neighbours_temp_bytes(n);
    cell_of = reinterpret_cast<int*>(base + 256 + temp_bytes);
    cell_nodes = cell_of + n;
    counts = cell_nodes + n;
    unsorted = counts + n + 1;
    cell_count = unsorted + n;
    cell_start = cell_count + ncell_max + 1;
  }
};

int launch_fill(const double* x, const double* y, const double* h, int32_t n, const Tables& tb,
                const int32_t* row_ptr, int32_t* col, hipStream_t st) {
  const int run = run_of(n);
  hipLaunchKernelGGL(search_kernel<true>, dim3(blocks_for(n, run)), dim3(kT), 0, st, x, y, h, n,
                     run, tb.head, tb.cell_of, tb.cell_start, tb.cell_nodes, tb.counts, row_ptr,
                     col);
  LABFM_LAUNCHED();
  return LABFM_OK;
}

}  // namespace
}  // namespace labfm

using namespace labfm;

extern "C" size_t labfm_neighbours_workspace_bytes(int32_t n) {
  if (n <= 0) return 0;
  return 256 + neighbours_temp_bytes(n) + neighbours_table_bytes(n);
}

extern "C" int labfm_build_neighbours(const double* x, const double* y, const double* h,
                                      int32_t n, labfm_box box, int32_t* row_ptr, int32_t* col,
                                      int64_t capacity, int64_t* nnz_out, void* workspace,
                                      size_t workspace_bytes, void* stream_) {
  clear_error();
  LABFM_REQUIRE(n > 0, "build_neighbours: n must be positive (got %d)", n);
  LABFM_REQUIRE(x && y && h && row_ptr && nnz_out, "build_neighbours: null pointer argument");
  LABFM_REQUIRE(box.Lx > 0.0 && box.Ly > 0.0, "build_neighbours: box sides must be positive");
  LABFM_WORKSPACE(workspace, workspace_bytes, labfm_neighbours_workspace_bytes(n),
                  "build_neighbours");
  hipStream_t st = as_stream(stream_);

  const Tables tb(workspace, n);
  hipLaunchKernelGGL(clear_kernel, dim3(1), dim3(kT), 0, st, reinterpret_cast<int*>(tb.head),
                     static_cast<int>(sizeof(Head) / sizeof(int)));
  hipLaunchKernelGGL(hmax_kernel, dim3(std::min(128u, blocks_for(n, 4 * kT))), dim3(kT), 0, st, h, n,
                     tb.head);
  LABFM_LAUNCHED();
  double hmax = 0.0;
  LABFM_HIP(hipMemcpyAsync(&hmax, &tb.head->hmax_bits, sizeof(double), hipMemcpyDeviceToHost, st));
  LABFM_HIP(hipStreamSynchronize(st));
  LABFM_REQUIRE(std::isfinite(hmax) && hmax > 0.0, "build_neighbours: max(h) must be positive");
  if (box.periodic_x)
    LABFM_REQUIRE(4.0 * hmax < box.Lx, "build_neighbours: periodic Lx must exceed 4 max(h)");
  if (box.periodic_y)
    LABFM_REQUIRE(4.0 * hmax < box.Ly, "build_neighbours: periodic Ly must exceed 4 max(h)");

  // Cells strictly wider than the largest stencil diameter.
  const double reach = 2.0 * hmax * (1.0 + 1e-9);
  Grid g;
  g.ncx = static_cast<int>(std::fmax(1.0, std::floor(box.Lx / reach)));
  g.ncy = static_cast<int>(std::fmax(1.0, std::floor(box.Ly / reach)));
  // keep the cell table modest for very small stencils
  while (static_cast<long long>(g.ncx) * g.ncy > 4LL * n + 64) {
    g.ncx = (g.ncx + 1) / 2;
    g.ncy = (g.ncy + 1) / 2;
  }
  g.wx = box.Lx / g.ncx;
  g.wy = box.Ly / g.ncy;
  g.Lx = box.Lx;
  g.Ly = box.Ly;
  g.px = box.periodic_x ? 1 : 0;
  g.py = box.periodic_y ? 1 : 0;
  const int ncell = g.ncx * g.ncy;

  size_t tbytes = tb.temp_bytes;
  const unsigned nb = blocks_for(n, kT);
  hipLaunchKernelGGL(clear_kernel, dim3(std::min(1024u, blocks_for(ncell + 1, kT))), dim3(kT), 0,
                     st, tb.cell_count, ncell + 1);
  hipLaunchKernelGGL(bin_kernel, dim3(nb), dim3(kT), 0, st, x, y, n, g, tb.head, tb.cell_of,
                     tb.cell_count, tb.counts);
  LABFM_LAUNCHED();
  LABFM_HIP(rocprim::exclusive_scan(tb.temp, tbytes, tb.cell_count, tb.cell_start, 0,
                                    static_cast<size_t>(ncell) + 1, rocprim::plus<int>(), st));
  hipLaunchKernelGGL(scatter_kernel, dim3(nb), dim3(kT), 0, st, tb.cell_of, tb.cell_start,
                     tb.counts, n, tb.unsorted);
  hipLaunchKernelGGL(rank_kernel, dim3(nb), dim3(kT), 0, st, tb.cell_of, tb.cell_start,
                     tb.unsorted, n, tb.cell_nodes);
  const int run = run_of(n);
  hipLaunchKernelGGL(search_kernel<false>, dim3(blocks_for(n, run)), dim3(kT), 0, st, x, y, h, n,
                     run, tb.head, tb.cell_of, tb.cell_start, tb.cell_nodes, tb.counts,
                     static_cast<const int*>(nullptr), static_cast<int*>(nullptr));
  LABFM_LAUNCHED();
  LABFM_HIP(rocprim::exclusive_scan(tb.temp, tbytes, tb.counts, row_ptr, 0,
                                    static_cast<size_t>(n) + 1, rocprim::plus<int>(), st));
  // the total in 64 bits (an int32 offset past INT_MAX is reported below)
  long long total = 0;
  LABFM_HIP(hipMemcpyAsync(&total, &tb.head->total, sizeof(long long), hipMemcpyDeviceToHost, st));
  LABFM_HIP(hipStreamSynchronize(st));
  *nnz_out = total;
  if (total > INT_MAX) {
    set_error("build_neighbours: %lld entries exceed the int32 CSR index range", total);
    return LABFM_ERR_UNSUPPORTED;
  }
  if (col == nullptr || capacity < total) {
    set_error("build_neighbours: col capacity %lld < nnz %lld", (long long)capacity, total);
    return LABFM_ERR_CAPACITY;
  }
  return launch_fill(x, y, h, n, tb, row_ptr, col, st);
}

extern "C" int labfm_fill_neighbours(const double* x, const double* y, const double* h, int32_t n,
                                     const int32_t* row_ptr, int32_t* col, int64_t capacity,
                                     int64_t nnz, void* workspace, size_t workspace_bytes,
                                     void* stream_) {
  clear_error();
  LABFM_REQUIRE(n > 0, "fill_neighbours: n must be positive (got %d)", n);
  LABFM_REQUIRE(x && y && h && row_ptr && (col || nnz == 0),
                "fill_neighbours: null pointer argument");
  LABFM_REQUIRE(nnz >= 0 && nnz <= INT_MAX, "fill_neighbours: bad entry count %lld",
                (long long)nnz);
  LABFM_WORKSPACE(workspace, workspace_bytes, labfm_neighbours_workspace_bytes(n),
                  "fill_neighbours");
  if (capacity < nnz) {
    set_error("fill_neighbours: col capacity %lld < nnz %lld", (long long)capacity,
              (long long)nnz);
    return LABFM_ERR_CAPACITY;
  }
  if (nnz == 0) return LABFM_OK;
  return launch_fill(x, y, h, n, Tables(workspace, n), row_ptr, col, as_stream(stream_));
}
