// Reverse mode (adjoint) of the filtered RK3(2)4[2R+]C time loop of the
// isothermal Navier-Stokes equations, float64.
//
// With A_d = [w^d_ij] - diag(S^d_i) (S^d_i = sum_j w^d_ij) every operator is
// L^d = A_d, so its transpose acts as
//     (A_d^T g)_j = sum_{i : j in N_i} w^d_ij g_i - S^d_j g_j,
// a gather over the transposed stencils (the edges i -> j grouped by j, in
// ascending i, with their own copy of the weights): no atomics touch
// floating-point data and every result is bitwise reproducible.
//
// One step q -> filter(q + dt sum_i b_i F_i), Y_i = q + dt sum_{j<i} a_ij F_j,
// F_i = R(Y_i), is reversed as
//     qbar' = qbar + A_hyp^T (kappa qbar)                       (filter)
//     Fbar_i = dt (b_i P_i + a_{i+1,i} Ybar_{i+1}),  Ybar_i = J_R(Y_i)^T Fbar_i
//     with P_4 = P_3 = qbar', P_2 = P_3 + Ybar_4, P_1 = P_2 + Ybar_3,
//     qbar = P_1 + Ybar_2 + Ybar_1,
// which uses the two-register structure of the scheme (a_ij = b_j for
// j < i - 1). J_R^T at Y_i needs the forward operator sums at Y_i in a
// pointwise part, which forms each node's operator-sum adjoints, and then a
// transposed gather of these. The forward sums come from the stage launches
// that recompute Y_2, Y_3, Y_4 (and one more at Y_4), which store them on the
// way: no gather is repeated for them. Everything the pointwise part of stage
// i - 1 reads besides is the node's own, so the transposed gather of stage i
// does it when it has the node's Ybar_i; the filter's gather does that of
// stage 4. A reversed step is then nine launches, all of them gathers.
// States are checkpointed every ckpt_every steps and each segment is
// recomputed once before it is reversed; the pass that makes the checkpoints
// stops at the last of them.
//
// 65,536 nodes, m = 6, ten steps with checkpoints every five, forward run
// included: 9.47 ms with a forward gather per stage, twelve operator-sum
// adjoints per node in place of six values and single-edge loads; now 6.5 ms.
#include <climits>

#include "gather.hpp"

namespace labfm {
namespace {

constexpr int kAdjLpn = 16;

// ----------------------------------------------------------- transpose build

__global__ void tcount_kernel(const int* __restrict__ col, long long nnz, int* __restrict__ cnt) {
  for (long long e = blockIdx.x * static_cast<long long>(blockDim.x) + threadIdx.x; e < nnz;
       e += static_cast<long long>(gridDim.x) * blockDim.x)
    atomicAdd(&cnt[col[e]], 1);
}

constexpr int kScan = 1024;
__global__ void __launch_bounds__(kScan)
tscan_kernel(const int* __restrict__ in, int* __restrict__ out, int n) {
  __shared__ long long sh[kScan];
  long long carry = 0;
  for (int base = 0; base < n; base += kScan) {
    const int i = base + threadIdx.x;
    const long long v = (i < n) ? static_cast<long long>(in[i]) : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < kScan; off <<= 1) {
      const long long t = (threadIdx.x >= off) ? sh[threadIdx.x - off] : 0;
      __syncthreads();
      sh[threadIdx.x] += t;
      __syncthreads();
    }
    if (i < n) out[i] = static_cast<int>(carry + sh[threadIdx.x] - v);
    carry += sh[kScan - 1];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[n] = static_cast<int>(carry);
}

__global__ void tfill_kernel(const int* __restrict__ row_ptr, const int* __restrict__ col, int n,
                             const int* __restrict__ tptr, int* __restrict__ cursor,
                             int* __restrict__ tsrc, int* __restrict__ tslot) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int e = row_ptr[i]; e < row_ptr[i + 1]; ++e) {
    const int j = col[e];
    const int pos = tptr[j] + atomicAdd(&cursor[j], 1);
    tsrc[pos] = i;
    tslot[pos] = e;
  }
}

// Orders each transposed row by source node (insertion sort, a few tens of
// entries), which makes the layout independent of the fill's thread order.
__global__ void tsort_kernel(const int* __restrict__ tptr, int n, int* __restrict__ tsrc,
                             int* __restrict__ tslot) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int b = tptr[j], e = tptr[j + 1];
  for (int k = b + 1; k < e; ++k) {
    const int s = tsrc[k], sl = tslot[k];
    int p = k - 1;
    while (p >= b && tsrc[p] > s) {
      tsrc[p + 1] = tsrc[p];
      tslot[p + 1] = tslot[p];
      --p;
    }
    tsrc[p + 1] = s;
    tslot[p + 1] = sl;
  }
}

__global__ void tweights_kernel(const double* __restrict__ w, const int* __restrict__ tslot,
                                long long nnz, double* __restrict__ tw) {
  for (long long e = blockIdx.x * static_cast<long long>(blockDim.x) + threadIdx.x; e < nnz;
       e += static_cast<long long>(gridDim.x) * blockDim.x) {
    const int s = tslot[e];
#pragma unroll
    for (int d = 0; d < LABFM_NUM_OPS; ++d) tw[d * nnz + e] = w[d * nnz + s];
  }
}

// ------------------------------------------------------------ adjoint kernels

// What the transposed gather reads of a source node i, kAdj values side by
// side: the adjoints of its rates and the factors that turn them into those of
// its operator sums, (rl, ru, rv, nu, u, v). From
//   R_l = -(u l_x + v l_y) - (u_x + v_y)
//   R_u = -(u u_x + v u_y) - c2 l_x + nu (Lu + (u_xx + v_xy)/3) + gx
//   R_v = -(u v_x + v v_y) - c2 l_y + nu (4/3 Lv - v_xx/3 + u_xy/3) + gy
// an edge of weights (a, b, c, d, f) (x, y, L, xx, xy) gives, with
// t = a u + b v,
//   ln rho:  -(rl t + c2 (a ru + b rv))
//   u:       -(a rl + ru t) + nu (ru (c + d/3) + rv f/3)
//   v:       -(b rl + rv t) + nu (rv (4 c - d)/3 + ru f/3).
// (Twelve operator-sum adjoints a node, 96 bytes an edge, took 57 us for
// 65,536 nodes of K = 60 with single-edge loads of the weights, eight 53 us
// with pairs, these six 42 us.)
constexpr int kAdj = 6;

// The same for one edge or, with the row sums as weights, a node's own part.
struct AdjSums {
  double tl = 0.0, cl = 0.0, u = 0.0, v = 0.0;  // ln rho: -(tl + c2 cl)
  __device__ __forceinline__ void add(double a, double b, double c, double d, double f,
                                      const double* __restrict__ g) {
    const double2* r = reinterpret_cast<const double2*>(g);
    const double2 lu = r[0], vn = r[1], w = r[2];
    constexpr double third = 1.0 / 3.0;
    const double t = fma(a, w.x, b * w.y);
    const double nru = vn.y * lu.y, nrv = vn.y * vn.x;
    const double f3 = third * f;
    tl = fma(lu.x, t, tl);
    cl = fma(a, lu.y, fma(b, vn.x, cl));
    u = fma(-a, lu.x, fma(-lu.y, t, u));
    u = fma(fma(third, d, c), nru, fma(f3, nrv, u));
    v = fma(-b, lu.x, fma(-vn.x, t, v));
    v = fma(third * (4.0 * c - d), nrv, fma(f3, nru, v));
  }
};

// The pointwise part at `node`: its record g from the stage's value Y and the
// rates' adjoints r, and, with the stage's operator sums, the adjoints of
// (ln rho, u, v) through the rates' own factors (d nu / d ln rho = -nu), loc.
__device__ __forceinline__ void adj_point(int node, int n, const double* __restrict__ Y,
                                          const double* __restrict__ sums, double rl, double ru,
                                          double rv, const Flow& fl, double* __restrict__ g,
                                          double* __restrict__ loc) {
  const long long n2 = 2 * static_cast<long long>(n);
  const double li = Y[node], ui = Y[n + node], vi = Y[n2 + node];
  const double2* s =
      reinterpret_cast<const double2*>(sums + kStageSums * static_cast<long long>(node));
  const double2 l = s[0], u = s[1], v = s[2], visc = s[3];
  const double nu = fl.mu / exp(li);
  double2* gn = reinterpret_cast<double2*>(g + kAdj * static_cast<long long>(node));
  gn[0] = make_double2(rl, ru);
  gn[1] = make_double2(rv, nu);
  gn[2] = make_double2(ui, vi);
  loc[node] = -nu * (ru * visc.x + rv * visc.y);
  loc[n + node] = -rl * l.x - ru * u.x - rv * v.x;
  loc[n2 + node] = -rl * l.y - ru * u.y - rv * v.y;
}

// Which of the weights' arrays start on a pair of edges (16 bytes): all, with
// an even nnz; those of even d, with an odd one; none need, where the weights
// themselves start off it.
enum { kAllPairs, kEvenPairs, kNoPairs };

// Edges e, e + 1 (e even) of an array of `end` entries: one 16-byte load where
// the array starts on a pair (the entry past the last one is then the next
// array's first), two loads where it does not.
template <bool kAligned>
__device__ __forceinline__ double2 edge_pair(const double* __restrict__ p, long long e,
                                             long long end) {
  if constexpr (kAligned) {
    return *reinterpret_cast<const double2*>(p + e);
  } else {
    return make_double2(p[e], e + 1 < end ? p[e + 1] : 0.0);
  }
}

// Sources of the pair at e; the node itself for an edge outside e0 .. e1, whose
// weights count as zero.
__device__ __forceinline__ int2 pair_sources(const int* __restrict__ tsrc, int e, int e0, int e1,
                                             int node) {
  return make_int2(e >= e0 ? tsrc[e] : node, e + 1 < e1 ? tsrc[e + 1] : node);
}

// Where a stage's transposed gather leads: the pointwise part of the stage
// before it (Y, sums, and its coefficients of P and Ybar), or, at stage 1
// (Y null), the step's result qbar and, for the filter of the step before,
// kappa qbar (kq, node-major in fours; null without the filter).
struct AdjNext {
  const double* Y;
  const double* sums;
  double dtb, dta;
  double* g;
  double* loc;
  double* qbar;
  double* kq;
  const double* kappa;
};

__device__ __forceinline__ void store_kq(double* __restrict__ kq, int node, double k, double ql,
                                         double qu, double qv) {
  double2* d = reinterpret_cast<double2*>(kq + 4LL * node);
  d[0] = make_double2(k * ql, k * qu);
  d[1] = make_double2(k * qv, 0.0);
}

// Transposed gather: Ybar_j = loc_j + the sum over the edges i -> j less the
// node's own part with the row sums, then P_j += Ynext_j when Ynext is set and what `nx` says. Bound by the
// weights' stream (44 bytes an edge) with the 48-byte gathers of g beside it;
// consecutive nodes go to one XCD, so that its L2 holds their sources.
template <int LPN, int PAIRS>
__global__ void __launch_bounds__(256)
adj_transpose_kernel(const int* __restrict__ tptr, const int* __restrict__ tsrc,
                     const double* __restrict__ tw, long long nnz,
                     const double* __restrict__ rowsum, const double* __restrict__ g,
                     const double* __restrict__ loc, int n, double* __restrict__ Ybar,
                     double* __restrict__ P, const double* __restrict__ Ynext, Flow fl,
                     AdjNext nx) {
  const int gid = static_cast<int>(xcd_tile(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x);
  const int node = gid / LPN;
  const int sub = gid % LPN;
  if (node >= n) return;
  AdjSums s;
  const int e0 = tptr[node], e1 = tptr[node + 1];
  for (int e = (e0 & ~1) + 2 * sub; e < e1; e += 2 * LPN) {
    const int2 src = pair_sources(tsrc, e, e0, e1, node);
    constexpr bool kEven = PAIRS != kNoPairs, kOdd = PAIRS == kAllPairs;
    const double2 a = edge_pair<kEven>(tw, e, nnz), b = edge_pair<kOdd>(tw + nnz, e, nnz);
    const double2 c = edge_pair<kEven>(tw + 2 * nnz, e, nnz);
    const double2 d = edge_pair<kOdd>(tw + 3 * nnz, e, nnz);
    const double2 f = edge_pair<kEven>(tw + 4 * nnz, e, nnz);
    const bool in0 = e >= e0, in1 = e + 1 < e1;
    s.add(in0 ? a.x : 0.0, in0 ? b.x : 0.0, in0 ? c.x : 0.0, in0 ? d.x : 0.0, in0 ? f.x : 0.0,
          g + kAdj * static_cast<long long>(src.x));
    s.add(in1 ? a.y : 0.0, in1 ? b.y : 0.0, in1 ? c.y : 0.0, in1 ? d.y : 0.0, in1 ? f.y : 0.0,
          g + kAdj * static_cast<long long>(src.y));
  }
  const double sl = -(group_sum<LPN>(s.tl) + fl.c2 * group_sum<LPN>(s.cl));
  const double su = group_sum<LPN>(s.u);
  const double sv = group_sum<LPN>(s.v);
  if (sub != 0) return;
  const long long n2 = 2 * static_cast<long long>(n);
  const double* S = rowsum + node;  // S[d * n]
  AdjSums own;
  own.add(S[0], S[n], S[n2], S[n2 + n], S[2 * n2], g + kAdj * static_cast<long long>(node));
  const double yl = loc[node] + (sl + (own.tl + fl.c2 * own.cl));
  const double yu = loc[n + node] + (su - own.u);
  const double yv = loc[n2 + node] + (sv - own.v);
  double pl = P[node], pu = P[n + node], pv = P[n2 + node];
  if (Ynext) {
    pl += Ynext[node];
    pu += Ynext[n + node];
    pv += Ynext[n2 + node];
  }
  if (nx.Y) {
    Ybar[node] = yl;
    Ybar[n + node] = yu;
    Ybar[n2 + node] = yv;
    if (Ynext) {
      P[node] = pl;
      P[n + node] = pu;
      P[n2 + node] = pv;
    }
    adj_point(node, n, nx.Y, nx.sums, nx.dtb * pl + nx.dta * yl, nx.dtb * pu + nx.dta * yu,
              nx.dtb * pv + nx.dta * yv, fl, nx.g, nx.loc);
  } else {
    // qbar = P_1 + Ybar_2 + Ybar_1
    const double ql = pl + yl, qu = pu + yu, qv = pv + yv;
    nx.qbar[node] = ql;
    nx.qbar[n + node] = qu;
    nx.qbar[n2 + node] = qv;
    if (nx.kq) store_kq(nx.kq, node, nx.kappa[node], ql, qu, qv);
  }
}

// Filter adjoint P = qbar + A_hyp^T (kappa qbar) per field, then the pointwise
// part of stage 4 (its rates' adjoints are dtb P).
template <int LPN, int PAIRS>
__global__ void __launch_bounds__(256)
adj_filter_kernel(const int* __restrict__ tptr, const int* __restrict__ tsrc,
                  const double* __restrict__ twhyp, long long nnz,
                  const double* __restrict__ Shyp, const double* __restrict__ kq,
                  const double* __restrict__ qbar, int n, double* __restrict__ P, Flow fl,
                  AdjNext nx) {
  const int gid = static_cast<int>(xcd_tile(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x);
  const int node = gid / LPN;
  const int sub = gid % LPN;
  if (node >= n) return;
  const long long n2 = 2 * static_cast<long long>(n);
  double sl = 0.0, su = 0.0, sv = 0.0;
  const int e0 = tptr[node], e1 = tptr[node + 1];
  for (int e = (e0 & ~1) + 2 * sub; e < e1; e += 2 * LPN) {
    const int2 src = pair_sources(tsrc, e, e0, e1, node);
    const double2 a = edge_pair<PAIRS == kAllPairs>(twhyp, e, nnz);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bool in = q ? e + 1 < e1 : e >= e0;
      const double w = in ? (q ? a.y : a.x) : 0.0;
      const double2* ki = reinterpret_cast<const double2*>(kq + 4LL * (q ? src.y : src.x));
      const double2 lu = ki[0];
      sl = fma(w, lu.x, sl);
      su = fma(w, lu.y, su);
      sv = fma(w, ki[1].x, sv);
    }
  }
  sl = group_sum<LPN>(sl);
  su = group_sum<LPN>(su);
  sv = group_sum<LPN>(sv);
  if (sub != 0) return;
  const double s = Shyp[node];
  const double2* kj = reinterpret_cast<const double2*>(kq + 4LL * node);
  const double pl = qbar[node] + (sl - s * kj[0].x);
  const double pu = qbar[n + node] + (su - s * kj[0].y);
  const double pv = qbar[n2 + node] + (sv - s * kj[1].x);
  P[node] = pl;
  P[n + node] = pu;
  P[n2 + node] = pv;
  adj_point(node, n, nx.Y, nx.sums, nx.dtb * pl, nx.dtb * pu, nx.dtb * pv, fl, nx.g, nx.loc);
}

// Without the filter: P = qbar and the pointwise part of stage 4.
__global__ void __launch_bounds__(256)
adj_start_kernel(const double* __restrict__ qbar, int n, double* __restrict__ P, Flow fl,
                 AdjNext nx) {
  const int node = blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= n) return;
  const long long n2 = 2 * static_cast<long long>(n);
  const double pl = qbar[node], pu = qbar[n + node], pv = qbar[n2 + node];
  P[node] = pl;
  P[n + node] = pu;
  P[n2 + node] = pv;
  adj_point(node, n, nx.Y, nx.sums, nx.dtb * pl, nx.dtb * pu, nx.dtb * pv, fl, nx.g, nx.loc);
}

// qbar = qbar_end, and kappa qbar when kq is set.
__global__ void __launch_bounds__(256)
adj_seed_kernel(const double* __restrict__ end, const double* __restrict__ kappa, int n,
                double* __restrict__ qbar, double* __restrict__ kq) {
  const int node = blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= n) return;
  const long long n2 = 2 * static_cast<long long>(n);
  const double ql = end[node], qu = end[n + node], qv = end[n2 + node];
  qbar[node] = ql;
  qbar[n + node] = qu;
  qbar[n2 + node] = qv;
  if (kq) store_kq(kq, node, kappa[node], ql, qu, qv);
}

long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }

}  // namespace
}  // namespace labfm

using namespace labfm;

extern "C" size_t labfm_transpose_workspace_bytes(int32_t n, int64_t nnz) {
  if (n <= 0 || nnz < 0) return 0;
  return align256(sizeof(int) * (2 * (static_cast<size_t>(n) + 1) + static_cast<size_t>(nnz) + 1));
}

extern "C" int labfm_build_transpose(const labfm_operators* ops, int32_t* tptr, int32_t* tsrc,
                                     double* tw, void* workspace, size_t workspace_bytes,
                                     void* stream_) {
  clear_error();
  LABFM_REQUIRE(ops && ops->n > 0 && ops->row_ptr && ops->w && tptr && tsrc && tw,
                "build_transpose: bad arguments");
  const int n = ops->n;
  const long long nnz = ops->nnz;
  LABFM_REQUIRE(nnz == 0 || ops->col, "build_transpose: missing col");
  LABFM_WORKSPACE(workspace, workspace_bytes, labfm_transpose_workspace_bytes(n, nnz),
                  "build_transpose");
  hipStream_t st = as_stream(stream_);
  int* tmp = static_cast<int*>(workspace);
  int* cnt = tmp;
  int* cursor = cnt + n + 1;
  int* tslot = cursor + n + 1;
  const int T = 256;
  const unsigned ge = static_cast<unsigned>(std::min<long long>(65535, ceil_div(nnz + 1, T)));
  hipError_t e = hipMemsetAsync(tmp, 0, sizeof(int) * 2 * (static_cast<size_t>(n) + 1), st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(tcount_kernel, dim3(ge), dim3(T), 0, st, ops->col, nnz, cnt);
    hipLaunchKernelGGL(tscan_kernel, dim3(1), dim3(kScan), 0, st, cnt, tptr, n);
    hipLaunchKernelGGL(tfill_kernel, dim3(blocks_for(n, T)), dim3(T), 0, st, ops->row_ptr,
                       ops->col, n, tptr, cursor, tsrc, tslot);
    hipLaunchKernelGGL(tsort_kernel, dim3(blocks_for(n, T)), dim3(T), 0, st, tptr, n, tsrc, tslot);
    hipLaunchKernelGGL(tweights_kernel, dim3(ge), dim3(T), 0, st, ops->w, tslot, nnz, tw);
    e = hipGetLastError();
  }
  LABFM_HIP(e);
  return LABFM_OK;
}

namespace labfm {
namespace {
// Doubles per node of a reversed step's registers. The most that is live at one
// time, in the filter's gather, fills them; what comes later lies where
// something has been read for the last time:
//   sums of stages 1..4   then the operator-sum adjoints of stages 3 and 1
//                         (g[0]) over those of stage 4
//   g[1], loc[1]          the adjoints of stages 4 and 2, their pointwise terms
//   kq                    kappa qbar
//   qbar                  then Ybar_4, then the step's result
//   Y2                    then Ybar_2; the forward steps' register
//   Y3                    then Ybar_3; the forward steps' other register
//   Y4                    then loc[0]
//   qs                    the recomputed step's q, then P
// No kernel writes what it also reads.
constexpr int kAdjRegs = 4 * kStageSums + kAdj + 3 + 4 + 5 * 3;
static_assert(kAdj <= kStageSums && kStageSums % 2 == 0 && kAdj % 2 == 0,
              "g[0] in the sums of a stage, all on 16 bytes");
}  // namespace
}  // namespace labfm

extern "C" size_t labfm_adjoint_workspace_bytes(int32_t n, int32_t n_steps, int32_t ckpt_every) {
  if (n <= 0 || n_steps < 0 || ckpt_every <= 0) return 0;
  // checkpoints, one recomputed segment, and a reversed step's registers
  const long long nck = ceil_div(n_steps, ckpt_every);
  const long long doubles = 3LL * n * (nck + ckpt_every) + static_cast<long long>(kAdjRegs) * n;
  return static_cast<size_t>(doubles) * sizeof(double) + 512;
}

extern "C" int labfm_rk_adjoint(const double* q0, const double* qbar_end, double* qbar_0,
                                const labfm_operators* ops, const labfm_transpose* tr,
                                const labfm_rk_params* prm, int32_t n_steps, int32_t ckpt_every,
                                void* workspace, size_t workspace_bytes, void* stream_) {
  clear_error();
  LABFM_REQUIRE(ops && ops->n > 0 && ops->w && ops->row_ptr && ops->kappa,
                "rk_adjoint: float64 operators with kappa required");
  if (ops->wall_normal) {
    set_error("rk_adjoint: operators with wall nodes are not supported");
    return LABFM_ERR_UNSUPPORTED;
  }
  LABFM_REQUIRE(tr && tr->tptr && tr->tsrc && tr->tw && tr->rowsum,
                "rk_adjoint: transposed stencils and row sums required");
  LABFM_REQUIRE(q0 && qbar_end && qbar_0 && prm, "rk_adjoint: null argument");
  LABFM_REQUIRE(n_steps >= 0 && ckpt_every > 0, "rk_adjoint: bad step counts");
  LABFM_REQUIRE(prm->dt > 0.0, "rk_adjoint: dt must be positive");
  const int n = ops->n;
  const size_t need = labfm_adjoint_workspace_bytes(n, n_steps, ckpt_every);
  LABFM_REQUIRE(workspace && workspace_bytes >= need, "rk_adjoint: workspace of %zu bytes required",
                need);
  hipStream_t st = as_stream(stream_);
  const long long N3 = 3LL * n;
  const size_t b3 = sizeof(double) * N3;
  // kAdjRegs says what lies where; the records read with 16-byte loads first, on
  // a 16-byte boundary
  double* sums = reinterpret_cast<double*>((reinterpret_cast<uintptr_t>(workspace) + 15) &
                                           ~static_cast<uintptr_t>(15));
  double* g[2];
  g[0] = sums + 3LL * kStageSums * n;
  g[1] = sums + 4LL * kStageSums * n;
  double* kq = g[1] + static_cast<long long>(kAdj) * n;
  double* loc[2];
  loc[1] = kq + 4LL * n;
  double* qbar = loc[1] + N3;
  double* Y2 = qbar + N3;
  double* Y3 = Y2 + N3;
  double* Y4 = Y3 + N3;
  double* qs = Y4 + N3;
  double* ck = qs + N3;
  double* seg = ck + ceil_div(n_steps, ckpt_every) * N3;
  loc[0] = Y4;
  double* P = qs;

  const Flow fl{prm->c2, prm->mu, prm->gx, prm->gy};
  const double dt = prm->dt;
  StepPlan plan;
  plan.ops = ops;
  plan.w = ops->w;
  plan.prec = LABFM_F64;
  plan.stage_cfg = cfg_for(LABFM_KERNEL_STAGE, LABFM_F64, n, ops->nnz);
  plan.filter_cfg = cfg_for(LABFM_KERNEL_FILTER, LABFM_F64, n, ops->nnz);
  plan.fl = fl;
  plan.dt = dt;
  plan.filter = prm->filter;
  plan.Ya = Y2;
  plan.Yb = Y3;
  const LaunchCfg scfg = plan.stage_cfg;
  const long long nnz = ops->nnz;
  const unsigned grid = blocks_for(static_cast<long long>(n) * kAdjLpn, 256);
  const unsigned grid1 = blocks_for(n, 256);
  const int pairs = reinterpret_cast<uintptr_t>(tr->tw) % 16 != 0
                        ? kNoPairs
                        : (nnz % 2 != 0 ? kEvenPairs : kAllPairs);
  const auto transpose = pairs == kAllPairs    ? adj_transpose_kernel<kAdjLpn, kAllPairs>
                         : pairs == kEvenPairs ? adj_transpose_kernel<kAdjLpn, kEvenPairs>
                                               : adj_transpose_kernel<kAdjLpn, kNoPairs>;
  const auto filter = pairs == kAllPairs ? adj_filter_kernel<kAdjLpn, kAllPairs>
                                         : adj_filter_kernel<kAdjLpn, kNoPairs>;

  // forward pass up to the last checkpoint
  const long long nseg = ceil_div(n_steps, ckpt_every);
  LABFM_HIP(hipMemcpyAsync(seg, q0, b3, hipMemcpyDeviceToDevice, st));
  for (long long s = 0; s < nseg; ++s) {
    LABFM_HIP(hipMemcpyAsync(ck + s * N3, seg, b3, hipMemcpyDeviceToDevice, st));
    if (s + 1 == nseg) break;
    plan.Q = seg;
    for (int k = 0; k < ckpt_every; ++k) LABFM_HIP(enqueue_step<F64>(plan, st, nullptr));
  }

  hipLaunchKernelGGL(adj_seed_kernel, dim3(grid1), dim3(256), 0, st, qbar_end, ops->kappa, n, qbar,
                     prm->filter ? kq : nullptr);
  LABFM_LAUNCHED();
  for (long long s = nseg - 1; s >= 0; --s) {
    const int k0 = static_cast<int>(s * ckpt_every);
    const int k1 = std::min(n_steps, k0 + ckpt_every);
    // recompute the segment's states q_k0 .. q_{k1-1}
    LABFM_HIP(hipMemcpyAsync(seg, ck + s * N3, b3, hipMemcpyDeviceToDevice, st));
    for (int k = k0 + 1; k < k1; ++k) {
      double* dst = seg + static_cast<long long>(k - k0) * N3;
      LABFM_HIP(hipMemcpyAsync(dst, dst - N3, b3, hipMemcpyDeviceToDevice, st));
      plan.Q = dst;
      LABFM_HIP(enqueue_step<F64>(plan, st, nullptr));
    }
    for (int k = k1 - 1; k >= k0; --k) {
      const double* q = seg + static_cast<long long>(k - k0) * N3;
      // stage values Y2, Y3, Y4 of this step, and the operator sums at
      // Y1 = q, Y2, Y3 and Y4
      const double* Ys[4] = {q, Y2, Y3, Y4};
      double* to[4] = {Y2, Y3, Y4, nullptr};
      for (int i = 0; i < 4; ++i) {
        Flow fs = fl;
        fs.sums = sums + static_cast<long long>(i) * kStageSums * n;
        LABFM_HIP(launch_stage<F64>(scfg, ops, ops->w, Ys[i], i == 0 ? q : qs, qs, to[i],
                                    i < 3 ? dt * kA[i] : 0.0, dt * kB[i], fs, st, i & 1));
      }
      // the pointwise part of stage i, from the kernel that comes before its
      // transposed gather
      auto next = [&](int i) {
        AdjNext nx{};
        if (i >= 0) {
          nx.Y = Ys[i];
          nx.sums = sums + static_cast<long long>(i) * kStageSums * n;
          nx.dtb = dt * kB[i];
          nx.dta = i == 3 ? 0.0 : dt * kA[i];
          nx.g = g[i % 2];
          nx.loc = loc[i % 2];
        } else {
          nx.qbar = qbar;
          nx.kq = prm->filter ? kq : nullptr;
          nx.kappa = ops->kappa;
        }
        return nx;
      };
      // filter adjoint: P = qbar + A_hyp^T (kappa qbar)
      if (prm->filter) {
        hipLaunchKernelGGL(filter, dim3(grid), dim3(256), 0, st, tr->tptr, tr->tsrc,
                           tr->tw + LABFM_OP_HYP * nnz, nnz, tr->rowsum + LABFM_OP_HYP * n, kq,
                           qbar, n, P, fl, next(3));
      } else {
        hipLaunchKernelGGL(adj_start_kernel, dim3(grid1), dim3(256), 0, st, qbar, n, P, fl,
                           next(3));
      }
      LABFM_LAUNCHED();
      // stages 4 .. 1 (index i = 3 .. 0), Ybar_{i+1} to out[i]. Stage index
      // i's transposed gather folds Ybar_{i+2} into P (P_2 = P_3 + Ybar_4,
      // P_1 = P_2 + Ybar_3) before the pointwise part of stage i - 1; the last
      // one leaves qbar = P_1 + Ybar_2 + Ybar_1.
      double* out[4] = {nullptr, Y2, Y3, qbar};
      for (int i = 3; i >= 0; --i) {
        hipLaunchKernelGGL(transpose, dim3(grid), dim3(256), 0, st, tr->tptr, tr->tsrc, tr->tw, nnz,
                           tr->rowsum, g[i % 2], loc[i % 2], n, out[i], P,
                           i == 3 ? nullptr : out[i + 1], fl, next(i - 1));
        LABFM_LAUNCHED();
      }
    }
  }
  LABFM_HIP(hipMemcpyAsync(qbar_0, qbar, b3, hipMemcpyDeviceToDevice, st));
  return LABFM_OK;
}
