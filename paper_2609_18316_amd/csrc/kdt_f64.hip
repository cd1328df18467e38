// Float64 coordinates: the double-precision real kind of Sec. 2.4 (the
// paper's library picks float32 or float64 coordinates when it is compiled;
// here both live in one library and the float64 variant has entry points of
// its own).
//
// Build: the tree's shape (its splits and the tree order) is built by the
// float32 build from the coordinates rounded to float32 (clamped to the
// float32 range) -- any partition of the points gives correct queries, and
// the shape only steers the work.  The float64 coordinates are then stored in
// tree order and every node gets the tight float64 box of its own points,
// leaves from their points and inner nodes from their children, so pruning
// is exact for the float64 points.
//
// kNN (k <= 64) takes one traversal per lane, depth first, nearer child first, with the
// node stack in LDS; closed-ball counts and CSR lists share a traversal by the
// wave (kdt_packet.h) on median trees.  Squared distances are float64 sums over the
// axes in order, each operation rounded on its own; a node is pruned when its box distance is
// above the current k-th key's distance (kNN) or above fl64(r * r) (balls),
// and taken whole when its farthest corner is within the ball (Algorithm 3).
// Rounding is monotone, so a box bound computed this way never exceeds the
// computed distance of a point inside the box: no point that belongs to the
// answer is pruned.  Keys are (d2, index) pairs compared lexicographically,
// as in the float32 path; the candidate list is a sorted register array.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <climits>
#include <cmath>
#include <cstdint>

#include "kdt.h"
#include "kdt_internal.h"
#include "kdt_query.h"

namespace kdt {
namespace {

constexpr int kF64Block = 64;  // one wave per workgroup: the LDS stack is 4 B x depth per lane

__device__ __forceinline__ TreeView shape_view(const View64& v) {
  TreeView t{};
  t.rec = nullptr;
  t.box = nullptr;
  t.n = v.n;
  t.levels = v.levels;
  t.nodes = v.nodes;
  return t;
}

View64 view64(const kdt_tree* t) {
  return View64{t->rec64, t->box64, t->perm, t->n, t->levels, t->nodes, visit_counters()};
}

__global__ void k_to_f32(const double* __restrict__ x, int64_t m, float* __restrict__ y,
                         int32_t* __restrict__ bad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const double v = x[i];
  if (!isfinite(v)) {
    atomicOr(bad, 1);
    y[i] = 0.0f;
    return;
  }
  y[i] = (float)fmin(fmax(v, -(double)FLT_MAX), (double)FLT_MAX);
}

template <int D>
__global__ void k_gather64(const double* __restrict__ x, const int32_t* __restrict__ perm,
                           int64_t n, double* __restrict__ rec) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int64_t i = perm[t];
#pragma unroll
  for (int a = 0; a < D; ++a) rec[t * D + a] = x[i * D + a];
}

// Leaves: the tight box of their points (an empty range gives lo = +inf,
// hi = -inf, a box every bound prunes).
template <int D, typename Shape>
__global__ void k_leaf_boxes64(View64 v, int64_t n_nodes, double* __restrict__ box) {
  const int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= n_nodes) return;
  const Shape shape(shape_view(v));
  if (!shape.is_leaf((uint32_t)node)) return;
  int64_t b, e;
  shape.range((uint32_t)node, b, e);
  double lo[D], hi[D];
#pragma unroll
  for (int a = 0; a < D; ++a) lo[a] = INFINITY, hi[a] = -INFINITY;
  for (int64_t r = b; r < e; ++r)
#pragma unroll
    for (int a = 0; a < D; ++a) {
      const double c = v.rec[r * D + a];
      lo[a] = fmin(lo[a], c);
      hi[a] = fmax(hi[a], c);
    }
#pragma unroll
  for (int a = 0; a < D; ++a) box[node * 2 * D + a] = lo[a], box[node * 2 * D + D + a] = hi[a];
}

// Inner nodes of one level: the union of their children's boxes.
template <int D, typename Shape>
__global__ void k_inner_boxes64(View64 v, int64_t first, int64_t count, int level,
                                double* __restrict__ box) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int64_t node = first + i;
  if (v.nodes && v.nodes[node].w != level) return;
  const Shape shape(shape_view(v));
  if (shape.is_leaf((uint32_t)node)) return;
  const int64_t c = shape.left((uint32_t)node);
#pragma unroll
  for (int a = 0; a < D; ++a) {
    box[node * 2 * D + a] = fmin(box[c * 2 * D + a], box[(c + 1) * 2 * D + a]);
    box[node * 2 * D + D + a] =
        fmax(box[c * 2 * D + D + a], box[(c + 1) * 2 * D + D + a]);
  }
}

template <int D>
__device__ __forceinline__ double box_min64(const double* __restrict__ box, uint32_t node,
                                            const double q[D]) {
  const double* lo = box + (size_t)node * 2 * D;
  const double* hi = lo + D;
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    double t = 0.0;
    if (q[a] < lo[a])
      t = lo[a] - q[a];
    else if (q[a] > hi[a])
      t = q[a] - hi[a];
    s += t * t;
  }
  return s;
}

template <int D>
__device__ __forceinline__ double box_max64(const double* __restrict__ box, uint32_t node,
                                            const double q[D]) {
  const double* lo = box + (size_t)node * 2 * D;
  const double* hi = lo + D;
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const double t = fmax(fabs(q[a] - lo[a]), fabs(hi[a] - q[a]));
    s += t * t;
  }
  return s;
}

template <int D>
__device__ __forceinline__ double sq_dist64(const double* __restrict__ p, const double q[D]) {
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const double t = p[a] - q[a];
    s += t * t;
  }
  return s;
}

// The query of lane slot i: its coordinates and the output row.
template <int D>
__device__ __forceinline__ int64_t load_query64(const View64& v, const double* __restrict__ q,
                                                const int32_t* __restrict__ order, int64_t i,
                                                double qq[D]) {
  if (q) {
    const int64_t row = order ? order[i] : i;
#pragma unroll
    for (int a = 0; a < D; ++a) qq[a] = q[row * D + a];
    return row;
  }
#pragma unroll
  for (int a = 0; a < D; ++a) qq[a] = v.rec[i * D + a];
  return order ? i : v.perm[i];  // self queries: tree order when order is set
}

// (127 VGPRs; three waves per SIMD 2.15, four 2.03 ms)
template <int D, int KC>
constexpr int lane64_waves() {
  return ListMerge<TopK<KC>, D>::kOn ? 4 : 1;
}
// kNN over a median tree by keys of 64 bits, the float64 squared distance with the tree
// position in its lowest bits (Space64): they take the float32 path's lists and
// traversal (knn_median), where a (float64, index) list is 96 registers and
// 12 instructions per slot and insertion at k = 32 (216 VGPRs, two waves per SIMD;
// the call for 500009 queries on 2000003 clustered points 9.0 ms; now 1.95).  The keys keep the
// order of all but nearly equal distances, so the list holds the k nearest points
// unless the k-th key's distance bits are also those of a point that was turned away, or the
// list has room left (infinite distances and NaN have no key).
// Such a query is left to k_knn64 (todo); every other row gets its exact
// float64 distances, computed again from the list's positions, and runs of
// equal bits are put into (d2, index) order in place.
template <int D, int KC>
__global__ __launch_bounds__(kF64Block)
__attribute__((amdgpu_waves_per_eu(lane64_waves<D, KC>()))) void k_knn64_median(
    View64 v, const double* __restrict__ q, int64_t nq, int k, const int32_t* __restrict__ order,
    int32_t* __restrict__ out_idx, double* __restrict__ out_d2, int32_t* __restrict__ todo,
    int32_t* __restrict__ n_todo) {
  extern __shared__ uint32_t stk[];  // [levels + 1][kF64Block]
  const int64_t i = xcd_block<kXcdRunLane>() * kF64Block + threadIdx.x;
  if (i >= nq) return;
  double qq[D];
  const int64_t row = load_query64<D>(v, q, order, i, qq);
  TopKTie<KC> best;
  best.init(k);
  const uint32_t low = Space64<D>::low_bits(v.n);
  knn_median<D, ListMerge<TopK<KC>, D>::kOn>(Space64<D>{v, low}, qq, best, stk + threadIdx.x,
                                             kF64Block);
  double* d2 = out_d2 + row * k;
  int32_t* idx = out_idx ? out_idx + row * k : nullptr;
  bool runs = false;
  int have = 0;
#pragma unroll
  for (int j = 0; j < KC; ++j) {
    if (j < KC - k) continue;
    const uint64_t key = best.key(j);
    const bool empty = key == kEmptyKeyTie;
    have += !empty;
    const int64_t pos = empty ? 0 : (int64_t)((uint32_t)key & low);
    if (j > KC - k) runs |= !empty && ((key ^ best.key(j - 1)) & ~(uint64_t)low) == 0;
    d2[j - (KC - k)] = empty ? INFINITY : sq_dist<D>(v.rec + pos * D, qq);
    if (idx) idx[j - (KC - k)] = empty ? -1 : v.perm[pos];
  }
  const int m = (int)(v.n < k ? v.n : k);
  const uint64_t lost = (uint64_t)__double_as_longlong(best.lost);
  if (have < m || (v.n > k && (lost & ~(uint64_t)low) <= (best.worst() & ~(uint64_t)low))) {
    todo[atomicAdd(n_todo, 1)] = (int32_t)i;
  } else if (runs) {
    for (int a = 1; a < m; ++a) {
      const double d = d2[a];
      const int32_t id = idx ? idx[a] : 0;
      int b = a;
      for (; b > 0 && (d < d2[b - 1] || (idx && d == d2[b - 1] && id < idx[b - 1])); --b) {
        d2[b] = d2[b - 1];
        if (idx) idx[b] = idx[b - 1];
      }
      d2[b] = d;
      if (idx) idx[b] = id;
    }
  }
}

// kNN by exact (d2, index) lists: sliding-midpoint trees (some == NULL), and
// the *n_some queries some[] that k_knn64_median has left (order positions).
template <int D, int KC, typename Shape>
__global__ __launch_bounds__(kF64Block) void k_knn64(View64 v, const double* __restrict__ q,
                                                     int64_t nq, int k,
                                                     const int32_t* __restrict__ order,
                                                     int32_t* __restrict__ out_idx,
                                                     double* __restrict__ out_d2, int depth,
                                                     const int32_t* __restrict__ some,
                                                     const int32_t* __restrict__ n_some) {
  extern __shared__ uint32_t stk[];  // [depth][kF64Block]
  int64_t i = (int64_t)blockIdx.x * kF64Block + threadIdx.x;
  if (i >= (some ? (int64_t)*n_some : nq)) return;
  if (some) i = some[i];
  double qq[D];
  const int64_t row = load_query64<D>(v, q, order, i, qq);
  const Shape shape(shape_view(v));
  double kd[KC];
  int32_t ki[KC];
  double wd = INFINITY;  // the k-th key
  int32_t wi = INT_MAX;
  if (some) {
    // the row holds k points already: none farther than they are can matter
    wd = 0.0;
    for (int j = 0; j < k; ++j) wd = fmax(wd, out_d2[row * k + j]);
  }
#pragma unroll
  for (int j = 0; j < KC; ++j) kd[j] = wd, ki[j] = INT_MAX;
  int sp = 0;
  uint32_t node = 0;
  bool have = true;
  while (have) {
    if (shape.is_leaf(node)) {
      int64_t b, e;
      shape.range(node, b, e);
      for (int64_t r = b; r < e; ++r) {
        double d = sq_dist64<D>(v.rec + r * D, qq);
        int32_t id = v.perm[r];
        if (!(d < wd || (d == wd && id < wi))) continue;
#pragma unroll
        for (int j = 0; j < KC; ++j) {
          const bool lt = d < kd[j] || (d == kd[j] && id < ki[j]);
          const double td = kd[j];
          const int32_t ti = ki[j];
          kd[j] = lt ? d : td;
          ki[j] = lt ? id : ti;
          d = lt ? td : d;
          id = lt ? ti : id;
        }
#pragma unroll
        for (int j = 0; j < KC; ++j)
          if (j == k - 1) wd = kd[j], wi = ki[j];
      }
    } else {
      const uint32_t l = shape.left(node), r = l + 1;
      const double dl = box_min64<D>(v.box, l, qq), dr = box_min64<D>(v.box, r, qq);
      const uint32_t nearc = dl <= dr ? l : r, farc = dl <= dr ? r : l;
      const double dn = fmin(dl, dr), df = fmax(dl, dr);
      if (df <= wd) stk[(sp++) * kF64Block + threadIdx.x] = farc;
      if (dn <= wd) {
        node = nearc;
        continue;
      }
    }
    // pop the next node still within reach
    have = false;
    while (sp > 0) {
      const uint32_t c = stk[(--sp) * kF64Block + threadIdx.x];
      if (box_min64<D>(v.box, c, qq) <= wd) {
        node = c;
        have = true;
        break;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < KC; ++j)
    if (j < k) {
      const bool pad = ki[j] == INT_MAX;
      if (out_idx) out_idx[row * k + j] = pad ? -1 : ki[j];
      out_d2[row * k + j] = pad ? INFINITY : kd[j];
    }
}

// Closed-ball counts (FILL false) or lists (FILL true: the input indices of
// row `row` written from offsets[row] on, in traversal order).  apart: only the waves
// that the wave-shared counts leave out.
template <int D, bool FILL, typename Shape>
__global__ __launch_bounds__(kF64Block) void k_range64(View64 v, const double* __restrict__ q,
                                                       int64_t nq, double r2,
                                                       const int32_t* __restrict__ order,
                                                       int32_t* __restrict__ count,
                                                       const int64_t* __restrict__ offsets,
                                                       int32_t* __restrict__ out, int depth,
                                                       bool apart) {
  extern __shared__ uint32_t stk[];
  const int64_t i = (int64_t)blockIdx.x * kF64Block + threadIdx.x;
  if constexpr (!FILL && D <= 4) {
    if (apart && lie_together<D>(q, nq, (int64_t)blockIdx.x * kF64Block)) return;
  }
  if (i >= nq) return;
  double qq[D];
  const int64_t row = load_query64<D>(v, q, order, i, qq);
  const Shape shape(shape_view(v));
  int64_t c = 0;
  int64_t at = FILL ? offsets[row] : 0;
  int sp = 0;
  stk[(sp++) * kF64Block + threadIdx.x] = 0;
  while (sp > 0) {
    const uint32_t node = stk[(--sp) * kF64Block + threadIdx.x];
    if (box_min64<D>(v.box, node, qq) > r2) continue;
    int64_t b, e;
    if (box_max64<D>(v.box, node, qq) <= r2) {
      shape.range(node, b, e);
      if (FILL)
        for (int64_t t = b; t < e; ++t) out[at++] = v.perm[t];
      c += e - b;
      continue;
    }
    if (shape.is_leaf(node)) {
      shape.range(node, b, e);
      for (int64_t t = b; t < e; ++t)
        if (sq_dist64<D>(v.rec + t * D, qq) <= r2) {
          if (FILL) out[at++] = v.perm[t];
          ++c;
        }
      continue;
    }
    const uint32_t l = shape.left(node);
    stk[(sp++) * kF64Block + threadIdx.x] = l + 1;
    stk[(sp++) * kF64Block + threadIdx.x] = l;
  }
  if (!FILL) count[row] = (int32_t)c;
}

__global__ void k_zero64(int32_t* p, int64_t* q) {
  if (p) *p = 0;
  if (q) *q = 0;
}

bool dim_ok64(int d) { return d == 2 || d == 3 || d == 4 || d == 8 || d == 16; }

template <typename F>
kdt_status by_dim(int d, F&& f) {
  switch (d) {
    case 2: return f(std::integral_constant<int, 2>());
    case 3: return f(std::integral_constant<int, 3>());
    case 4: return f(std::integral_constant<int, 4>());
    case 8: return f(std::integral_constant<int, 8>());
    case 16: return f(std::integral_constant<int, 16>());
  }
  return KDT_EUNSUPPORTED;
}

// Stack entries a traversal can hold: the depth-first kNN keeps one pending
// sibling per level, the ball traversal two children per level.
int stack_depth(const kdt_tree* t) { return 2 * (t->levels + 1) + 2; }

// Above so many external queries in input order, on trees of at least so many points and in up
// to 4 dimensions, waves of queries that do not lie together take a traversal per lane:
// shared, 64 strangers visit the union of their paths.
// Balls of 50 points, us per lane / shared / so: 300000 in random order of 300000 uniform points
// 1606 / 3839 / 1641, 10^6 of 2000003 4828 / 10673 / 4944; in the order of a curve
// 877 / 318 / 329.  Few queries in a large clustered tree are the exception (65536 in random order
// of 2000003 points 3378 / 1048 / 3162: the lanes wait for the halos).  Below the lines the shared
// ones win in any order (100000 of 1000 points 230 / 184, 20000 of 300000 610 / 478; d = 8, 65536
// of 20000 5828 / 1223).
constexpr int64_t kUnsortedRows = int64_t(1) << 15;
constexpr int64_t kUnsortedPoints = int64_t(1) << 13;

// The query order (Hilbert curve over the root box, d <= 4; tree leaf
// otherwise), taken from the float32 rounding of the queries.
kdt_status order64(const kdt_tree* t, const double* d_q, int64_t nq, PoolBuffers& buf,
                   int32_t** order, hipStream_t stream) {
  float* qf = nullptr;
  int32_t* bad = nullptr;
  int32_t* ord = nullptr;
  if (!buf.get(&qf, (size_t)nq * t->d) || !buf.get(&bad, 1) || !buf.get(&ord, (size_t)nq)) {
    kdt_set_error("float64 queries: device allocation failed for the query order");
    return KDT_ENOMEM;
  }
  const int64_t m = nq * t->d;
  k_to_f32<<<(unsigned)((m + 255) / 256), 256, 0, stream>>>(d_q, m, qf, bad);
  const kdt_status st = kdt_query_order(t, qf, nq, 0, ord, stream);
  if (st != KDT_OK) return st;
  *order = ord;
  return KDT_OK;
}

}  // namespace

}  // namespace kdt

using namespace kdt;

extern "C" kdt_status kdt_build_f64(const double* d_pts, int64_t n, int32_t d,
                                    const kdt_build_opts* opts, hipStream_t stream,
                                    kdt_tree** out) {
  kdt_clear_error();
  if (!out || !d_pts || n < 1 || n > INT32_MAX) {
    kdt_set_error("kdt_build_f64: NULL pointer or n=%lld outside [1, 2^31-1]", (long long)n);
    return KDT_EINVAL;
  }
  *out = nullptr;
  if (!dim_ok64(d)) {
    kdt_set_error("kdt_build_f64: dimension %d is not one of 2, 3, 4, 8, 16", d);
    return KDT_EUNSUPPORTED;
  }
  const bool check = opts ? opts->check_finite != 0 : true;
  PoolBuffers buf(stream);
  float* xf = nullptr;
  int32_t* bad = nullptr;
  if (!buf.get(&xf, (size_t)n * d) || !buf.get(&bad, 1)) {
    kdt_set_error("kdt_build_f64: device allocation failed (%lld points)", (long long)n);
    return KDT_ENOMEM;
  }
  k_zero64<<<1, 1, 0, stream>>>(bad, nullptr);
  const int64_t m = n * d;
  k_to_f32<<<(unsigned)((m + 255) / 256), 256, 0, stream>>>(d_pts, m, xf, bad);
  if (check) {
    int32_t h = 0;
    if (hipMemcpyAsync(&h, bad, sizeof(h), hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess) {
      kdt_set_error("kdt_build_f64: reading the finiteness flag failed");
      return KDT_EDEVICE;
    }
    if (h) {
      kdt_set_error("kdt_build_f64: non-finite coordinate (NaN or Inf)");
      return KDT_EINVAL;
    }
  }
  kdt_build_opts o{};
  if (opts) o = *opts;
  o.check_finite = 0;  // the float32 copy is finite by construction
  kdt_tree* t = nullptr;
  kdt_status st = kdt_build(xf, n, d, &o, stream, &t);
  if (st != KDT_OK) return st;
  const size_t b_rec = sizeof(double) * (size_t)n * d;
  const size_t b_box = sizeof(double) * (size_t)t->n_nodes * 2 * d;
  void* block = nullptr;
  if (dev_alloc(&block, ((b_rec + 255) & ~size_t(255)) + b_box, stream) != hipSuccess) {
    kdt_free(t);
    kdt_set_error("kdt_build_f64: cannot allocate the float64 tree (%lld points)", (long long)n);
    return KDT_ENOMEM;
  }
  t->f64_block = block;
  t->rec64 = static_cast<double*>(block);
  t->box64 = reinterpret_cast<double*>(static_cast<char*>(block) + ((b_rec + 255) & ~size_t(255)));
  const View64 v = view64(t);
  st = by_dim(d, [&](auto dd) -> kdt_status {
    constexpr int D = decltype(dd)::value;
    k_gather64<D><<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(d_pts, t->perm, n, t->rec64);
    const unsigned gn = (unsigned)((t->n_nodes + 255) / 256);
    if (t->nodes) {
      k_leaf_boxes64<D, StoredShape><<<gn, 256, 0, stream>>>(v, t->n_nodes, t->box64);
      for (int l = t->levels - 1; l >= 0; --l)
        k_inner_boxes64<D, StoredShape><<<gn, 256, 0, stream>>>(v, 0, t->n_nodes, l, t->box64);
    } else {
      k_leaf_boxes64<D, MedianShape><<<gn, 256, 0, stream>>>(v, t->n_nodes, t->box64);
      for (int l = t->levels - 1; l >= 0; --l) {
        const int64_t first = (int64_t(1) << l) - 1, count = int64_t(1) << l;
        k_inner_boxes64<D, MedianShape><<<(unsigned)((count + 255) / 256), 256, 0, stream>>>(
            v, first, count, l, t->box64);
      }
    }
    return hipGetLastError() == hipSuccess ? KDT_OK : KDT_EDEVICE;
  });
  if (st != KDT_OK) {
    kdt_free(t);
    kdt_set_error("kdt_build_f64: kernel launch failed");
    return st;
  }
  *out = t;
  return KDT_OK;
}

extern "C" kdt_status kdt_knn_f64(const kdt_tree* tree, const double* d_q, int64_t nq, int32_t k,
                                  int32_t* d_idx, double* d_d2, const kdt_query_opts* opts,
                                  hipStream_t stream) {
  kdt_clear_error();
  if (tree && tree->rec64 && nq == 0 && k >= 1 && k <= KDT_MAX_K) return KDT_OK;
  if (!tree || !tree->rec64 || !d_d2 || nq < 0 || nq > INT32_MAX) {
    kdt_set_error("kdt_knn_f64: NULL tree or output, a tree not built by kdt_build_f64, or nq "
                  "outside [0, 2^31-1]");
    return KDT_EINVAL;
  }
  if (k < 1) {
    kdt_set_error("kdt_knn_f64: k=%d below 1", k);
    return KDT_EINVAL;
  }
  if (k > KDT_MAX_K) {
    kdt_set_error("kdt_knn_f64: k=%d above %d", k, KDT_MAX_K);
    return KDT_EUNSUPPORTED;
  }
  if (opts && opts->period) {
    kdt_set_error("kdt_knn_f64: periodic boundaries are not available for float64 coordinates");
    return KDT_EUNSUPPORTED;
  }
  if (!d_q && nq != tree->n) {
    kdt_set_error("kdt_knn_f64: self queries need nq == n (%lld)", (long long)tree->n);
    return KDT_EINVAL;
  }
  const int32_t* rows = nullptr;
  const kdt_status rs = self_rows(tree, d_q, opts, "kdt_knn_f64", &rows);
  if (rs != KDT_OK) return rs;
  PoolBuffers buf(stream);
  // self queries: the tree-order row marker (or NULL)
  const int32_t* order = d_q ? (opts ? opts->order : nullptr) : rows;
  int32_t* own = nullptr;
  if (d_q && !order && (!opts || opts->sort_queries) && nq > 1) {
    const kdt_status st = order64(tree, d_q, nq, buf, &own, stream);
    if (st != KDT_OK) return st;
    order = own;
  }
  const View64 v = view64(tree);
  const int depth = stack_depth(tree);
  const size_t smem = sizeof(uint32_t) * (size_t)depth * kF64Block;
  const size_t smem1 = sizeof(uint32_t) * (size_t)(tree->levels + 1) * kF64Block;
  const unsigned g = (unsigned)((nq + kF64Block - 1) / kF64Block);
  int32_t *todo = nullptr, *n_todo = nullptr;
  if (!tree->nodes && (!buf.get(&todo, (size_t)nq) || !buf.get(&n_todo, 1))) {
    kdt_set_error("kdt_knn_f64: device allocation failed");
    return KDT_ENOMEM;
  }
  const kdt_status st = by_dim(tree->d, [&](auto dd) -> kdt_status {
    constexpr int D = decltype(dd)::value;
    auto go = [&](auto kc) {
      constexpr int KC = decltype(kc)::value;
      if (tree->nodes) {
        k_knn64<D, KC, StoredShape><<<g, kF64Block, smem, stream>>>(
            v, d_q, nq, k, order, d_idx, d_d2, depth, nullptr, nullptr);
      } else {
        k_zero64<<<1, 1, 0, stream>>>(n_todo, nullptr);
        k_knn64_median<D, KC><<<g, kF64Block, smem1, stream>>>(v, d_q, nq, k, order, d_idx, d_d2,
                                                               todo, n_todo);
        k_knn64<D, KC, MedianShape><<<g, kF64Block, smem, stream>>>(
            v, d_q, nq, k, order, d_idx, d_d2, depth, todo, n_todo);
      }
    };
    switch (lane_list(k, tree->n)) {
      case 8: go(std::integral_constant<int, 8>()); break;
      case 16: go(std::integral_constant<int, 16>()); break;
      case 32: go(std::integral_constant<int, 32>()); break;
      default: go(std::integral_constant<int, 64>());
    }
    return hipGetLastError() == hipSuccess ? KDT_OK : KDT_EDEVICE;
  });
  if (st != KDT_OK) kdt_set_error("kdt_knn_f64: kernel launch failed");
  return st;
}

extern "C" kdt_status kdt_range_f64(const kdt_tree* tree, const double* d_q, int64_t nq, double r,
                                    int32_t* d_count, int64_t* d_offsets, int32_t* d_idx,
                                    int64_t capacity, int64_t* required,
                                    const kdt_query_opts* opts, hipStream_t stream) {
  kdt_clear_error();
  if (tree && tree->rec64 && nq == 0 && r >= 0.0 && capacity >= 0) {
    if (required) *required = 0;
    if (d_offsets) k_zero64<<<1, 1, 0, stream>>>(nullptr, d_offsets);
    return hipGetLastError() == hipSuccess ? KDT_OK : KDT_EDEVICE;
  }
  if (!tree || !tree->rec64 || !d_count || nq < 0 || nq > INT32_MAX || !(r >= 0.0) ||
      capacity < 0 || (d_idx && !d_offsets)) {
    kdt_set_error("kdt_range_f64: NULL tree or counts, a tree not built by kdt_build_f64, nq "
                  "outside [0, 2^31-1], r not >= 0, negative capacity or lists without offsets");
    return KDT_EINVAL;
  }
  if (opts && opts->period) {
    kdt_set_error("kdt_range_f64: periodic boundaries are not available for float64 coordinates");
    return KDT_EUNSUPPORTED;
  }
  if (!d_q && nq != tree->n) {
    kdt_set_error("kdt_range_f64: self queries need nq == n (%lld)", (long long)tree->n);
    return KDT_EINVAL;
  }
  const int32_t* rows = nullptr;
  const kdt_status rs = self_rows(tree, d_q, opts, "kdt_range_f64", &rows);
  if (rs != KDT_OK) return rs;
  if (required) *required = 0;
  PoolBuffers buf(stream);
  const int32_t* order = opts ? opts->order : nullptr;
  int32_t* own = nullptr;
  if (d_q && !order && (!opts || opts->sort_queries) && nq > 1) {
    const kdt_status st = order64(tree, d_q, nq, buf, &own, stream);
    if (st != KDT_OK) return st;
    order = own;
  }
  if (!d_q) order = rows;  // self queries: the tree-order row marker (or NULL)
  const View64 v = view64(tree);
  const double r2 = r * r;
  const int depth = stack_depth(tree);
  const size_t smem = sizeof(uint32_t) * (size_t)depth * kF64Block;
  const unsigned g = (unsigned)((nq + kF64Block - 1) / kF64Block);
  // Median trees take the wave-shared counts (and their list fill): one
  // traversal per lane waits for the few lanes whose balls sit in a dense halo.
  // The call for 500009 balls of about 28 points on 2000003 clustered points took
  // 11.1 ms with a traversal per lane and takes 1.6 ms shared by a wave, its lists
  // 68 and 7.9 ms.  A leaf has to fit the wave's mask (64 points), and the
  // leaves and packed queries of a workgroup the 64 KiB of LDS a launch gets
  // (16 dimensions: leaves of up to 56 points).
  int cap = 0;
  // (a stored tree's depth is no shift: it may pass 64)
  const View64 vc = tree->nodes ? v : count_view(v, tree->leaf, &cap);
  const bool shared = !tree->nodes && cap <= 64 && range64_packet_lds(tree->d, cap) <= 65536;
  const bool apart = shared && d_q && !order && !d_offsets && nq > kUnsortedRows &&
                     v.n >= kUnsortedPoints && tree->d <= 4;
  int32_t* cur = nullptr;
  auto launch = [&](bool fill, int32_t* out) {
    return by_dim(tree->d, [&](auto dd) -> kdt_status {
      constexpr int D = decltype(dd)::value;
      if (shared) {
        const FillOut fo{out, d_offsets, cur};
        const kdt_status st = range64_packet_launch<D>(vc, cap, d_q, nq, r2, order, d_count,
                                                       stream, fill ? &fo : nullptr, apart);
        if (st != KDT_OK || !apart) return st;
        k_range64<D, false, MedianShape><<<g, kF64Block, smem, stream>>>(
            v, d_q, nq, r2, order, d_count, d_offsets, out, depth, true);
        return hipGetLastError() == hipSuccess ? KDT_OK : KDT_EDEVICE;
      }
      if (tree->nodes) {
        if (fill)
          k_range64<D, true, StoredShape><<<g, kF64Block, smem, stream>>>(
              v, d_q, nq, r2, order, d_count, d_offsets, out, depth, false);
        else
          k_range64<D, false, StoredShape><<<g, kF64Block, smem, stream>>>(
              v, d_q, nq, r2, order, d_count, d_offsets, out, depth, false);
      } else {
        if (fill)
          k_range64<D, true, MedianShape><<<g, kF64Block, smem, stream>>>(
              v, d_q, nq, r2, order, d_count, d_offsets, out, depth, false);
        else
          k_range64<D, false, MedianShape><<<g, kF64Block, smem, stream>>>(
              v, d_q, nq, r2, order, d_count, d_offsets, out, depth, false);
      }
      return hipGetLastError() == hipSuccess ? KDT_OK : KDT_EDEVICE;
    });
  };
  kdt_status st = launch(false, nullptr);
  if (st != KDT_OK) {
    if (st == KDT_EDEVICE) kdt_set_error("kdt_range_f64: kernel launch failed");
    return st;
  }
  if (!d_offsets) return KDT_OK;
  // offsets: exclusive running sum of the counts, then the total
  void* tmp = nullptr;
  if (!buf.get((char**)&tmp, scan_scratch_bytes(nq))) {
    kdt_set_error("kdt_range_f64: device allocation failed for the list offsets");
    return KDT_ENOMEM;
  }
  if (exclusive_scan<int64_t>(d_count, d_offsets, nq, d_offsets + nq, tmp, stream) != KDT_OK) {
    kdt_set_error("kdt_range_f64: offset scan failed");
    return KDT_EDEVICE;
  }
  int64_t total = 0;
  if (hipMemcpyAsync(&total, d_offsets + nq, sizeof(total), hipMemcpyDeviceToHost, stream) !=
          hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess) {
    kdt_set_error("kdt_range_f64: reading the list size failed");
    return KDT_EDEVICE;
  }
  if (required) *required = total;
  if (!d_idx) return KDT_OK;
  if (total > capacity) {
    kdt_set_error("kdt_range_f64: the lists need %lld entries, capacity is %lld",
                  (long long)total, (long long)capacity);
    return KDT_ECAPACITY;
  }
  if (total == 0) return KDT_OK;
  int32_t* unsorted = nullptr;
  if (!buf.get(&unsorted, (size_t)total) || (shared && !buf.get(&cur, (size_t)nq))) {
    kdt_set_error("kdt_range_f64: device allocation failed for the lists");
    return KDT_ENOMEM;
  }
  st = launch(true, unsorted);
  if (st != KDT_OK) {
    if (st == KDT_EDEVICE) kdt_set_error("kdt_range_f64: kernel launch failed");
    return st;
  }
  // every row ascending by input index
  st = sort_list_rows(unsorted, d_idx, d_offsets, nq, total, tree->n, stream);
  if (st != KDT_OK) return st;
  // the scratch goes back to the pool in stream order; the caller's arrays
  // are complete when the stream reaches this point
  return KDT_OK;
}
