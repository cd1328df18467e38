// kdt_packet.hip -- single-tree kernels of the wave-coherent traversals
// (kNN, Sec. 2.3 / Algorithm 2; ball counts, Algorithm 3) for gfx950.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kdt_packet.h"
#include "kdt_torus.h"

namespace kdt {

constexpr int kPWaves = 4;  // waves per workgroup (independent packets)
// Ball-count work splitting: passes; node visits per wave before it hands the
// rest of its stack on, in the first pass and in the later ones; task slots per
// pass; workgroups of a task pass.  A later pass walks its subtrees widest first
// (kWideBudget) and so cuts the largest of them into about as many parts as its
// budget; depth first, a hand-off's largest part was half of the subtree, and after
// 8 passes single waves still had 500 visits of 1.2 us before them.  Launches of few
// waves hand on at once, since most of the chip is idle (50021 queries, k = 1000 of
// 2^23 clustered points: 15.5 ms with 8 depth-first passes of 512 and 32 visits
// of one node; 14.3 with 256 and 16 of two nodes, 11.7 widest first, 10.2 with 24 and
// 24), unless the balls are small (131072 balls of 2 of 65536 points, us with the few
// waves' budget and without: 212 / 90); in large ones ordinary waves must not reach the budget
// (2^22 uniform balls, r = 0.01, of 2^24 uniform points: 4.29, 3.63 and 3.56 ms with 192, 320
// and 384; lists of 1000003 balls of clustered points 4.68, 4.98 and 5.22).  Where a pass has
// so many tasks that the chip stays full, cutting them into parts only fills the list, and a
// task that finds no room runs to its end whatever its size: there a task keeps
// kRangeManyBudget visits (131073 balls of r = 0.3 of 2^22 uniform points, ms: 18.6 with
// 8 depth-first passes, 22.5 without this rule, 18.6 so; clustered 14.8, 17.3, 13.8; lists of
// 1000003 balls 4.73 and 4.75).
constexpr int kRangePasses = 5;
constexpr uint32_t kRangeBudgetFirst = 320;
constexpr uint32_t kRangeBudget = 10;
constexpr uint32_t kRangeBudgetFew = 24;  // both budgets of launches of few waves:
constexpr int64_t kRangeFewWaves = 768;       // counts
constexpr int64_t kRangeFewWavesList = 2048;  // lists
// Counts of up to so many waves more: small balls should not hand on and large ones should
// (float64 counts over trees of 1000 to 8 * 10^6 points, time relative to the few waves' budgets,
// mean and worst: 40000 balls 1.03 and 1.24 so, 1.15 and 1.59 with the large launches' budgets;
// 65536 0.96 and 1.16, 1.01 and 1.38; 131072 0.86 and 1.08, 0.81 and 1.17).  Lists keep the
// few waves' budgets: their fill waits for single waves more than it loses by handing on (75931
// balls of 12 of 134189 clustered points 1.08 ms, 1.28 so and 1.43; of 131072 balls of 30 of
// 130000 uniform points the order is the other, up to 1.3).
constexpr int64_t kRangeMidWaves = 1024;
constexpr int64_t kRangeMidWaves64 = 2048;  // float64, which has no search by a wave per ball
constexpr uint32_t kRangeBudgetMid = 96;    // the first budget; the few waves' later one
constexpr uint32_t kRangeManyTasks = 300000;  // from here on:
constexpr uint32_t kRangeManyBudget = 96;     // the later budget
constexpr uint32_t kRangeTaskCap = 1u << 20;
// Task slots per wave of the first pass, where that is fewer (launches below 2^16
// queries): the lists' 67 MB for 2^20 slots are far more than a small call's own data.
// (256 per wave cost the counts of large k: 50021 queries, k = 1000, 15.9 -> 17.6 ms.)
constexpr int64_t kRangeTasksPerWave = 1024;
constexpr unsigned kRangeTaskBlocks = 8192;
// The first pass hands work on only once fewer than this many of its waves
// are left (half of what the chip holds at once: with all of it ordinary waves hand on too,
// 256 visits, 2^20 uniform balls 1.88 and 2.06 ms).
constexpr int64_t kRangeTailWaves = 4096;

// Up to this many shapes are counted by a wave each (wave_ball), above (and from d = 16
// on, where a ball cuts most nodes) by the wave-shared traversal of 64 shapes, whose few
// waves leave the chip idle in smaller launches.  A wave's search has a fixed cost of its own
// that a shared traversal of small balls in a small tree, above all in 2 dimensions, does
// not; the larger the tree and the higher the dimension, the longer the shared one.
// Ball counts, shared and by wave, us (balls of 30 points unless said): 1000 balls of 1000
// points 78 and 14; 65536 of 65536 169 and 107; 131072 of 4096 points 74 and 142, of 65536 120
// and 196, of 2^20 371 and 255; d = 2, 65536 of 65536 points 66 and 95, 131072 of 2^20 146 and
// 237; d = 4, 131072 of 65536 points 302 and 221; d = 8, 65536 of 300 points 77 and 87, 131072
// of 1000 139 and 192, of 16384 858 and 376.  Where the two are close the points decide: 75000
// balls of 130000 uniform points 160 and 130, of clustered ones 277 and 132, 131072 140 and 219,
// 281 and 221.
constexpr int64_t kWaveRowsMost = int64_t(1) << 17;
inline int64_t wave_rows(int d, int64_t n) {
  constexpr int64_t rows = int64_t(1) << 16;
  if (d == 2) return n >= (1 << 18) ? rows : rows / 2;
  const int64_t large = d == 3 ? 1 << 18 : d == 4 ? 1 << 16 : 1 << 12;
  if (n >= large) return 2 * rows;
  return d == 8 ? rows / 2 : d == 3 && n >= rows ? rows + rows / 4 : rows;
}
// The balls of large k hold many points: the 7 counts of 50021 balls of 2^23 clustered
// points took 4.0 ms and take 1.05; kNN with k = 100, 262000 queries 4.86 and 3.94 ms,
// 2^20 (k = 128) 13.7 and 15.1; d = 16, 5000: 50.6 and 54.0.
constexpr int64_t kWaveRowsLarge = int64_t(1) << 18;

// LDS of a workgroup of the grouping: a slice per wave.
template <int D>
size_t fof_lds_bytes(int leaf) {
  return sizeof(float) * fof_wave_floats<D>(leaf) * kPWaves;
}

template <int D>
__device__ __forceinline__ float* fof_slice(float* lds, int wave, int leaf_cap) {
  return lds + (size_t)wave * fof_wave_floats<D>(leaf_cap);
}

template <int D>
__device__ __forceinline__ bool load_query(const TreeView& t, const float* __restrict__ q,
                                           int64_t nq, const int32_t* __restrict__ order,
                                           int64_t s, float p[D], int64_t& row) {
  if (s >= nq) {
#pragma unroll
    for (int a = 0; a < D; ++a) p[a] = 0.0f;
    return false;
  }
  if (q == nullptr) {
    // self queries: row = input index, or s (tree order) when order is set
    int32_t id = 0;
    load_rec<D>(t.rec, s, p, id);
    row = order ? s : id;
  } else {
    row = order ? order[s] : s;
#pragma unroll
    for (int a = 0; a < D; ++a) p[a] = q[row * D + a];
  }
  return true;
}

template <int D>
__device__ __forceinline__ bool load_query(const View64& t, const double* __restrict__ q,
                                           int64_t nq, const int32_t* __restrict__ order,
                                           int64_t s, double p[D], int64_t& row) {
  const bool active = s < nq;
  row = !active ? 0 : order && q ? order[s] : order || q ? s : t.perm[s];
#pragma unroll
  for (int a = 0; a < D; ++a) p[a] = !active ? 0.0 : q ? q[row * D + a] : t.rec[s * D + a];
  return active;
}

// MODE 0 writes k (index, d2) pairs per row, 1 the k-th d2, 2 the k-th
// distance (a compile-time choice, so each output form is its own kernel).
template <int D, int KC, int MODE>
__global__ __launch_bounds__(64 * kPWaves) void k_knn_packet(TreeView t, const float* __restrict__ q,
                                                             int64_t nq, int k,
                                                             const int32_t* __restrict__ order,
                                                             int32_t* __restrict__ oidx,
                                                             float* __restrict__ od2, int leaf_cap) {
  extern __shared__ __align__(16) float lds[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t s0 = (xcd_block<kXcdRunPacket>() * kPWaves + wave) * 64;
  if (s0 >= nq) return;  // whole wave idle
  float p[D];
  int64_t row = 0;
  const bool active = load_query<D>(t, q, nq, order, s0 + lane, p, row);
  TopK<KC> best;
  best.init(k);
  packet_knn<D, KC>(t, p, active, best, lds + (size_t)wave * knn_wave_floats<D>(leaf_cap),
                    leaf_cap);
  if (active) knn_write<KC>(best, k, MODE, row, oidx, od2);
}

// Where the queries of a count come from: balls (centres, or the tree's own
// points, and one squared radius) or boxes (corners).
template <int D, class V = TreeView>
struct BallQueries {
  static constexpr bool kLarge = false;  // kWaveRowsLarge
  using View = V;
  using Real = typename View::Real;
  using Shape = BallShape<D, Real>;
  const Real* q;  // [nq][D], or nullptr: the tree's own points
  Real r2;
  bool apart = false;  // float64: only waves whose queries lie together
  __device__ __forceinline__ bool load(const View& t, int64_t nq, const int32_t* order,
                                       int64_t s, Shape& sh, int64_t& row) const {
    sh.r2 = r2;
    return load_query<D>(t, q, nq, order, s, sh.p, row);
  }
};

template <int D>
struct TorusBallQueries {
  static constexpr bool kLarge = false;  // kWaveRowsLarge
  using View = TreeView;
  using Shape = TorusBallShape<D>;
  const float* q;  // [nq][D], or nullptr: the tree's own points
  float r2;
  Torus<D> T;
  __device__ __forceinline__ bool load(const TreeView& t, int64_t nq, const int32_t* order,
                                       int64_t s, Shape& sh, int64_t& row) const {
    sh.r2 = r2;
    sh.T = T;
    return load_query<D>(t, q, nq, order, s, sh.p, row);
  }
};

template <int D, class Metric>
struct VarBallQueries {
  static constexpr bool kLarge = true;
  using View = TreeView;
  using Shape = VarBallShape<D, Metric>;
  const float* q;   // [rows][D]
  const float* r2;  // [rows]
  Metric m;
  __device__ __forceinline__ bool load(const TreeView& t, int64_t nq, const int32_t* order,
                                       int64_t s, Shape& sh, int64_t& row) const {
    sh.m = m;
    const bool ok = load_query<D>(t, q, nq, order, s, sh.p, row);
    sh.r2 = ok ? r2[row] : 0.0f;
    return ok;
  }
};

template <int D>
struct BoxQueries {
  static constexpr bool kLarge = false;  // kWaveRowsLarge
  using View = TreeView;
  using Shape = BoxShape<D>;
  const float* lo;  // [nq][D]
  const float* hi;
  __device__ __forceinline__ bool load(const TreeView&, int64_t nq, const int32_t* order,
                                       int64_t s, Shape& sh, int64_t& row) const {
    if (s >= nq) {
#pragma unroll
      for (int a = 0; a < D; ++a) {
        sh.lo[a] = 1.0f;  // an empty box
        sh.hi[a] = 0.0f;
      }
      return false;
    }
    row = order ? order[s] : s;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      sh.lo[a] = lo[row * D + a];
      sh.hi[a] = hi[row * D + a];
    }
    return true;
  }
};

template <int D, class Q>
__host__ __device__ constexpr size_t count_wave_bytes(int leaf) {
  return range_wave_bytes<D, typename Q::View, Q::Shape::kFloats>(leaf);
}
template <int D, class Q>
__device__ __forceinline__ typename Q::View::Real* count_slice(char* lds, int wave, int leaf) {
  return reinterpret_cast<typename Q::View::Real*>(lds + wave * count_wave_bytes<D, Q>(leaf));
}

// First pass of the counts: one 64-query group per wave from the root; writes
// each count (partial if the wave handed subtrees on), or with FILL the
// lists.
// (8 waves a SIMD: at 67 registers and 7 waves 2^22 GRF balls took 3.48 ms, now 3.30.)
template <int D, class Q, bool FILL>
__global__ __launch_bounds__(64 * kPWaves)
    __attribute__((amdgpu_waves_per_eu(sizeof(typename Q::View::Real) == 4 && D <= 4 ? 8 : 1))) void
    k_count_packet(typename Q::View t, Q src, int64_t nq,
                                                               const int32_t* __restrict__ order,
                                                               int32_t* __restrict__ count,
                                                               int leaf_cap, PacketSpill spill,
                                                               FillOut fo) {
  extern __shared__ __align__(16) char count_lds[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t s0 = (xcd_block<kXcdRunPacket>() * kPWaves + wave) * 64;
  if (s0 >= nq) return;
  if constexpr (std::is_same_v<typename Q::View, View64> && !FILL && D <= 4) {
    if (src.apart && !lie_together<D>(src.q, nq, s0)) {
      wave_done(spill);
      return;
    }
  }
  typename Q::Shape sh;
  int64_t row = 0;
  const bool active = src.load(t, nq, order, s0 + lane, sh, row);
  const int64_t c = packet_range_count<D, typename Q::Shape, FILL>(
      t, sh, active, count_slice<D, Q>(count_lds, wave, leaf_cap), leaf_cap, 0u, ~0ull,
      (uint32_t)(s0 / 64), spill, row, fo);
  if (!FILL && active) count[row] = (int32_t)c;
  wave_done(spill);
}

// A later pass: each wave takes tasks left by the previous pass (a fixed
// count, read at start, so every wave's loop ends) and adds its counts.  given: the budget is
// the caller's.
template <int D, class Q, bool FILL>
__global__ __launch_bounds__(64 * kPWaves) void k_count_tasks(
    typename Q::View t, Q src, int64_t nq, const int32_t* __restrict__ order,
    int32_t* __restrict__ count, int leaf_cap, const PacketTask* __restrict__ in,
    const uint32_t* __restrict__ in_count, uint32_t in_cap, PacketSpill spill, FillOut fo,
    bool given) {
  extern __shared__ __align__(16) char count_lds[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t n = min(*in_count, in_cap);
  auto* slice = count_slice<D, Q>(count_lds, wave, leaf_cap);
  if (!given && n >= kRangeManyTasks) spill.budget = kRangeManyBudget;
  for (uint32_t k = blockIdx.x * kPWaves + wave; k < n; k += gridDim.x * kPWaves) {
    const PacketTask task = in[k];
    if (task.node == kNoNode) continue;
    typename Q::Shape sh;
    int64_t row = 0;
    const bool active = src.load(t, nq, order, (int64_t)task.group * 64 + lane, sh, row);
    const uint64_t mask = ((uint64_t)task.hi << 32) | task.lo;
    const int64_t c = packet_range_count<D, typename Q::Shape, FILL>(
        t, sh, active, slice, leaf_cap, task.node, mask, task.group, spill, row, fo);
    if (!FILL && active && c != 0) atomicAdd(count + row, (int32_t)c);
  }
}

// One query shape per wave.
template <int D, class Q>
__global__ __launch_bounds__(64 * kPWaves) void k_count_wave(TreeView t, Q src, int64_t nq,
                                                             const int32_t* __restrict__ order,
                                                             int32_t* __restrict__ count,
                                                             int leaf_cap, int slice) {
  extern __shared__ uint32_t wave_lds[];
  const int wave = threadIdx.x >> 6;
  const int64_t s = (int64_t)blockIdx.x * kPWaves + wave;
  if (s >= nq) return;  // uniform over the wave
  typename Q::Shape sh;
  int64_t row = 0;
  src.load(t, nq, order, s, sh, row);
  const int64_t c = wave_ball<D, false>(t, sh, wave_lds + wave * slice, leaf_cap);
  if ((threadIdx.x & 63) == 0) count[row] = (int32_t)c;
}

__global__ void k_zero_tasks(uint32_t* c, int n) {
  if ((int)threadIdx.x < n) c[threadIdx.x] = 0u;
}

__global__ void k_zero_i32(int32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

template <int D>
__global__ __launch_bounds__(64 * kPWaves) void k_fof_packet(TreeView t, float l2,
                                                             int32_t* __restrict__ parent,
                                                             uint32_t* __restrict__ conn,
                                                             int leaf_cap) {
  extern __shared__ __align__(16) float lds[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t s0 = (xcd_block<kXcdRunFof>() * kPWaves + wave) * 64;
  if (s0 >= t.n) return;
  const int64_t pos = s0 + lane;
  const bool active = pos < t.n;
  float p[D];
  int32_t me = 0;
  if (active) {
    load_rec<D>(t.rec, pos, p, me);
  } else {
#pragma unroll
    for (int a = 0; a < D; ++a) p[a] = 0.0f;
  }
  packet_fof<D>(t, p, pos, me, active, l2, 0, parent, conn, fof_slice<D>(lds, wave, leaf_cap),
                leaf_cap);
}

template <int D>
kdt_status fof_packet_launch(const TreeView& v, int leaf, float l2, int32_t* parent, uint32_t* conn,
                             hipStream_t stream) {
  const unsigned grid = (unsigned)((v.n + 64 * kPWaves - 1) / (64 * kPWaves));
  k_fof_packet<D><<<grid, 64 * kPWaves, fof_lds_bytes<D>(leaf), stream>>>(v, l2, parent, conn,
                                                                            leaf);
  if (hipGetLastError() != hipSuccess) {
    kdt_set_error("kdt_fof: packet kernel launch failed");
    return KDT_EDEVICE;
  }
  return KDT_OK;
}

template <int D>
__global__ __launch_bounds__(64 * kPWaves) void k_fof_torus_packet(TreeView t, float l2,
                                                                   Torus<D> T,
                                                                   int32_t* __restrict__ parent,
                                                                   uint32_t* __restrict__ conn,
                                                                   int leaf_cap) {
  extern __shared__ __align__(16) float lds[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t s0 = (xcd_block<kXcdRunFof>() * kPWaves + wave) * 64;
  if (s0 >= t.n) return;
  const int64_t pos = s0 + lane;
  const bool active = pos < t.n;
  float p[D];
  int32_t me = 0;
  if (active) {
    load_rec<D>(t.rec, pos, p, me);
  } else {
#pragma unroll
    for (int a = 0; a < D; ++a) p[a] = 0.0f;
  }
  packet_fof<D>(t, p, pos, me, active, l2, 0, parent, conn, fof_slice<D>(lds, wave, leaf_cap),
                leaf_cap, TorusMetric<D>{T});
}

template <int D>
kdt_status torus_fof_packet_launch(const TreeView& v, int leaf, float l2, const Torus<D>& T,
                                   int32_t* parent, uint32_t* conn, hipStream_t stream) {
  const unsigned grid = (unsigned)((v.n + 64 * kPWaves - 1) / (64 * kPWaves));
  k_fof_torus_packet<D><<<grid, 64 * kPWaves, fof_lds_bytes<D>(leaf), stream>>>(
      v, l2, T, parent, conn, leaf);
  if (hipGetLastError() != hipSuccess) {
    kdt_set_error("kdt_fof_torus: packet kernel launch failed");
    return KDT_EDEVICE;
  }
  return KDT_OK;
}

template <int D>
kdt_status knn_packet_launch(const TreeView& v, int leaf, const float* d_q, int64_t nq, int k,
                             int32_t* d_idx, float* d_d2, int mode, const int32_t* order,
                             hipStream_t stream) {
  const unsigned grid = (unsigned)((nq + 64 * kPWaves - 1) / (64 * kPWaves));
  const size_t smem = sizeof(float) * knn_wave_floats<D>(leaf) * kPWaves;
#define KDT_LAUNCH(KC, M)                                                                      \
  k_knn_packet<D, KC, M><<<grid, 64 * kPWaves, smem, stream>>>(v, d_q, nq, k, order, d_idx, d_d2, \
                                                               leaf)
#define KDT_BY_MODE(KC)          \
  if (mode == 0) KDT_LAUNCH(KC, 0); \
  else if (mode == 1) KDT_LAUNCH(KC, 1); \
  else KDT_LAUNCH(KC, 2);
  if (k <= 8) {
    KDT_BY_MODE(8)
  } else if (k <= 16) {
    KDT_BY_MODE(16)
  } else if (k <= 32) {
    KDT_BY_MODE(32)
  } else {
    KDT_BY_MODE(64)
  }
#undef KDT_BY_MODE
#undef KDT_LAUNCH
  if (hipGetLastError() != hipSuccess) {
    kdt_set_error("kdt_knn: packet kernel launch failed");
    return KDT_EDEVICE;
  }
  return KDT_OK;
}

// The wave-shared counts (balls or boxes), with heavy traversals split over
// kRangePasses launches: the first kRangePasses - 1 hand off what exceeds their
// budget of node visits, the last finishes everything.
//
// With `fill` the same launches write the CSR lists instead (fill->cur zeroed
// here first); d_count is then not written.
template <int D, class Q>
static kdt_status count_packet_launch(const typename Q::View& v, int leaf, Q src, int64_t nq,
                                      const int32_t* order, int32_t* d_count,
                                      uint32_t split_budget, hipStream_t stream,
                                      const char* who, const FillOut* fill = nullptr) {
  constexpr bool kByWave = std::is_same_v<typename Q::View, TreeView> && D <= 8;
  [[maybe_unused]] const auto by_wave = [&]() -> kdt_status {
    if constexpr (kByWave) {
      int cap = 0;
      const TreeView w = coarse_view(v, leaf, kWaveLeafCap, &cap);
      const size_t slice = wave_ball_bytes(w.levels);
      k_count_wave<D, Q><<<(unsigned)((nq + kPWaves - 1) / kPWaves), 64 * kPWaves, slice * kPWaves,
                           stream>>>(w, src, nq, order, d_count, cap,
                                     (int)(slice / sizeof(uint32_t)));
      if (hipGetLastError() != hipSuccess) {
        kdt_set_error("%s: packet kernel launch failed", who);
        return KDT_EDEVICE;
      }
    }
    return KDT_OK;
  };
  // A wave per shape needs no scratch: so, up to kWaveRowsMost, also where there is none left
  // for the task lists, and in a graph, which would own them.
  const bool may = kByWave && !fill && split_budget == 0 &&
                   nq <= (Q::kLarge ? kWaveRowsLarge : kWaveRowsMost);
  if (may && (Q::kLarge || nq <= wave_rows(D, v.n) || stream_capturing(stream))) return by_wave();
  const unsigned grid = (unsigned)((nq + 64 * kPWaves - 1) / (64 * kPWaves));
  const size_t smem = count_wave_bytes<D, Q>(leaf) * kPWaves;
  PoolBuffers buf(stream);
  PacketTask* tasks = nullptr;
  uint32_t* counts = nullptr;
  const int64_t waves = (nq + 63) / 64;
  const uint32_t cap =
      (uint32_t)std::min<int64_t>(kRangeTaskCap, std::max<int64_t>(1, waves) * kRangeTasksPerWave);
  // counts[0 .. kRangePasses - 1): tasks per pass; then the first pass's
  // finished-wave counters
  if (!buf.get(&tasks, (size_t)cap * (kRangePasses - 1)) ||
      !buf.get(&counts, kRangePasses + kDoneShards)) {
    if (may) return by_wave();
    kdt_set_error("%s: device allocation failed for the task lists", who);
    return KDT_ENOMEM;
  }
  k_zero_tasks<<<1, 64, 0, stream>>>(counts, kRangePasses + kDoneShards);
  // a caller's budget applies to every wave of every launch
  constexpr int64_t most =
      std::is_same_v<typename Q::View, View64> ? kRangeMidWaves64 : kRangeMidWaves;
  const bool few = waves <= (fill ? kRangeFewWavesList : kRangeFewWaves);
  const bool mid = !fill && !few && waves <= most;
  const uint32_t first = split_budget ? split_budget
                         : few        ? kRangeBudgetFew
                         : mid        ? kRangeBudgetMid
                                      : kRangeBudgetFirst;
  const uint32_t later = split_budget ? split_budget
                         : few || mid ? kRangeBudgetFew
                                      : kRangeBudget;
  const uint32_t tail_from = split_budget                ? 0u
                             : waves > kRangeTailWaves ? (uint32_t)(waves - kRangeTailWaves)
                                                       : 0u;
  const FillOut fo = fill ? *fill : FillOut{nullptr, nullptr, nullptr};
  if (fill) k_zero_i32<<<(unsigned)((nq + 255) / 256), 256, 0, stream>>>(fill->cur, nq);
  const PacketSpill sp0{tasks, counts, cap, first, counts + kRangePasses, tail_from};
  if (fill)
    k_count_packet<D, Q, true><<<grid, 64 * kPWaves, smem, stream>>>(v, src, nq, order, d_count,
                                                                     leaf, sp0, fo);
  else
    k_count_packet<D, Q, false><<<grid, 64 * kPWaves, smem, stream>>>(v, src, nq, order, d_count,
                                                                      leaf, sp0, fo);
  for (int pass = 1; pass < kRangePasses; ++pass) {
    const bool last = pass == kRangePasses - 1;
    const PacketSpill out = last ? PacketSpill{nullptr, nullptr, 0u, 0u, nullptr, 0u}
                                : PacketSpill{tasks + (size_t)pass * cap, counts + pass, cap, later, nullptr, 0u};
    const PacketTask* in = tasks + (size_t)(pass - 1) * cap;
    if (fill)
      k_count_tasks<D, Q, true><<<kRangeTaskBlocks, 64 * kPWaves, smem, stream>>>(
          v, src, nq, order, d_count, leaf, in, counts + pass - 1, cap, out, fo,
          split_budget != 0);
    else
      k_count_tasks<D, Q, false><<<kRangeTaskBlocks, 64 * kPWaves, smem, stream>>>(
          v, src, nq, order, d_count, leaf, in, counts + pass - 1, cap, out, fo,
          split_budget != 0);
  }
  if (hipGetLastError() != hipSuccess) {
    kdt_set_error("%s: packet kernel launch failed", who);
    return KDT_EDEVICE;
  }
  return KDT_OK;
}

template <int D>
kdt_status range_packet_launch(const TreeView& v, int leaf, const float* d_q, int64_t nq, float r2,
                               const int32_t* order, int32_t* d_count, uint32_t split_budget,
                               hipStream_t stream, const FillOut* fill) {
  return count_packet_launch<D>(v, leaf, BallQueries<D>{d_q, r2}, nq, order, d_count,
                                split_budget, stream, "kdt_range", fill);
}

template <int D>
kdt_status range64_packet_launch(const View64& v, int leaf, const double* d_q, int64_t nq,
                                 double r2, const int32_t* order, int32_t* d_count,
                                 hipStream_t stream, const FillOut* fill, bool apart) {
  return count_packet_launch<D>(v, leaf, BallQueries<D, View64>{d_q, r2, apart}, nq, order,
                                d_count, 0u, stream, "kdt_range_f64", fill);
}

template <int D>
kdt_status box_packet_launch(const TreeView& v, int leaf, const float* d_lo, const float* d_hi,
                             int64_t nq, const int32_t* order, int32_t* d_count,
                             uint32_t split_budget, hipStream_t stream, const FillOut* fill) {
  return count_packet_launch<D>(v, leaf, BoxQueries<D>{d_lo, d_hi}, nq, order, d_count,
                                split_budget, stream, "kdt_box", fill);
}

template <int D>
kdt_status torus_range_packet_launch(const TreeView& v, int leaf, const float* d_q, int64_t nq,
                                     float r2, const Torus<D>& T, const int32_t* order,
                                     int32_t* d_count, uint32_t split_budget,
                                     hipStream_t stream, const FillOut* fill) {
  return count_packet_launch<D>(v, leaf, TorusBallQueries<D>{d_q, r2, T}, nq, order, d_count,
                                split_budget, stream, "kdt_range", fill);
}

template <int D, class Metric>
kdt_status var_ball_count_launch(const TreeView& v, int leaf, const float* d_q, const float* d_r2,
                                 int64_t nq, const int32_t* order, const Metric& m,
                                 int32_t* d_count, hipStream_t stream) {
  return count_packet_launch<D>(v, leaf, VarBallQueries<D, Metric>{d_q, d_r2, m}, nq, order,
                                d_count, 0u, stream, "kdt_knn");
}

size_t range64_packet_lds(int d, int leaf) {
  return kPWaves * (d == 2   ? range_wave_bytes<2, View64, 2>(leaf)
                    : d == 3 ? range_wave_bytes<3, View64, 3>(leaf)
                    : d == 4 ? range_wave_bytes<4, View64, 4>(leaf)
                    : d == 8 ? range_wave_bytes<8, View64, 8>(leaf)
                             : range_wave_bytes<16, View64, 16>(leaf));
}

#define KDT_INST(D)                                                                                \
  template kdt_status knn_packet_launch<D>(const TreeView&, int, const float*, int64_t, int,       \
                                           int32_t*, float*, int, const int32_t*, hipStream_t);    \
  template kdt_status range_packet_launch<D>(const TreeView&, int, const float*, int64_t, float,   \
                                             const int32_t*, int32_t*, uint32_t, hipStream_t,    \
                                             const FillOut*);                                    \
  template kdt_status range64_packet_launch<D>(const View64&, int, const double*, int64_t, double, \
                                               const int32_t*, int32_t*, hipStream_t,            \
                                               const FillOut*, bool);                            \
  template kdt_status box_packet_launch<D>(const TreeView&, int, const float*, const float*,       \
                                           int64_t, const int32_t*, int32_t*, uint32_t,          \
                                           hipStream_t, const FillOut*);                         \
  template kdt_status fof_packet_launch<D>(const TreeView&, int, float, int32_t*, uint32_t*,       \
                                           hipStream_t);                                         \
  template kdt_status torus_range_packet_launch<D>(const TreeView&, int, const float*, int64_t,    \
                                                   float, const Torus<D>&, const int32_t*,       \
                                                   int32_t*, uint32_t, hipStream_t,              \
                                                   const FillOut*);                              \
  template kdt_status torus_fof_packet_launch<D>(const TreeView&, int, float, const Torus<D>&,     \
                                                 int32_t*, uint32_t*, hipStream_t);              \
  template kdt_status var_ball_count_launch<D, OpenMetric<D>>(                                     \
      const TreeView&, int, const float*, const float*, int64_t, const int32_t*,                  \
      const OpenMetric<D>&, int32_t*, hipStream_t);                                               \
  template kdt_status var_ball_count_launch<D, TorusMetric<D>>(                                    \
      const TreeView&, int, const float*, const float*, int64_t, const int32_t*,                  \
      const TorusMetric<D>&, int32_t*, hipStream_t);
KDT_INST(2)
KDT_INST(3)
KDT_INST(4)
KDT_INST(8)
KDT_INST(16)
#undef KDT_INST

}  // namespace kdt
