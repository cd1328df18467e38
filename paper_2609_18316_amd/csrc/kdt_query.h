// kdt_query.h -- device-side tree view and traversal helpers shared by the
// query, grouping and batched kernels.
#pragma once

#include <type_traits>

#include "kdt_internal.h"

namespace kdt {

constexpr int kMaxDepth = 32;  // levels <= 30 for n < 2^31 and leaf_size >= 2

struct TreeView {
  using Real = float;
  const float* rec;  // [n][rec_stride(D)] tree-ordered records
  const float* box;  // [n_nodes][2 * pad4(D)]
  int64_t n;
  int32_t levels;    // depth of the deepest leaf
  const int4* nodes = nullptr;  // stored node records (sliding-midpoint trees), else NULL
  unsigned long long* visits = nullptr;  // work counters of the instrumented build, else NULL
};

// A tree over float64 coordinates (kdt_build_f64).
struct View64 {
  using Real = double;
  const double* rec;    // [n][D] tree-ordered coordinates
  const double* box;    // [n_nodes][2][D] lo then hi
  const int32_t* perm;  // [n] input index of each tree position
  int64_t n;
  int32_t levels;
  const int4* nodes;    // stored nodes (sliding-midpoint trees) or NULL
  unsigned long long* visits = nullptr;
};

// The wave-shared counts (and their list fill) over a median tree treat the
// nodes of one level as their leaves: the coarsest level whose nodes hold at
// most kCountLeaf points, never below the tree's own leaves.  Node ranges
// and tight boxes exist at every level, so the counts are the same; only
// the cost differs -- ball counts at r = 0.01 on 2^24 clustered points took
// 3.6 ms with 32-point leaves and 4.8 ms with 16-point ones.  Returns that
// view and, in *cap, its largest node (the LDS slices' leaf capacity).
constexpr int kCountLeaf = 32;
// The view at the coarsest level whose nodes hold at most `most` points.
template <class View>
inline View coarse_view(View v, int leaf, int most, int* cap) {
  int l = v.levels;
  while (l > 0 && ((v.n + (int64_t(1) << (l - 1)) - 1) >> (l - 1)) <= most) --l;
  const int64_t big = (v.n + (int64_t(1) << l) - 1) >> l;
  *cap = big > leaf ? (int)big : leaf;
  v.levels = l;
  return v;
}
template <class View>
inline View count_view(View v, int leaf, int* cap) {
  return coarse_view(v, leaf, kCountLeaf, cap);
}

// Where the wave-shared counts write CSR lists in fill mode: the indices of
// row r go to out[off[r] ..], a slot at a time reserved with an atomic on the
// row's cursor cur[r] (zero before the first pass), so the subtrees a wave
// hands on to later passes append the same way.  The order within a row
// depends on the schedule; callers sort each row afterwards.
struct FillOut {
  int32_t* out;
  const int64_t* off;
  int32_t* cur;
};

// Work counters of the instrumented build (compiled with KDT_COUNT_VISITS):
// how many node boxes and point records the traversals read, for the
// algorithmic bytes of the roofline.  Slots: kVisitNodes / kVisitPoints /
// kVisitInsert for one traversal per lane (nodes visited, i.e. node boxes
// tested -- the root and both children of every expanded node --, leaf
// records scanned, candidates among them), kVisitReload
// for a box read again when its node leaves the stack (sliding-midpoint
// trees, whose stack keeps node ids only), kVisitWaveNodes / kVisitWavePoints for the wave-shared
// traversals (one box read and one leaf staged into LDS count once per
// wave).  Each slot has kVisitShards
// counters (workgroup b adds to shard b % kVisitShards).  In the product
// build the macros compile to nothing.
enum : int { kVisitNodes = 0, kVisitPoints = 1, kVisitInsert = 2, kVisitWaveNodes = 3,
             kVisitWavePoints = 4, kVisitReload = 5, kVisitSlots = 8 };
constexpr int kVisitShards = 64;
#ifdef KDT_COUNT_VISITS
template <class View>
__device__ __forceinline__ void count_visit(const View& t, int slot, uint32_t n) {
  if (t.visits)
    atomicAdd(t.visits + slot * kVisitShards + (blockIdx.x % kVisitShards),
              (unsigned long long)n);
}
#define KDT_LANE_VISIT(t, slot, n) count_visit((t), (slot), (uint32_t)(n))
#define KDT_WAVE_VISIT(t, slot, n)                                  \
  do {                                                              \
    if (lane_id() == 0) count_visit((t), (slot), (uint32_t)(n));    \
  } while (0)
#else
#define KDT_LANE_VISIT(t, slot, n) ((void)0)
#define KDT_WAVE_VISIT(t, slot, n) ((void)0)
#endif

// Node layout of a tree, as the traversals see it.  A median tree is
// implicit: node (l, j) sits at 2^l - 1 + j, its children at 2v + 1 and
// 2v + 2, and it owns points [floor(j n / 2^l), floor((j + 1) n / 2^l)), so
// every leaf holds floor(n / 2^L) or one more.  A sliding-midpoint tree
// (Sec. 2.1, data-dependent depth) stores per node (left child or -1 for a
// leaf, first point, end point, level); its right child follows the left.
struct MedianShape {
  int64_t n;
  int levels;
  uint32_t first_leaf;
  __device__ __forceinline__ explicit MedianShape(const TreeView& t)
      : n(t.n), levels(t.levels), first_leaf((1u << t.levels) - 1u) {}
  __device__ __forceinline__ bool is_leaf(uint32_t v) const { return v >= first_leaf; }
  __device__ __forceinline__ uint32_t left(uint32_t v) const { return 2 * v + 1; }
  __device__ __forceinline__ void range(uint32_t v, int64_t& b, int64_t& e) const {
    const int lev = 31 - __clz(v + 1);
    const int64_t j = (int64_t)v - ((int64_t(1) << lev) - 1);
    b = (j * n) >> lev;
    e = ((j + 1) * n) >> lev;
  }
};

struct StoredShape {
  const int4* node;
  __device__ __forceinline__ explicit StoredShape(const TreeView& t) : node(t.nodes) {}
  __device__ __forceinline__ bool is_leaf(uint32_t v) const { return node[v].x < 0; }
  __device__ __forceinline__ uint32_t left(uint32_t v) const { return (uint32_t)node[v].x; }
  __device__ __forceinline__ void range(uint32_t v, int64_t& b, int64_t& e) const {
    const int4 r = node[v];
    b = r.y;
    e = r.z;
  }
};

template <int D>
struct Pt {
  float v[D];
};

template <int D>
__device__ __forceinline__ void load_box(const float* __restrict__ box, uint32_t node, float lo[D],
                                         float hi[D]) {
  constexpr int P = pad4(D);
  const float4* b = reinterpret_cast<const float4*>(box + (size_t)node * 2 * P);
#pragma unroll
  for (int q = 0; q < P / 4; ++q) {
    float4 l = b[q], h = b[P / 4 + q];
    if (4 * q + 0 < D) lo[4 * q + 0] = l.x, hi[4 * q + 0] = h.x;
    if (4 * q + 1 < D) lo[4 * q + 1] = l.y, hi[4 * q + 1] = h.y;
    if (4 * q + 2 < D) lo[4 * q + 2] = l.z, hi[4 * q + 2] = h.z;
    if (4 * q + 3 < D) lo[4 * q + 3] = l.w, hi[4 * q + 3] = h.w;
  }
}

// Smallest squared distance from p to the box: the same float32 operations,
// in the same axis order, as the point distance, so it never exceeds the
// rounded distance of any point inside the box.
// The axis gap max(lo - p, p - hi, 0) is exactly lo - p below the box, p - hi
// above it and 0 inside (a max does not round), taken without branches.
template <int D>
__device__ __forceinline__ float box_mindist(const float lo[D], const float hi[D], const float p[D]) {
  float s = 0.0f;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const float t = fmaxf(fmaxf(lo[a] - p[a], p[a] - hi[a]), 0.0f);
    float t2 = t * t;
    s = s + t2;
  }
  return s;
}
// The same in float64 (float64 trees), NaN treated alike (a gap of 0).
template <int D>
__device__ __forceinline__ double box_mindist(const double lo[D], const double hi[D],
                                              const double p[D]) {
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const double t = fmax(fmax(lo[a] - p[a], p[a] - hi[a]), 0.0);
    s += t * t;
  }
  return s;
}

// Largest squared distance from p to the box (never below any point's).
template <int D>
__device__ __forceinline__ float box_maxdist(const float lo[D], const float hi[D], const float p[D]) {
  float s = 0.0f;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    float t1 = fabsf(p[a] - lo[a]);
    float t2 = fabsf(p[a] - hi[a]);
    float t = t1 > t2 ? t1 : t2;
    float tt = t * t;
    s = s + tt;
  }
  return s;
}

template <int D>
__device__ __forceinline__ double box_maxdist(const double lo[D], const double hi[D],
                                              const double p[D]) {
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const double t1 = fabs(p[a] - lo[a]), t2 = fabs(p[a] - hi[a]);
    const double t = t1 > t2 ? t1 : t2;
    s += t * t;
  }
  return s;
}

// Squared Euclidean distance (Eq. 1, p = 2): float32 (float64 over float64
// trees), axes left to right, every operation rounded on its own (the library
// is built without FMA contraction).
template <int D>
__device__ __forceinline__ double sq_dist(const double* __restrict__ x, const double p[D]) {
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const double t = x[a] - p[a];
    s += t * t;
  }
  return s;
}
template <int D>
__device__ __forceinline__ float sq_dist(const float* __restrict__ x, const float p[D]) {
  float s = 0.0f;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    float t = x[a] - p[a];
    float t2 = t * t;
    s = s + t2;
  }
  return s;
}

template <int D>
__device__ __forceinline__ void load_rec(const float* __restrict__ rec, int64_t i, float x[D],
                                         int32_t& idx) {
  constexpr int S = rec_stride(D);
  const float4* r = reinterpret_cast<const float4*>(rec + i * S);
#pragma unroll
  for (int q = 0; q < S / 4; ++q) {
    float4 v = r[q];
    float w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      int a = 4 * q + c;
      if (a < D) x[a] = w[c];
      if (a == D) idx = __float_as_int(w[c]);
    }
  }
}

// Reads of wave-uniform addresses in data that no kernel writes while it
// runs (node boxes): through the constant address space, so the compiler
// issues scalar loads, one per wave.
typedef const __attribute__((address_space(4))) float cfloat;
__device__ __forceinline__ const cfloat* as_uniform(const float* p) {
  return (const cfloat*)p;
}

// Box of a node whose index is wave-uniform.
template <int D>
__device__ __forceinline__ void load_box_uniform(const float* box, uint32_t node, float lo[D],
                                                 float hi[D]) {
  constexpr int P = pad4(D);
  const cfloat* b = as_uniform(box) + (size_t)node * 2 * P;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    lo[a] = b[a];
    hi[a] = b[P + a];
  }
}

typedef const __attribute__((address_space(4))) double cdouble;
template <int D>
__device__ __forceinline__ void load_node_uniform(const TreeView& t, uint32_t node, float lo[D],
                                                  float hi[D]) {
  load_box_uniform<D>(t.box, node, lo, hi);
}
template <int D>
__device__ __forceinline__ void load_node_uniform(const View64& t, uint32_t node, double lo[D],
                                                  double hi[D]) {
  const cdouble* b = (const cdouble*)t.box + (size_t)node * 2 * D;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    lo[a] = b[a];
    hi[a] = b[D + a];
  }
}
// The input index of the point at tree position i.
template <int D>
__device__ __forceinline__ int32_t input_index(const TreeView& t, int64_t i) {
  return __float_as_int(t.rec[i * rec_stride(D) + D]);
}
template <int D>
__device__ __forceinline__ int32_t input_index(const View64& t, int64_t i) {
  return t.perm[i];
}
// Elements of View::Real per point record.
template <int D, class View>
__host__ __device__ constexpr int point_stride() {
  return std::is_same_v<View, View64> ? D : rec_stride(D);
}

// Leaf points a wave-uniform scan keeps in flight (a loop unroll factor).
template <int D>
constexpr int uniform_batch() {
  return D <= 4 ? 8 : (32 / D > 0 ? 32 / D : 1);
}

// Key of an empty candidate slot: squared distance +inf, index 0xFFFFFFFF, so
// it sorts after every real point (indices are below 2^31).
constexpr uint64_t kEmptyKey = 0x7F800000FFFFFFFFull;

// Sorted register list of the KC smallest 64-bit keys (d2 bits << 32 | index).
// Only the last k slots are live: the first KC - k hold 0 and never move.
//
// The keys are stored as float64 bit patterns: for d2 >= 0 (never NaN) the
// key's sign bit is 0 and its exponent field can never be all ones, so the
// float64 order of the patterns is exactly the unsigned order of the keys
// (keys below 2^52 are subnormal doubles, which the float64 min/max keep
// exact because float64 subnormals are not flushed).  That turns each
// compare-and-carry step into one v_min_f64 and one v_max_f64.
constexpr int kListBatch = 16;  // keys that a merge takes

template <int KC>
struct TopK {
  double a[KC];
  using Key = double;
  __device__ __forceinline__ void init(int k) {
#pragma unroll
    for (int i = 0; i < KC; ++i) a[i] = (i < KC - k) ? 0.0 : __longlong_as_double((long long)kEmptyKey);
  }
  __device__ __forceinline__ uint64_t key(int i) const {
    return (uint64_t)__double_as_longlong(a[i]);
  }
  __device__ __forceinline__ uint64_t worst() const { return key(KC - 1); }
  __device__ __forceinline__ float worst_d2() const {
    return __uint_as_float((uint32_t)(worst() >> 32));
  }
  // Inserts x if it is below worst(), otherwise leaves the list unchanged
  // (no branch, so it can run on every lane of a wave).  One bottom-up pass
  // of compare-and-carry: each slot keeps the smaller of itself and the carry
  // and hands the larger upwards; the largest key falls off the top.
  //
  // Every key read as a float64 is finite and non-negative (the high word is
  // a non-negative float32, so the float64 exponent stays below 0x7FF), so
  // the hardware min/max order keys exactly.  They are issued directly: the
  // library fmin/fmax would first canonicalise both operands of every slot
  // (IEEE mode), half as many instructions again.
  // Returns the key that fell off.
  __device__ __forceinline__ uint64_t insert(uint64_t x) {
    double carry = __longlong_as_double((long long)x);
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      double up;
      asm("v_max_f64 %1, %0, %2\n\tv_min_f64 %0, %0, %2"
          : "+v"(a[i]), "=&v"(up)
          : "v"(carry));
      carry = up;
    }
    return (uint64_t)__double_as_longlong(carry);
  }
  __device__ __forceinline__ void offer(float d2, int32_t id);
  // The KC smallest keys of the list and of a batch of keys (in any order;
  // kEmptyKey where there is none): the batch is sorted, its smallest keys
  // are laid in reverse against the list's largest -- the smaller of each
  // pair stays -- and the bitonic list that leaves is sorted.
  __device__ __forceinline__ void merge(double (&c)[kListBatch]);
};

// a <- the smaller, b <- the larger of two keys (see TopK::insert), both in
// the registers they came in: with two fresh results per step the register
// allocator keeps a second copy of the list (k = 32: 165 instead of 130
// VGPRs), which costs a wave per SIMD and more time than the move.
__device__ __forceinline__ void order_in_place(double& a, double& b) {
  double lo;
  asm("v_min_f64 %0, %1, %2\n\tv_max_f64 %2, %1, %2\n\tv_mov_b64 %1, %0"
      : "=&v"(lo), "+v"(a), "+v"(b));
}
__device__ __forceinline__ void order_in_place(uint32_t& a, uint32_t& b) {
  uint32_t lo;
  asm("v_min_u32 %0, %1, %2\n\tv_max_u32 %2, %1, %2\n\tv_mov_b32 %1, %0"
      : "=&v"(lo), "+v"(a), "+v"(b));
}

// Batcher's odd-even merge sort (K. E. Batcher, "Sorting networks and their
// applications", AFIPS SJCC 1968).
template <class T, int N>
__device__ __forceinline__ void sort_network(T (&c)[N]) {
#pragma unroll
  for (int p = 1; p < N; p *= 2)
#pragma unroll
    for (int k = p; k >= 1; k /= 2)
#pragma unroll
      for (int j = k % p; j + k < N; j += 2 * k)
#pragma unroll
        for (int i = 0; i < k; ++i)
          if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p))
            order_in_place(c[i + j], c[i + j + k]);
}

// Sorts a bitonic sequence (Batcher's half-cleaners).
template <class T, int N>
__device__ __forceinline__ void sort_bitonic(T (&a)[N]) {
#pragma unroll
  for (int k = N / 2; k >= 1; k /= 2)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if ((i & k) == 0) order_in_place(a[i], a[i + k]);
}

template <int KC>
__device__ __forceinline__ void TopK<KC>::merge(double (&c)[kListBatch]) {
  sort_network(c);
  constexpr int M = KC < kListBatch ? KC : kListBatch;
#pragma unroll
  for (int i = 0; i < M; ++i)
    asm("v_min_f64 %0, %0, %1" : "+v"(a[KC - M + i]) : "v"(c[M - 1 - i]));
  sort_bitonic(a);
}

__device__ __forceinline__ uint64_t make_key(float d2, int32_t idx) {
  return ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)idx;
}

template <int KC>
__device__ __forceinline__ void TopK<KC>::offer(float d2, int32_t id) {
  const uint64_t key = make_key(d2, id);
  if (key < worst()) insert(key);
}

// Key of an empty slot of TopKTie: it sorts after every point and is a finite float64.
constexpr uint64_t kEmptyKeyTie = 0x7FEFFFFFFFFFFFFFull;

// TopK for float64 trees: its keys are float64 squared distances whose lowest bits hold the
// point's tree position (Space64).  It also knows the smallest key that it has turned away: if
// all but the position is the k-th key's, which of the equals belongs into the list is
// open to the caller.  Distances are compared by their upper words.
template <int KC>
struct TopKTie : TopK<KC> {
  double lost;
  __device__ __forceinline__ void init(int k) {
    lost = __longlong_as_double((long long)kEmptyKeyTie);
#pragma unroll
    for (int i = 0; i < KC; ++i) this->a[i] = (i < KC - k) ? 0.0 : lost;
  }
  __device__ __forceinline__ uint32_t worst_d2() const { return (uint32_t)(this->worst() >> 32); }
  __device__ __forceinline__ void turn_away(double key) {
    asm("v_min_f64 %0, %0, %1" : "+v"(lost) : "v"(key));
  }
  __device__ __forceinline__ void offer(uint32_t d2, int32_t id) {
    uint64_t key = ((uint64_t)d2 << 32) | (uint32_t)id;
    if (key < this->worst()) key = this->insert(key);
    turn_away(__longlong_as_double((long long)key));
  }
  __device__ __forceinline__ void merge(double (&c)[kListBatch]) {
    static_assert(KC >= kListBatch, "the whole batch fits the list");
    sort_network(c);
#pragma unroll
    for (int i = 0; i < kListBatch; ++i) {
      double& mine = this->a[KC - 1 - i];
      order_in_place(mine, c[i]);
      turn_away(c[i]);
    }
    sort_bitonic(this->a);
  }
};

// The k smallest squared distances alone, for queries that want only the
// k-th distance: its value does not depend on how equal distances are
// ordered, so no index is kept and the list takes half the registers of
// TopK.  Entries are the bit patterns of non-negative float32 values (or
// +inf), which order like the values, so integer min/max keep the list
// sorted without any float rounding or denormal handling.
template <int KC>
struct TopD {
  uint32_t a[KC];
  using Key = uint32_t;
  __device__ __forceinline__ void init(int k) {
#pragma unroll
    for (int i = 0; i < KC; ++i) a[i] = (i < KC - k) ? 0u : 0x7F800000u;
  }
  __device__ __forceinline__ float worst_d2() const { return __uint_as_float(a[KC - 1]); }
  __device__ __forceinline__ void offer(float d2, int32_t) {
    const uint32_t x = __float_as_uint(d2);
    if (x < a[KC - 1]) {
      // every slot becomes the middle one of (slot below, x, itself), from
      // the top down so that the slot below is still the old one: one
      // instruction per slot where compare-and-carry takes two
#pragma unroll
      for (int i = KC - 1; i > 0; --i)
        asm("v_med3_u32 %0, %1, %2, %0" : "+v"(a[i]) : "v"(a[i - 1]), "v"(x));
      a[0] = min(a[0], x);
    }
  }
  // As TopK::merge.
  __device__ __forceinline__ void merge(uint32_t (&c)[kListBatch]) {
    sort_network(c);
    constexpr int M = KC < kListBatch ? KC : kListBatch;
#pragma unroll
    for (int i = 0; i < M; ++i) a[KC - M + i] = min(a[KC - M + i], c[M - 1 - i]);
    sort_bitonic(a);
  }
};

// The entry of a leaf point in a merge's batch (empty: no such point).
template <int KC>
__device__ __forceinline__ double batch_key(const TopK<KC>&, bool there, float d2, int32_t id) {
  return __longlong_as_double((long long)(there ? make_key(d2, id) : kEmptyKey));
}
template <int KC>
__device__ __forceinline__ double batch_key(const TopKTie<KC>&, bool there, uint32_t d2,
                                            int32_t id) {
  return __longlong_as_double(
      (long long)(there ? ((uint64_t)d2 << 32) | (uint32_t)id : kEmptyKeyTie));
}
template <int KC>
__device__ __forceinline__ uint32_t batch_key(const TopD<KC>&, bool there, float d2, int32_t) {
  return there ? __float_as_uint(d2) : 0x7F800000u;
}

// Open-space metric of the traversals: the point distance (Eq. 1, p = 2) and
// the lower and upper bounds over a node box.  Other metrics (the D-torus of
// periodic boundaries) supply the same three.
template <int D>
struct OpenMetric {
  __device__ __forceinline__ float dist(const float x[D], const float p[D]) const {
    return sq_dist<D>(x, p);
  }
  __device__ __forceinline__ float mindist(const float lo[D], const float hi[D],
                                           const float p[D]) const {
    return box_mindist<D>(lo, hi, p);
  }
  __device__ __forceinline__ float maxdist(const float lo[D], const float hi[D],
                                           const float p[D]) const {
    return box_maxdist<D>(lo, hi, p);
  }
};

// What a per-lane kNN traversal measures: the float32 points of a tree
// under a metric.
template <int D, class Metric>
struct Space32 {
  using Coord = float;
  using Dist = float;
  const TreeView& t;
  const Metric& m;
  static __device__ __forceinline__ uint32_t bits(float d) { return __float_as_uint(d); }
  static __device__ __forceinline__ float from_bits(uint32_t d) { return __uint_as_float(d); }
  // Box distances of the nodes c and c + 1.
  __device__ __forceinline__ void pair(uint32_t c, const float p[D], float& d0, float& d1) const {
    float lo[D], hi[D];
    load_box<D>(t.box, c, lo, hi);
    d0 = m.mindist(lo, hi, p);
    load_box<D>(t.box, c + 1, lo, hi);
    d1 = m.mindist(lo, hi, p);
  }
  // The records from tree position `base` on, and the squared distance and
  // identity (input index) of the i-th.
  __device__ __forceinline__ const float* run(int32_t base) const {
    return t.rec + (int64_t)base * rec_stride(D);
  }
  __device__ __forceinline__ float dist(const float* r, int32_t, int i, const float p[D],
                                        int32_t& id) const {
    float x[D];
    load_rec<D>(r, i, x, id);
    return m.dist(x, p);
  }
};

// The points of a float64 tree by keys of 64 bits: the float64 squared distance, its lowest
// bits (`low`, as many as a position has) replaced by the tree position.  That keeps
// float64's whole range, so coordinates of any scale are told apart, and 31 bits of the
// mantissa at 2^21 points.  Cutting bits off is monotone; nodes and candidates are
// tested by the upper words alone, which lets a few more through.  (An infinite distance is
// above every key's, and a NaN too.)
template <int D>
struct Space64 {
  using Coord = double;
  using Dist = uint32_t;
  const View64& t;
  uint32_t low;
  static __device__ __forceinline__ uint32_t low_bits(int64_t n) {
    return n > 1 ? 0xFFFFFFFFu >> __clz((uint32_t)(n - 1)) : 0u;
  }
  static __device__ __forceinline__ uint32_t bits(uint32_t d) { return d; }
  static __device__ __forceinline__ uint32_t from_bits(uint32_t d) { return d; }
  static __device__ __forceinline__ uint32_t upper(double d) {
    return (uint32_t)__double2hiint(d);
  }
  __device__ __forceinline__ void pair(uint32_t c, const double p[D], uint32_t& d0,
                                       uint32_t& d1) const {
    const double* b = t.box + (size_t)c * 2 * D;
    double x[4 * D];
#pragma unroll
    for (int a = 0; a < 4 * D; ++a) x[a] = b[a];
    d0 = upper(box_mindist<D>(x, x + D, p));
    d1 = upper(box_mindist<D>(x + 2 * D, x + 3 * D, p));
  }
  __device__ __forceinline__ const double* run(int32_t base) const {
    return t.rec + (int64_t)base * D;
  }
  // id: the key's lower word
  __device__ __forceinline__ uint32_t dist(const double* r, int32_t base, int i,
                                           const double p[D], int32_t& id) const {
    const double d2 = sq_dist<D>(r + i * D, p);
    id = (int32_t)(((uint32_t)__double2loint(d2) & ~low) | (uint32_t)(base + i));
    return upper(d2);
  }
};

// Which lists take a leaf's points in sorted batches (ListMerge<...>::kOn): those of
// 17 to 32 entries below five dimensions.  Inserting one key costs 64
// (TopK) or 32 (TopD) instructions at k = 32 and runs for the wave when any
// lane inserts -- about ten times per leaf of 16 points --, a merge of 16 keys
// 430, whatever the number of candidates; a merge also needs no second pass
// over the points.  Measured against insertion alone: 5.10 and 5.88 ms for 2^22
// external queries on 2^24 clustered points (k = 32), 2.66 and 3.12 ms for the
// smoothing lengths of 2^22 points.  At 16 entries the merge loses its 16
// registers' worth of waves for nothing (1.86 against 1.78 ms, 2^21 points), at
// 64 it does not fit the registers, and in 8 dimensions the batch's
// coordinates do not (8.9 against 7.7 ms, 200003 points, k = 16).
// kMin: the wave merges when some lane has more candidates than this, else
// each lane inserts its own (equal within 1 % from 1 to 5).
template <class List, int D>
struct ListMerge;
template <int KC, int D>
struct ListMerge<TopK<KC>, D> {
  static constexpr bool kOn = KC == 32 && D <= 4;
  static constexpr int kMin = 3;
};
template <int KC, int D>
struct ListMerge<TopKTie<KC>, D> : ListMerge<TopK<KC>, D> {};
template <int KC, int D>
struct ListMerge<TopD<KC>, D> {
  static constexpr bool kOn = KC == 32 && D <= 4;
  static constexpr int kMin = 5;
};
// Waves per SIMD that a per-lane kNN kernel is compiled for: its list with a
// batch takes 128 VGPRs, which the compiler reaches only when asked to.
template <int D, int KC, bool KTH, class Shape = MedianShape, bool kMerge = true>
constexpr int lane_waves() {
  return !KTH && kMerge && std::is_same_v<Shape, MedianShape> && ListMerge<TopK<KC>, D>::kOn ? 4
                                                                                             : 1;
}
// Where a list that can merge does (most: points of the largest leaf): everywhere but in
// 4 dimensions on large trees whose leaves take more than one batch -- few of their points
// are candidates.  All points as queries, us merging / inserting / inserting before the vote:
// 400000 points, leaves of 32, k = 24 1058 / 823 / 1002, k = 32 1196 / 945 / 1135, leaves
// of 16 1039 / 992 / 1143; 2 * 10^6 points, leaves of 64, k = 32 5839 / 4251 / 6682; below the
// line the two are closer and cross: 100000 points, leaves of 32 462 / 420 / 496, of 16 428 / 474
// / 498 (queries of their own), 4000 points 257 / 307 / 341.
template <int D>
inline bool lane_merges(int most, int64_t n) {
  return D != 4 || most <= kListBatch || n < (1 << 18);
}
// The list length of k for kNN over n points with one traversal per lane: k
// rounded up, except that a merge reads kListBatch consecutive points, so
// smaller trees take a list that inserts.
inline int lane_list(int k, int64_t n) {
  return k <= 8 ? 8 : k <= 16 ? 16 : k <= 32 && n >= kListBatch ? 32 : 64;
}

// Whether kNN takes one traversal per lane by default, whatever the compiled-in tuning
// table says of the shape (an entry set at run time decides by itself): in up to 4 dimensions, where the largest leaf (`most`
// points) is small or the list long.  All points as queries, us per lane / per
// wave: 65536 uniform points, leaves of 32, k = 8 111 / 130, of 64 139 / 116,
// k = 32 186 / 272 and 220 / 247; 1000 points, leaves of 32, 66 / 90
// (k = 8); 2^20 clustered points, leaves of 32, k = 16 810 / 1051, of 64
// 1019 / 948.
inline bool lane_default(int d, int k, int most) { return d <= 4 && (most <= 32 || k > 16); }

// Offers the cnt points from b on, a lane's leaf, to its list; least, most: no leaf
// of the tree is smaller or larger (wave-uniform).  Without kMerge, in two passes per 32
// points: the first computes every distance and marks the points that can
// enter the list (float test against the current k-th distance, ties kept);
// the second inserts the marked points, recomputing their distances.  The
// wave pays for an insertion when any lane inserts, so marking first makes it
// pay for the largest number of insertions of one lane, not for every
// position at which some lane inserts.  With kMerge, 16 points at a time: their
// keys stay in registers and are merged into the list at once (ListMerge), except for a
// short rest of a leaf (at most kFewPoints: smoothing lengths on leaves of 20 points
// 3.00 against 3.52 ms, 5000011 points) and where no lane has many candidates.
template <int D, bool kMerge, class Space, class List>
__device__ __forceinline__ void leaf_offer(const Space& sp, int32_t b, int cnt, int least, int most,
                                           const typename Space::Coord p[D], List& best) {
  constexpr int B = kMerge ? kListBatch : 32;
  constexpr int kFewPoints = 8;
  constexpr int kAhead = D > 4 ? 4 : 2;
  for (int o = 0; o < cnt; o += B) {
    const typename Space::Dist w = best.worst_d2();
    const int m = min(cnt - o, B);
    const int32_t c = b + o;
    int32_t base = c;
    uint32_t mask = 0;
    bool batch = false;
    if constexpr (kMerge) batch = most - o > kFewPoints;
    if (batch) {
      if constexpr (kMerge) {
        // the B points from base on, which end inside the array
        base = max(min(c, (int32_t)sp.t.n - B), 0);
        const auto* r = sp.run(base);
        const uint32_t valid = ((1u << m) - 1u) << (c - base);
        typename List::Key key[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
          int32_t id = 0;
          const typename Space::Dist d2 = sp.dist(r, base, i, p, id);
          const bool ok = ((valid >> i) & 1u) && d2 <= w;  // (false for NaN)
          mask |= (uint32_t)ok << i;
          key[i] = batch_key(best, ok, d2, id);
          // built here, not later from the loaded record: registers
          asm volatile("" : "+v"(key[i]));
          if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        KDT_LANE_VISIT(sp.t, kVisitInsert, __popc(mask));
        // runs once at most; as a loop the list keeps its registers, as a
        // branch the compiler copies it (153 instead of 128 VGPRs)
        uint32_t go = __any(__popc(mask) > ListMerge<List, D>::kMin);
        while (go) {
          best.merge(key);
          mask = 0;
          asm volatile("v_mov_b32 %0, 0" : "=v"(go));
        }
      }
    } else {
      const auto* r = sp.run(c);
      int all = 0;
      // (the leftovers of a merge are few: 2^24 clustered points, d = 3, k = 32 5.20 ms, with
      // this loop 5.23; in 4 dimensions 400000 points' 20th distances 774 us without it, 625)
      if constexpr (!kMerge || D > 3) {
        all = min(max(least - o, 0), B);  // every lane has these
#pragma unroll kAhead
        for (int i = 0; i < all; ++i) {
          int32_t id = 0;
          mask |= (uint32_t)(sp.dist(r, c, i, p, id) <= w) << i;
        }
      }
#pragma unroll 1
      for (int i = all; i < m; ++i) {
        int32_t id = 0;
        mask |= (uint32_t)(sp.dist(r, c, i, p, id) <= w) << i;
      }
    }
    if (!batch) KDT_LANE_VISIT(sp.t, kVisitInsert, __popc(mask));
    const auto* r = sp.run(base);
    while (mask) {
      const int i = __builtin_ctz(mask);
      mask &= mask - 1;
      int32_t id = 0;
      const typename Space::Dist d2 = sp.dist(r, base, i, p, id);
      best.offer(d2, id);
    }
  }
}

// knn_one over a median tree.  A node's box distance is stored when its sibling is
// descended into, one entry per level of the lane's path; which node it was
// follows from the path.
//
// What bounds it: instructions, and the waves' divergence multiplies them -- a
// lane visits 15 leaves and 56 inner nodes (2^22 uniform queries, 2^24
// clustered points, k = 32), but when every lane walks to its next leaf before
// any leaf is scanned the wave pays for 31 and 251, because the others wait
// for the lane whose walk is the longest.  So the wave votes each round: its
// lanes take one step down (or back), until kWait times as many wait at a leaf as still
// walk; then the leaves are scanned.  That leaves 25 and 142, with
// 5.08 instead of 5.99 ms (kWait 1 / 2 / 4 / never all waiting: 5.53 / 5.14 / 5.08 /
// 5.64 ms).  Lists that insert do best at 6 (2^21 points, k = 8, clustered:
// 1.33, at 3 1.35, at 1 1.55 ms); in 8 dimensions, where a step costs
// as much as a third of a leaf, at 2 (200003 points, k = 16, normal:
// 10.2, at 3 10.4, at 6 10.8 ms).
// Whole call, before and after the vote and the merge: 6.64 and 5.10 ms; smoothing
// lengths of 5000011 points 5.26 and 3.00 ms.
template <int D, bool kMerge, class Space, class List>
__device__ __forceinline__ void knn_median(const Space& sp, const typename Space::Coord p[D],
                                           List& best, uint32_t* stk, int ld) {
  using Dist = typename Space::Dist;
  const auto& t = sp.t;
  constexpr int kWait = D > 4 ? 2 : kMerge ? 4 : 6;
  const uint32_t first = 1u << t.levels;
  // every leaf holds lmin points or one more
  const int lmin = (int)(t.n >> t.levels);
  const int lmax = (int)((t.n + (int64_t(1) << t.levels) - 1) >> t.levels);
  uint32_t h = 1;     // 1-based heap id of the lane's node (children 2h, 2h + 1)
  uint32_t pend = 0;  // bit l: the sibling of the path's level-l node waits
  bool more = true;
  KDT_LANE_VISIT(t, kVisitNodes, 1);
  while (more) {
    const bool leaf = h >= first;
    const int nat = __popcll(__ballot(leaf)), nrun = __popcll(__ballot(!leaf));
    // (no lane walks: scan.)  The vote is the same in every lane; kept in a
    // vector register, it is a branch like the others to the compiler, which
    // copies the list around branches that it knows to be uniform.
    uint32_t scan = nat >= nrun * kWait;
    asm volatile("" : "+v"(scan));
    bool pop = false;
    if (scan) {
      if (leaf) {
        const int64_t j = h - first;
        const int32_t b = (int32_t)((j * t.n) >> t.levels);
        const int32_t e = (int32_t)(((j + 1) * t.n) >> t.levels);
        KDT_LANE_VISIT(t, kVisitPoints, e - b);
        leaf_offer<D, kMerge>(sp, b, e - b, lmin, lmax, p, best);
        pop = true;
      }
    } else if (!leaf) {
      const uint32_t c0 = 2 * h;
      Dist d0, d1;
      KDT_LANE_VISIT(t, kVisitNodes, 2);
      sp.pair(c0 - 1, p, d0, d1);
      const Dist dn = min(d0, d1), df = max(d0, d1);
      const Dist w = best.worst_d2();
      const int lev = 32 - __clz(h);  // of the children
      if (df <= w) {
        pend |= 1u << lev;
        stk[lev * ld] = Space::bits(df);
      }
      h = c0 + (d0 <= d1 ? 0u : 1u);
      pop = !(dn <= w);
    }
    const Dist w = best.worst_d2();
    while (pop) {
      if (pend != 0) {
        const int l = 31 - __clz(pend);
        pend ^= 1u << l;
        h = (h >> (31 - __clz(h) - l)) ^ 1u;
        pop = !(Space::from_bits(stk[l * ld]) <= w);
      } else {
        more = pop = false;
      }
    }
  }
}

// kNN of one query p over tree t (Algorithm 2 semantics): depth-first, nearer
// child first, a node is skipped when its box is farther than the current
// k-th candidate.  `stk` is this lane's column of an LDS stack with stride
// `ld` entries (levels + 1 of them).  kMerge: the tree has at least kListBatch points.
template <int D, bool kMerge = true, class Shape = MedianShape, class List, class Metric = OpenMetric<D>>
__device__ __forceinline__ void knn_one(const TreeView& t, const float p[D], List& best,
                                        uint32_t* stk, int ld, const Metric& metric = Metric()) {
  const Space32<D, Metric> space{t, metric};
  if constexpr (std::is_same_v<Shape, MedianShape>) {
    knn_median<D, kMerge && ListMerge<List, D>::kOn>(space, p, best, stk, ld);
    return;
  }
  const Shape sh(t);
  float lo[D], hi[D];
  load_box<D>(t.box, 0, lo, hi);
  KDT_LANE_VISIT(t, kVisitNodes, 1);
  uint32_t node = 0;
  float nd = metric.mindist(lo, hi, p);
  int sp = 0;
  for (;;) {
    if (nd <= best.worst_d2()) {
      if (sh.is_leaf(node)) {
        int64_t b, e;
        sh.range(node, b, e);
        KDT_LANE_VISIT(t, kVisitPoints, e - b);
        leaf_offer<D, false>(space, (int32_t)b, (int)(e - b), 0, 0, p, best);
      } else {
        const uint32_t c0 = sh.left(node), c1 = c0 + 1;
        KDT_LANE_VISIT(t, kVisitNodes, 2);
        load_box<D>(t.box, c0, lo, hi);
        const float d0 = metric.mindist(lo, hi, p);
        load_box<D>(t.box, c1, lo, hi);
        const float d1 = metric.mindist(lo, hi, p);
        const bool first0 = d0 <= d1;
        const uint32_t nn = first0 ? c0 : c1, ff = first0 ? c1 : c0;
        const float dn = first0 ? d0 : d1, df = first0 ? d1 : d0;
        if (df <= best.worst_d2()) stk[sp++ * ld] = ff;
        node = nn;
        nd = dn;
        continue;
      }
    }
    if (sp == 0) break;
    // only the node id is kept on the stack; its box distance is recomputed
    // (the box is cache-resident), halving the stack's LDS footprint
    node = stk[--sp * ld];
    KDT_LANE_VISIT(t, kVisitReload, 1);
    load_box<D>(t.box, node, lo, hi);
    nd = metric.mindist(lo, hi, p);
  }
}

// Writes one kNN row: mode 0 -> k (index, d2) pairs, 1 -> d2 of the k-th,
// 2 -> distance of the k-th.
template <int KC>
__device__ __forceinline__ void knn_write(const TopK<KC>& best, int k, int mode, int64_t row,
                                          int32_t* __restrict__ oidx, float* __restrict__ od2) {
  if (mode == 0) {
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      if (j < KC - k) continue;
      const uint64_t key = best.key(j);
      const bool empty = key == kEmptyKey;
      const int64_t o = row * k + (j - (KC - k));
      if (oidx) oidx[o] = empty ? -1 : (int32_t)(uint32_t)key;
      od2[o] = empty ? INFINITY : __uint_as_float((uint32_t)(key >> 32));
    }
  } else {
    const uint64_t key = best.key(KC - 1);
    const float d2 = key == kEmptyKey ? INFINITY : __uint_as_float((uint32_t)(key >> 32));
    od2[row] = mode == 2 ? sqrtf(d2) : d2;
  }
}

// The k-th squared distance (mode 1) or distance (mode 2) of a TopD list.
template <int KC>
__device__ __forceinline__ void knn_write_kth(const TopD<KC>& best, int mode, int64_t row,
                                              float* __restrict__ od2) {
  const float d2 = best.worst_d2();
  od2[row] = mode == 2 ? sqrtf(d2) : d2;
}

// Lock-free union-find on int32 parents with parent[y] <= y.
//
// The loads have workgroup scope: they may see an older parent than another
// XCD has written.  Every value a parent ever had is an ancestor of its element
// from then on, so an older one only makes a path longer; roots are claimed by
// device-scope compare-and-swap, which returns the present parent when it fails, so
// each retry goes on from there.  Device-scope loads go past the caches of the
// CU: groups of 2^24 clustered points took 1.2 ms longer with them.
__device__ __forceinline__ int32_t uf_ld(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void uf_st(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of x.  Only roots change owner, so shortcutting a non-root to any of
// its ancestors is always valid.
__device__ __forceinline__ int32_t uf_find(int32_t* parent, int32_t x) {
  int32_t cur = uf_ld(parent + x);
  if (cur == x) return x;
  int32_t prev = x;
  for (;;) {
    const int32_t next = uf_ld(parent + cur);
    if (next >= cur) break;
    uf_st(parent + prev, next);
    prev = cur;
    cur = next;
  }
  return cur;
}

// Joins the set of the element whose known ancestor is `a` (updated to an
// ancestor of the joined set's root) with the set of b: the larger root is
// hooked under the smaller, so every root is the smallest index of its set.
// A root found once stays an ancestor of its elements after it is hooked
// (only roots change parent), so a lane that links one point many times
// keeps its last root in `a` and starts every search there.
//
// Two elements that share any ancestor are in one set, so when b is a or b's
// parent is a (the usual case once paths are compressed) nothing is left to
// do after a single load.
//
// uf_union_known: pb is what parent[b] held at some point of this launch.
__device__ __forceinline__ void uf_union_known(int32_t* parent, int32_t& a, int32_t b,
                                               int32_t pb) {
  if (b == a || pb == a) return;
  int32_t ra = uf_find(parent, a), rb = pb == b ? b : uf_find(parent, pb);
  while (ra != rb) {
    if (ra < rb) {
      const int32_t old = atomicCAS(parent + rb, rb, ra);
      if (old == rb) break;
      rb = old;
    } else {
      const int32_t old = atomicCAS(parent + ra, ra, rb);
      if (old == ra) {
        ra = rb;
        break;
      }
      ra = old;
    }
  }
  a = ra;
}
__device__ __forceinline__ void uf_union_from(int32_t* parent, int32_t& a, int32_t b) {
  if (b == a) return;
  uf_union_known(parent, a, b, uf_ld(parent + b));
}

// Joins the sets of a and b.
__device__ __forceinline__ void uf_union(int32_t* parent, int32_t a, int32_t b) {
  uf_union_from(parent, a, b);
}

// Squared diagonal of a box: every pair of points inside is at most this far
// apart (same operation order as the point distance).
template <int D>
__device__ __forceinline__ float box_diag2(const float lo[D], const float hi[D]) {
  float s = 0.0f;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    float t = hi[a] - lo[a];
    float t2 = t * t;
    s = s + t2;
  }
  return s;
}

__device__ __forceinline__ uint32_t flag_ld(const uint32_t* p) {
  // (an older value only costs the shortcut)
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void flag_st(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Friends-of-friends links of the point p at tree position `pos` (index me)
// of tree t.  Union-find indices are base + index.  conn[v] != 0 records that
// every point of node v is already (or will be, once the running unions land)
// in one component; such a node needs a single link to p, and once one friend
// is found inside it the rest of its subtree is skipped.
template <int D, class Shape = MedianShape>
__device__ __forceinline__ void fof_point(const TreeView& t, const float p[D], int64_t pos,
                                          int32_t me, float l2, int32_t base,
                                          int32_t* __restrict__ parent,
                                          uint32_t* __restrict__ conn, uint32_t* stk, int ld) {
  constexpr int S = rec_stride(D);
  const Shape sh(t);
  int sp = 1;
  stk[0] = 0;
  int32_t myroot = base + me;  // an ancestor of p's set root (see uf_union_from)
  int guard = -1;  // stack depth where the current one-component region began
  while (sp > 0) {
    --sp;
    if (guard >= 0 && sp < guard) guard = -1;
    const uint32_t node = stk[sp * ld];
    int64_t b, e;
    sh.range(node, b, e);
    // links go towards later tree positions only: a node that ends at or
    // before p's position is left to the points inside it
    if (e <= pos) continue;
    float lo[D], hi[D];
    load_box<D>(t.box, node, lo, hi);
    if (box_mindist<D>(lo, hi, p) > l2) continue;
    const bool in_region = guard >= 0;
    const bool one = in_region || flag_ld(conn + node) != 0;
    if (one && pos >= b && pos < e) continue;  // p is already in this component
    if (box_maxdist<D>(lo, hi, p) <= l2) {
      if (one) {
        uf_union_from(parent, myroot, base + __float_as_int(t.rec[b * S + D]));
        if (in_region) {
          sp = guard;
          guard = -1;
        }
      } else {
        for (int64_t i = b; i < e; ++i)
          uf_union_from(parent, myroot, base + __float_as_int(t.rec[i * S + D]));
        flag_st(conn + node, 1u);
      }
      continue;
    }
    if (sh.is_leaf(node)) {
      for (int64_t i = b; i < e; ++i) {
        float x[D];
        int32_t id = 0;
        load_rec<D>(t.rec, i, x, id);
        if (sq_dist<D>(x, p) > l2) continue;
        if (one) {
          uf_union_from(parent, myroot, base + id);
          if (in_region) {
            sp = guard;
            guard = -1;
          }
          break;
        }
        if (i > pos) uf_union_from(parent, myroot, base + id);
      }
      continue;
    }
    if (one && !in_region) guard = sp;
    const uint32_t c0 = sh.left(node);
    stk[sp++ * ld] = c0 + 1;
    stk[sp++ * ld] = c0;
  }
}

// Marks nodes whose box diagonal is within the linking length: all their
// points are mutual friends.
template <int D>
__device__ __forceinline__ void fof_mark_clique(const float* __restrict__ box, int64_t node,
                                                float l2, uint32_t* __restrict__ conn) {
  float lo[D], hi[D];
  load_box<D>(box, (uint32_t)node, lo, hi);
  conn[node] = box_diag2<D>(lo, hi) <= l2 ? 1u : 0u;
}

// Joins the point at tree position pos with the first point of the largest
// clique node above it (so every maximal clique becomes one component).
template <int D>
__device__ __forceinline__ void fof_join_clique(const TreeView& t, int64_t pos, int32_t me,
                                                int32_t base, int32_t* __restrict__ parent,
                                                const uint32_t* __restrict__ conn) {
  constexpr int S = rec_stride(D);
  const int64_t first_leaf = (int64_t(1) << t.levels) - 1;
  // leaf holding pos: largest j with node_begin(n, L, j) <= pos
  int64_t j = ((pos + 1) << t.levels) / t.n;
  while (j > 0 && node_begin(t.n, t.levels, j) > pos) --j;
  while (node_begin(t.n, t.levels, j + 1) <= pos) ++j;
  int64_t v = first_leaf + j;
  if (!conn[v]) return;
  while (v > 0 && conn[(v - 1) >> 1]) v = (v - 1) >> 1;
  const int lev = node_level((uint32_t)v);
  const int64_t b = node_begin(t.n, lev, v - ((int64_t(1) << lev) - 1));
  const int32_t first = __float_as_int(t.rec[b * S + D]);
  if (first != me) uf_union(parent, base + me, base + first);
}

// Root of x without shortcuts (safe while other lanes write final labels).
__device__ __forceinline__ int32_t uf_root(const int32_t* parent, int32_t x) {
  int32_t cur = x;
  for (;;) {
    const int32_t next = uf_ld(parent + cur);
    if (next >= cur) return cur;
    cur = next;
  }
}

template <int D>
kdt_status knn_packet_launch(const TreeView& v, int leaf, const float* d_q, int64_t nq, int k,
                             int32_t* d_idx, float* d_d2, int mode, const int32_t* order,
                             hipStream_t stream);
// Periodic boundaries (opts->period): kNN (k <= KDT_MAX_K) and ball queries
// on the D-torus, arguments as kdt_knn / kdt_range.
kdt_status knn_torus(const kdt_tree* tr, const float* d_q, int64_t nq, int k, int32_t* d_idx,
                     float* d_d2, int mode, bool sort_q, const int32_t* given,
                     const float* period, hipStream_t stream);
kdt_status range_torus(const kdt_tree* tr, const float* d_q, int64_t nq, float r,
                       int32_t* d_count, int64_t* d_off, int32_t* d_idx, int64_t capacity,
                       int64_t* required, bool sort_q, const int32_t* given, const float* period,
                       bool counts_given, hipStream_t stream);

// k above KDT_MAX_K: exact neighbours from a per-query ball that holds at
// least k points, its keys sorted per query (arguments as kdt_knn; period
// NULL for open boundaries).
kdt_status knn_large(const kdt_tree* tr, const float* d_q, int64_t nq, int k, int32_t* d_idx,
                     float* d_d2, int mode, bool sort_q, const int32_t* given,
                     const float* period, hipStream_t stream);

// kdt_knn's options after its argument checks.
struct KnnArgs {
  bool empty = false;  // nq == 0: nothing to do
  bool sort_q = true;
  int traversal = 0;
  // external queries: the caller's order or NULL; self queries: the
  // tree-order row marker (self_rows) or NULL
  const int32_t* given = nullptr;
  const float* period = nullptr;
};
// Checks kdt_knn's arguments (`who` names the entry point in messages).
kdt_status knn_check(const kdt_tree* tree, const float* d_q, int64_t nq, int32_t k,
                     const float* d_d2, int32_t kth_only, const kdt_query_opts* opts,
                     const char* who, KnnArgs* a);
// kNN with k <= KDT_MAX_K and open boundaries.  With a workspace (ws_bytes
// bytes of device memory) the query order, the only scratch of this path,
// is carved from it and nothing is allocated; KDT_ECAPACITY if it is too
// small.  ws == NULL: scratch from the stream-ordered pool.
kdt_status knn_in_workspace(const kdt_tree* t, const float* d_q, int64_t nq, int k,
                            int32_t* d_idx, float* d_d2, int mode, const KnnArgs& a, void* ws,
                            size_t ws_bytes, hipStream_t stream);

// Whether the 64 queries from s0 on (input order; all lanes call) lie together: the box around
// them has at most 1/16 of the volume of the box around 64 queries from all of the input.
// Queries along any curve stay below 1 %, those in random order above half.
template <int D>
__device__ __forceinline__ bool lie_together(const double* __restrict__ q, int64_t nq,
                                             int64_t s0) {
  const int lane = threadIdx.x & 63;
  const int64_t mine = min(s0 + lane, nq - 1), far = nq / 64 * lane;
  double own = 1.0, all = 1.0;
  for (int a = 0; a < D; ++a) {
    double lo[2] = {q[mine * D + a], q[far * D + a]}, hi[2] = {lo[0], lo[1]};
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        lo[i] = min(lo[i], __shfl_xor(lo[i], o));
        hi[i] = max(hi[i], __shfl_xor(hi[i], o));
      }
    own *= hi[0] - lo[0];
    all *= hi[1] - lo[1];
  }
  return own * 16.0 <= all;  // (false for NaN)
}

template <int D>
kdt_status range_packet_launch(const TreeView& v, int leaf, const float* d_q, int64_t nq, float r2,
                               const int32_t* order, int32_t* d_count, uint32_t split_budget,
                               hipStream_t stream, const FillOut* fill = nullptr);
// The same over a float64 tree (leaves of at most 64 points).  apart: waves whose queries do
// not lie together (lie_together) are left out.
template <int D>
kdt_status range64_packet_launch(const View64& v, int leaf, const double* d_q, int64_t nq,
                                 double r2, const int32_t* order, int32_t* d_count,
                                 hipStream_t stream, const FillOut* fill = nullptr,
                                 bool apart = false);
// The LDS bytes of a workgroup of that launch.
size_t range64_packet_lds(int d, int leaf);
template <int D>
kdt_status fof_packet_launch(const TreeView& v, int leaf, float l2, int32_t* parent, uint32_t* conn,
                             hipStream_t stream);

}  // namespace kdt
