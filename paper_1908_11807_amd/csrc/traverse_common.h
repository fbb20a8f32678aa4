// Device code shared by the traversal kernels (plain trees and forests):
// tree views, node decoding, per-lane stacks and the nearest-neighbour walk.
// See traverse.hip for the method (ArborX paper, section 2.2).
#pragma once

#include <climits>

#include "abx_internal.h"

namespace abx {

constexpr int kTravBlock = 256;
constexpr int kMaxDepth = 128;
constexpr int kLdsDepthSpatial = 16;
constexpr int kLdsDepthNearest = 8;
// LDS stack window of the one-lane nearest pass (16-bit stack distances,
// six-byte entries) for an occupancy target of `waves` per SIMD: 16 entries
// take 6 KB a wavefront (six wavefronts a SIMD), 32 take 12 KB (three).  The 16
// entries also cap the k <= 4 walks, whose target is eight waves, at six: at k =
// 1 on the C3 shell that ran 9 % faster than 8 entries at eight waves.
constexpr int lane_window(int waves) { return waves > 3 ? 16 : 32; }
constexpr int kMaxRegK = 64;    // largest k kept in registers (lists of 1..64 keys)
constexpr int kMaxHeapK = 128;  // largest k (the LDS-heap kernel serves 65..128)

// Occupancy target of the one-lane nearest pass (waves per SIMD).  Six beat
// eight at k = 10 on the C3 shell (fewer walks competing for L2, no spills);
// the k = 32 list alone takes 64 registers.
// 4-wide walks hold four slots' distances and keys: at the binary targets
// they spilled (66 registers at k = 10); these targets leave them unspilled.
constexpr int nearest_waves_per_eu(int K, int FMT = 0) {
  return FMT == ABX_NODES_Q16W ? (K > 16 ? 2 : (K > 10 ? 3 : (K > 4 ? 5 : 6)))
                               : (K > 48 ? 2 : (K > 16 ? 3 : (K > 10 ? 4 : (K > 4 ? 6 : 8))));
}

struct TreeArgs {
  const void *nodes;
  const void *leaves;
  int64_t n;
  int64_t nint;            // internal nodes stored (n - 1; fewer for 4-wide nodes)
  int32_t root;            // internal node at the root (n >= 2)
  float scene[6];
  float qo[3], qs[3];
  const float *scene_dev;  // the same scene box in device memory
  const float *qframe;     // if set: Q16 origin[3], scale[3] in device memory (read at
                           // kernel start; used where the host has not read them back)
  const TreeHeader *guard; // if set: the construction's header, read at kernel start
                           // (forests, whose build the host does not wait for)
};

// A tree whose construction reported a problem (any flag, or a height the
// stacks cannot hold) is not walked: its nodes may not form a tree.
__device__ __forceinline__ bool tree_unusable(const TreeArgs &t) {
  return t.guard && (t.guard->bad != 0 || t.guard->height + 8 >= kMaxDepth);
}

__device__ __forceinline__ void resolve_qframe(TreeArgs &t) {
  if (t.qframe) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      t.qo[a] = t.qframe[a];
      t.qs[a] = t.qframe[3 + a];
    }
  }
}

struct QueryArgs {
  const float *data;
  int64_t m;
  const float *radii;
  float radius;
  const int32_t *order;  // sorted position -> caller's query index (or null)
  KeptRows kept;         // keeping pass, and the fill after it
  // one-pass (1P) scheme only
  int32_t *buf;          // [m * bufsize] stored hits, one row per sorted position
  int32_t bufsize;
  uint32_t *flag;        // [0] != 0: some query found more than bufsize hits
  const int64_t *total;  // device total of the scanned counts
  int64_t capacity;      // entries the caller's index buffer holds
};

// hardware dispatches workgroup b to XCD b % 8; hand XCD x a contiguous
// range of tiles so neighbouring (Morton-adjacent) tiles share an L2
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t nb) {
  const int64_t x = b & 7, k = b >> 3, q = nb >> 3, rem = nb & 7;
  return x * q + (x < rem ? x : rem) + k;
}

struct Kids {
  float l[6], r[6];
  int32_t lref, rref;
};

// Child references: r >= 0 is internal node r; r < 0 is a leaf holding
// primitive ~r.  Whether a node's child slot already holds a leaf's exact
// box: always for FP32 nodes (the slot is the primitive's box), and for Q16
// point trees (the slot holds the point's float32 coordinates).  Q16 box
// trees keep a quantised box in the slot and the exact box in a record
// addressed by primitive index.
template <int KIND, int FMT>
constexpr bool exact_leaf_slots() {
  return FMT == ABX_NODES_FP32 || KIND == ABX_PRIM_POINTS;
}

// The node's loads are kept together, ahead of everything that uses them: the
// lanes of a wavefront read 64 different lines, far more wavefronts run than
// a CU's L1 holds lines for, and a load scheduled behind arithmetic finds the
// line that its predecessor fetched evicted (k = 10 on the C3 shell, one-lane
// pass 133 ms with the loads left to the scheduler, 119 ms together).
template <int KIND, int FMT>
__device__ __forceinline__ void load_kids(const TreeArgs &t, int32_t node, Kids &k) {
  if (FMT == ABX_NODES_FP32) {
    const float4 *p = reinterpret_cast<const float4 *>(t.nodes) + 4 * (int64_t)node;
    const float4 a = p[0], b = p[1], c = p[2];
    const int2 d = *reinterpret_cast<const int2 *>(p + 3);
    __builtin_amdgcn_sched_barrier(0);
    k.l[0] = a.x; k.l[1] = a.y; k.l[2] = a.z; k.l[3] = a.w; k.l[4] = b.x; k.l[5] = b.y;
    k.r[0] = b.z; k.r[1] = b.w; k.r[2] = c.x; k.r[3] = c.y; k.r[4] = c.z; k.r[5] = c.w;
    k.lref = d.x;
    k.rref = d.y;
  } else {
    const uint4 *p = reinterpret_cast<const uint4 *>(t.nodes) + 2 * (int64_t)node;
    const uint4 a = p[0], b = p[1];
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t w[6] = {a.x, a.y, a.z, a.w, b.x, b.y};
    k.lref = (int32_t)b.z;
    k.rref = (int32_t)b.w;
    const bool pl = KIND == ABX_PRIM_POINTS && k.lref < 0;
    const bool pr = KIND == ABX_PRIM_POINTS && k.rref < 0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const uint32_t q = (w[j / 2] >> (16 * (j & 1))) & 0xffffu;
      const int ax = j % 3;
      const float v = deq(q, t.qs[ax], t.qo[ax]);
      k.l[j] = pl ? __uint_as_float(w[ax]) : v;
    }
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const uint32_t q = (w[3 + j / 2] >> (16 * (j & 1))) & 0xffffu;
      const int ax = j % 3;
      const float v = deq(q, t.qs[ax], t.qo[ax]);
      k.r[j] = pr ? __uint_as_float(w[3 + ax]) : v;
    }
  }
}

// The four children of a 4-wide node (FMT == ABX_NODES_Q16W).  An unused
// slot has reference kEmptyRef and is never taken.
struct Kids4 {
  float b[4][6];
  int32_t ref[4];
};

template <int KIND>
__device__ __forceinline__ void load_kids4(const TreeArgs &t, int32_t node, Kids4 &k) {
  const uint4 *p = reinterpret_cast<const uint4 *>(t.nodes) + 4 * (int64_t)node;
  const uint4 a = p[0], b = p[1], c = p[2], d = p[3];
  const uint32_t w[12] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w};
  k.ref[0] = (int32_t)d.x;
  k.ref[1] = (int32_t)d.y;
  k.ref[2] = (int32_t)d.z;
  k.ref[3] = (int32_t)d.w;
#pragma unroll
  for (int c4 = 0; c4 < 4; ++c4) {
    const bool pt = KIND == ABX_PRIM_POINTS && k.ref[c4] < 0;  // a point leaf (or unused)
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const uint32_t q = (w[3 * c4 + j / 2] >> (16 * (j & 1))) & 0xffffu;
      const int ax = j % 3;
      const float v = deq(q, t.qs[ax], t.qo[ax]);
      k.b[c4][j] = pt ? __uint_as_float(w[3 * c4 + ax]) : v;
    }
  }
}

// exact box of primitive `idx` of a Q16 box tree (its leaf record)
__device__ __forceinline__ void load_leaf_box(const TreeArgs &t, int32_t idx, float b[6]) {
  const float4 *p = reinterpret_cast<const float4 *>(t.leaves) + 2 * (int64_t)idx;
  const float4 u = p[0], v = p[1];
  b[0] = u.x; b[1] = u.y; b[2] = u.z; b[3] = u.w; b[4] = v.x; b[5] = v.y;
}

// Per-lane stack with its top in LDS.  Positions [sp - nl, sp) (at most S
// entries) live in a circular LDS window, slot (position mod S) of the
// lane's column (stride B lanes); deeper positions live in the lane's
// private memory at ovf[position].  A push into a full window first moves
// the window's bottom entry to private memory; a pop from an empty window
// reads private memory directly.  A walk that pushes and pops near the top
// (a depth-first traversal oscillating around some depth) therefore stays in
// LDS, and private memory is touched only when the depth drifts by more than
// S.  The LDS part is addressed through an explicit LDS (address space 3)
// pointer so the two paths stay separate instructions.
#define ABX_LDS __attribute__((address_space(3)))

template <typename T, int S, int B>
__device__ __forceinline__ void stack_push(ABX_LDS T *lds, T *ovf, int &sp, int &nl, T x) {
  static_assert((S & (S - 1)) == 0, "window size is a power of two");
  const int slot = (sp & (S - 1)) * B;
  if (nl == S) ovf[sp - S] = lds[slot];
  else ++nl;
  lds[slot] = x;
  ++sp;
}

template <typename T, int S, int B>
__device__ __forceinline__ T stack_pop(ABX_LDS T *lds, const T *ovf, int &sp, int &nl) {
  --sp;
  T v;
  if (nl > 0) {
    --nl;
    v = lds[(sp & (S - 1)) * B];
  } else {
    v = ovf[sp];
  }
  return v;
}

// The nearest traversal's stack holds (node, box distance) pairs.  The
// distance is stored as a float, or as its upper 16 bits (DT = uint16_t):
// truncating a non-negative float rounds it down, so the stored value is a
// lower bound of the box distance, and a node that the exact value would
// have pruned when popped is visited instead, its children (boxes inside
// its box, no nearer) then pruned: the same results, 6-byte entries.
__device__ __forceinline__ float stk_enc(float d, float) { return d; }
__device__ __forceinline__ uint16_t stk_enc(float d, uint16_t) {
  return (uint16_t)(__float_as_uint(d) >> 16);
}
__device__ __forceinline__ float stk_dec(float d) { return d; }
__device__ __forceinline__ float stk_dec(uint16_t d) { return __uint_as_float((uint32_t)d << 16); }

template <int S, int B, typename DT>
__device__ __forceinline__ void stack_push2(ABX_LDS int32_t *ln, ABX_LDS DT *ld, int32_t *on,
                                            DT *od, int &sp, int &nl, int32_t n, float d) {
  static_assert((S & (S - 1)) == 0, "window size is a power of two");
  const int slot = (sp & (S - 1)) * B;
  if (nl == S) {
    on[sp - S] = ln[slot];
    od[sp - S] = ld[slot];
  } else {
    ++nl;
  }
  ln[slot] = n;
  ld[slot] = stk_enc(d, DT());
  ++sp;
}

template <int S, int B, typename DT>
__device__ __forceinline__ void stack_pop2(ABX_LDS int32_t *ln, ABX_LDS DT *ld, const int32_t *on,
                                           const DT *od, int &sp, int &nl, int32_t &n, float &d) {
  --sp;
  if (nl > 0) {
    --nl;
    const int slot = (sp & (S - 1)) * B;
    n = ln[slot];
    d = stk_dec(ld[slot]);
  } else {
    n = on[sp];
    d = stk_dec(od[sp]);
  }
}

enum { MODE_COUNT = 0, MODE_FILL = 1, MODE_STATS = 2, MODE_STORE = 3, MODE_KEEP = 4 };

// ------------------------------------------------------------------ nearest
// A candidate (squared distance d, primitive index i) packed into one
// signed 64-bit key: the float bits of d (d >= 0, so its bit pattern orders
// like the value) in the high word, i in the low word.  Key order is then
// exactly the (distance, index) order, and one 64-bit compare replaces the
// two-field comparison.  NaN distances pack above +inf and are never taken.
__device__ __forceinline__ int64_t knn_key(float d, int32_t i) {
  return (int64_t)(((uint64_t)__float_as_uint(d) << 32) | (uint32_t)i);
}
__device__ __forceinline__ float key_dist(int64_t key) {
  return __uint_as_float((uint32_t)((uint64_t)key >> 32));
}
__device__ __forceinline__ int32_t key_index(int64_t key) { return (int32_t)(uint32_t)key; }

// precedes every candidate (as a double: -inf)
constexpr int64_t kKeySentinel = (int64_t)0xfff0000000000000ull;
// an empty slot: (+inf, INT_MAX), preceded by every finite candidate
constexpr int64_t kKeyEmpty = (int64_t)(((uint64_t)0x7f800000u << 32) | 0x7fffffffu);

// Smaller and larger of two keys.  Read as doubles, keys order like the
// integers: candidates and the empty slot are finite and not negative (their
// top bits are those of a float up to +inf, whose pattern is below a double's
// exponent of infinity), denormal ones included, which the double-precision
// minimum and maximum keep.  One instruction each, where the integer form
// takes a compare and two selects.  (asm: the compiler would first
// canonicalise both operands, an instruction each.)
__device__ __forceinline__ int64_t key_min(int64_t a, int64_t b) {
  int64_t r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ int64_t key_max(int64_t a, int64_t b) {
  int64_t r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// The k best candidates of one lane, ascending keys.  Slots [0, K-k) hold
// sentinels that precede everything and never move; the k live slots start
// empty.
template <int K>
struct KnnList {
  int64_t key[K];
  __device__ __forceinline__ void init(int k) {
#pragma unroll
    for (int j = 0; j < K; ++j) key[j] = j < K - k ? kKeySentinel : kKeyEmpty;
  }
  __device__ __forceinline__ float kth() const { return key_dist(key[K - 1]); }
  // Insert x if it precedes the last entry, dropping the last entry: slot j
  // becomes the median of x, its entry and its predecessor's entry.  Fully
  // unrolled from the back (constant register indices, no copies): 2K - 1
  // instructions, no chain between the slots.  Cheap enough for a wavefront
  // to run at once for one lane: holding candidates back until several lanes
  // had one, which paid while an insertion took ~7K instructions, was slower
  // (k = 16 forest walk 13.6 ms with that, 11.6 with this insertion behind
  // it, 11.2 inserting at once; k = 32 on the 1e7 shell, 1e5 queries,
  // one-lane pass 8.2 -> 5.7 ms; k = 10 on 1e6 cube points 0.78 -> 0.69).
  __device__ __forceinline__ void offer_key(int64_t x) {
    if (x < key[K - 1]) {
#pragma unroll
      for (int j = K - 1; j > 0; --j) key[j] = key_max(key[j - 1], key_min(key[j], x));
      key[0] = key_min(key[0], x);
    }
  }
  __device__ __forceinline__ void offer(float d, int32_t idx) { offer_key(knn_key(d, idx)); }
};

struct KnnQuery {
  float x, y, z;
};

// A leaf child (primitive idx) whose node-stored box is at squared distance
// dbox: confirm with the exact box where the slot is quantised, and offer
// it to the list.  Candidates beyond `thr` (an upper bound of the final k-th
// distance) cannot be in the result.
template <int KIND, int FMT, int K>
__device__ __forceinline__ void knn_leaf(const TreeArgs &t, const KnnQuery &q, int32_t idx,
                                         float dbox, float thr, KnnList<K> &L, int32_t &reads) {
  if (!(dbox <= thr)) return;
  if (exact_leaf_slots<KIND, FMT>()) {
    L.offer(dbox, idx);
  } else {
    ++reads;
    float b[6];
    load_leaf_box(t, idx, b);
    const float d = box_dist2(b[0], b[1], b[2], b[3], b[4], b[5], q.x, q.y, q.z);
    if (d <= thr) L.offer(d, idx);
  }
}

// One step of the nearest walk: visit `node`, offer its leaf children, and
// return the nearer qualifying internal child (the farther one is pushed),
// or -1 when neither qualifies.
template <int KIND, int FMT, int K, int B, int S = kLdsDepthNearest, typename DT>
__device__ __forceinline__ int32_t knn_visit2(const TreeArgs &t, const KnnQuery &q, int32_t node,
                                              KnnList<K> &L, ABX_LDS int32_t *lds_n,
                                              ABX_LDS DT *lds_d, int32_t *ovf_n, DT *ovf_d,
                                              int &sp, int &nl, int32_t &reads) {
  Kids c;
  load_kids<KIND, FMT>(t, node, c);
  const float dl = box_dist2(c.l[0], c.l[1], c.l[2], c.l[3], c.l[4], c.l[5], q.x, q.y, q.z);
  const float dr = box_dist2(c.r[0], c.r[1], c.r[2], c.r[3], c.r[4], c.r[5], q.x, q.y, q.z);
  const bool ll = c.lref < 0, lr = c.rref < 0;
  if (exact_leaf_slots<KIND, FMT>()) {
    // both leaves tested against the bound before either enters the list: one
    // insertion's code runs for whichever child offers
    const float thr0 = L.kth();
    const bool ol = ll && dl <= thr0, orr = lr && dr <= thr0;
    if (ol || orr) {
      L.offer_key(ol ? knn_key(dl, ~c.lref) : knn_key(dr, ~c.rref));
      if (ol && orr) L.offer_key(knn_key(dr, ~c.rref));
    }
  } else {
    if (ll) knn_leaf<KIND, FMT, K>(t, q, ~c.lref, dl, L.kth(), L, reads);
    if (lr) knn_leaf<KIND, FMT, K>(t, q, ~c.rref, dr, L.kth(), L, reads);
  }
  const float thr = L.kth();
  const bool gl = !ll && dl <= thr, gr = !lr && dr <= thr;
  if (gl && gr) {
    // Visit order only (pruning uses the box distances): the child whose box
    // centre is nearer goes first.  Box distances of the large boxes near
    // the root say little about where the nearest primitives are (a box
    // around a curved or slanted patch reaches far in front of it); the
    // centre tracks the primitives better, so the list fills with near
    // candidates sooner and prunes more (C3: 16 % fewer visits).
    // (lo - q) - (q - hi) = 2 (centre - q), from the differences the box
    // distances already formed
    float cl = 0.0f, cr = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float qa = a == 0 ? q.x : (a == 1 ? q.y : q.z);
      const float ml = (c.l[a] - qa) - (qa - c.l[3 + a]);
      const float mr = (c.r[a] - qa) - (qa - c.r[3 + a]);
      cl = __fmaf_rn(ml, ml, cl);
      cr = __fmaf_rn(mr, mr, cr);
    }
    const bool left_first = cl <= cr;
    if (sp < kMaxDepth)
      stack_push2<S, B>(lds_n, lds_d, ovf_n, ovf_d, sp, nl, left_first ? c.rref : c.lref,
                        left_first ? dr : dl);
    return left_first ? c.lref : c.rref;
  }
  if (gl) return c.lref;
  if (gr) return c.rref;
  return -1;
}

// One 4-wide node decoded for a walk: per slot the squared box distance to
// q (+inf for an unused slot), the squared distance to the box centre
// (times 4; visit order only) and the reference.
template <int KIND>
__device__ __forceinline__ void wide_slots(const TreeArgs &t, int32_t node, const KnnQuery &q,
                                           float d[4], float key[4], int32_t r[4]) {
  const uint4 *p = reinterpret_cast<const uint4 *>(t.nodes) + 4 * (int64_t)node;
  const uint4 a = p[0], b = p[1], c = p[2], e = p[3];
  const uint32_t w[12] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w};
  r[0] = (int32_t)e.x;
  r[1] = (int32_t)e.y;
  r[2] = (int32_t)e.z;
  r[3] = (int32_t)e.w;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool pt = KIND == ABX_PRIM_POINTS && r[j] < 0;  // a point leaf (or unused)
    float lo[3], hi[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      const uint32_t ql = (w[3 * j + ax / 2] >> (16 * (ax & 1))) & 0xffffu;
      const uint32_t qh = (w[3 * j + (ax + 3) / 2] >> (16 * ((ax + 3) & 1))) & 0xffffu;
      const float pv = __uint_as_float(w[3 * j + ax]);
      lo[ax] = pt ? pv : deq(ql, t.qs[ax], t.qo[ax]);
      hi[ax] = pt ? pv : deq(qh, t.qs[ax], t.qo[ax]);
    }
    d[j] = r[j] == kEmptyRef ? INFINITY
                             : box_dist2(lo[0], lo[1], lo[2], hi[0], hi[1], hi[2], q.x, q.y, q.z);
    const float qv[3] = {q.x, q.y, q.z};
    float cc = 0.0f;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      const float m = (lo[ax] - qv[ax]) - (qv[ax] - hi[ax]);
      cc = __fmaf_rn(m, m, cc);
    }
    key[j] = cc;
  }
}

// The same step over a 4-wide node: leaf children are offered as above;
// the qualifying internal children are visited nearest box centre first:
// the nearest is returned and the others are pushed farthest first, so they
// come off the stack in the same order.
template <int KIND, int K, int B, int S = kLdsDepthNearest, typename DT>
__device__ __forceinline__ int32_t knn_visit_w(const TreeArgs &t, const KnnQuery &q, int32_t node,
                                               KnnList<K> &L, ABX_LDS int32_t *lds_n,
                                               ABX_LDS DT *lds_d, int32_t *ovf_n, DT *ovf_d,
                                               int &sp, int &nl, int32_t &reads) {
  // each slot is decoded straight into its box distance and centre key, so
  // the 24 coordinates are never live together (they made the walk spill)
  float d[4], key[4];
  int32_t r[4];
  wide_slots<KIND>(t, node, q, d, key, r);
  if (exact_leaf_slots<KIND, ABX_NODES_Q16W>()) {
    const float thr0 = L.kth();
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (r[j] < 0 && r[j] != kEmptyRef && d[j] <= thr0) L.offer_key(knn_key(d[j], ~r[j]));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (r[j] < 0 && r[j] != kEmptyRef)
        knn_leaf<KIND, ABX_NODES_Q16W, K>(t, q, ~r[j], d[j], L.kth(), L, reads);
  }
  const float thr = L.kth();
  // the qualifying internal children keep their key; the others sort last
  // with reference -1
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool g = r[j] >= 0 && d[j] <= thr;
    key[j] = g ? key[j] : INFINITY;
    r[j] = g ? r[j] : -1;
  }
  // sorting network on four (key, reference, distance) triples; a NaN key
  // only changes the order, never drops a child
  auto cx = [&](int i, int j) {
    if (key[j] < key[i] || (r[i] < 0 && r[j] >= 0)) {
      const float tk = key[i];
      key[i] = key[j];
      key[j] = tk;
      const int32_t tr = r[i];
      r[i] = r[j];
      r[j] = tr;
      const float td = d[i];
      d[i] = d[j];
      d[j] = td;
    }
  };
  cx(0, 1);
  cx(2, 3);
  cx(0, 2);
  cx(1, 3);
  cx(1, 2);
#pragma unroll
  for (int j = 3; j >= 1; --j)
    if (r[j] >= 0 && sp < kMaxDepth) stack_push2<S, B>(lds_n, lds_d, ovf_n, ovf_d, sp, nl, r[j], d[j]);
  return r[0];
}

template <int KIND, int FMT, int K, int B, int S = kLdsDepthNearest, typename DT>
__device__ __forceinline__ int32_t knn_visit(const TreeArgs &t, const KnnQuery &q, int32_t node,
                                             KnnList<K> &L, ABX_LDS int32_t *lds_n,
                                             ABX_LDS DT *lds_d, int32_t *ovf_n, DT *ovf_d,
                                             int &sp, int &nl, int32_t &reads) {
  if constexpr (FMT == ABX_NODES_Q16W)
    return knn_visit_w<KIND, K, B, S>(t, q, node, L, lds_n, lds_d, ovf_n, ovf_d, sp, nl, reads);
  else
    return knn_visit2<KIND, FMT, K, B, S>(t, q, node, L, lds_n, lds_d, ovf_n, ovf_d, sp, nl,
                                          reads);
}

// pop deferred nodes until one still qualifies; -1 when the stack runs dry
template <int B, int S = kLdsDepthNearest, typename DT>
__device__ __forceinline__ int32_t knn_pop(float thr, ABX_LDS int32_t *lds_n, ABX_LDS DT *lds_d,
                                           const int32_t *ovf_n, const DT *ovf_d, int &sp, int &nl) {
  while (sp > 0) {
    int32_t en;
    float ed;
    stack_pop2<S, B>(lds_n, lds_d, ovf_n, ovf_d, sp, nl, en, ed);
    if (ed <= thr) return en;
  }
  return -1;
}

// Where each query's walk starts and where its row goes.
struct QInfo {
  int32_t root;        // internal node to start from, or ~primitive for a one-leaf tree
  int kk;              // row length min(k, n of the query's tree)
  int64_t out;         // first output slot of the row
  int32_t base;        // subtracted from primitive indices (tree-local rows)
  const float *lbox;   // exact box of the leaf when root < 0
};

// One tree, every row of length k.
struct PlainMap {
  int k;
  __device__ __forceinline__ QInfo info(int64_t qi, const TreeArgs &t) const {
    QInfo r;
    r.root = t.n == 1 ? ~0 : t.root;
    r.kk = k;
    r.out = qi * k;
    r.base = 0;
    r.lbox = t.scene_dev;
    return r;
  }
};

template <int K>
__device__ __forceinline__ void knn_write(const KnnList<K> &L, int k, int32_t base, int32_t *oi,
                                          float *od) {
#pragma unroll
  for (int j = 0; j < K; ++j) {
    if (j >= K - k) {
      oi[j - (K - k)] = key_index(L.key[j]) - base;
      od[j - (K - k)] = sqrtf(key_dist(L.key[j]));
    }
  }
}

// Lists of more than 32 keys are not saved, their walks restart from the root:
// the save code's registers made them spill (48 keys: 9 -> 525 spill accesses).
constexpr bool saves_walk(int K) { return K <= 32; }

struct HeavyList {
  int32_t *q = nullptr;      // caller's query index
  float *bound = nullptr;    // k-th distance reached before the hand-off
  uint32_t *count = nullptr; // [0] entries, [1] next entry to serve
  int32_t *state = nullptr;  // saved walks, kHeavyStateWords words each (optional)
  uint32_t state_cap = 0;    // entries below this keep their walk
  uint32_t cap = UINT32_MAX; // entries from here on are not taken: their lanes walk on
};
static_assert(kHeavyStateWords == 2 + 2 * kHeavyStateEntries + 2 * kMaxRegK, "saved walk layout");

// Pass 1 for one query (one lane).  A walk that exceeds `budget` node
// visits stops and hands the query to the cooperative pass with the k-th
// distance it has found so far (an upper bound of the final one), unless the
// list is full: then it walks to its end.
template <int KIND, int FMT, int K, bool STATS, int B, int W, class Map, typename DT>
__device__ __forceinline__ void nearest_lane(const TreeArgs &t, const Map &map,
                                             const float *__restrict__ pts, int64_t qi,
                                             ABX_LDS int32_t *lds_n, ABX_LDS DT *lds_d,
                                             int32_t *__restrict__ indices, float *__restrict__ dist,
                                             int32_t *__restrict__ stats, int64_t budget,
                                             const HeavyList &heavy) {
  constexpr int kWin = W;  // LDS window entries per lane (lds_n, lds_d: stride B)
  const QInfo info = map.info(qi, t);
  if (info.kk == 0) {
    if (STATS) stats[2 * qi] = stats[2 * qi + 1] = 0;
    return;
  }
  const KnnQuery q{pts[3 * qi], pts[3 * qi + 1], pts[3 * qi + 2]};
  KnnList<K> L;
  L.init(info.kk);
  int32_t visited = 0, reads = 0;
  bool done = true;
  if (info.root < 0) {
    const float *b = info.lbox;
    const float d = box_dist2(b[0], b[1], b[2], b[3], b[4], b[5], q.x, q.y, q.z);
    knn_leaf<KIND, FMT, K>(t, q, ~info.root, d, INFINITY, L, reads);
  } else {
    int32_t ovf_n[kMaxDepth];
    DT ovf_d[kMaxDepth];
    int sp = 0, nl = 0;
    int32_t node = info.root;
    const int64_t limit = budget < t.n ? budget : t.n;
    done = false;
    // (two loops, not one of two parts: that costs every walk of k = 1 5 %)
    auto walk = [&](int64_t from, int64_t to) {
      for (int64_t it = from; it < to; ++it) {
        if (STATS) ++visited;
        node = knn_visit<KIND, FMT, K, B, kWin>(t, q, node, L, lds_n, lds_d, ovf_n,
                                                       ovf_d, sp, nl, reads);
        if (node < 0) node = knn_pop<B, kWin>(L.kth(), lds_n, lds_d, ovf_n, ovf_d, sp, nl);
        if (node < 0) {
          done = true;
          break;
        }
      }
    };
    walk(0, limit);
    uint32_t h = 0;
    if (!STATS && !done) {
      h = atomicAdd(heavy.count, 1u);
      if (h >= heavy.cap) walk(limit, t.n);
    }
    if (!STATS && !done && h < heavy.cap) {
      heavy.q[h] = (int32_t)qi;
      heavy.bound[h] = L.kth();
      // the walk so far: the next node (not yet visited), the unexplored
      // subtrees on the stack, the candidates; the workgroup resumes it.
      if (saves_walk(K) && heavy.state && h < heavy.state_cap) {
        int32_t *st = heavy.state + (int64_t)h * kHeavyStateWords;
        if (sp + 1 > kHeavyStateEntries) {
          st[0] = -1;  // too deep to save: the workgroup restarts from the root
        } else {
          st[2] = node;
          st[3] = __float_as_int(0.0f);
          int c = 1;
          while (sp > 0) {
            int32_t en;
            float ed;
            stack_pop2<kWin, B>(lds_n, lds_d, ovf_n, ovf_d, sp, nl, en, ed);
            st[2 + 2 * c] = en;
            st[3 + 2 * c] = __float_as_int(ed);
            ++c;
          }
          st[0] = c;
          st[1] = K;
          int64_t *keys = reinterpret_cast<int64_t *>(st + 2 + 2 * kHeavyStateEntries);
#pragma unroll
          for (int j = 0; j < K; ++j) keys[j] = L.key[j];
        }
      }
      return;
    }
  }
  if (STATS) {
    stats[2 * qi] = visited;
    stats[2 * qi + 1] = reads;
    return;
  }
  knn_write<K>(L, info.kk, info.base, indices + info.out, dist + info.out);
}

// Pass 2: a workgroup of T threads per heavy query.  The unexplored nodes
// stand in one LDS stack for the workgroup; a step takes a node per thread off
// its top, and the children that still qualify go back on top.  So every
// thread has a node as long as the stack has enough, whatever the shape of the
// subtrees, and the stack grows as a depth-first walk's does.  Candidates
// before the shared bound gather in LDS as well.  Once kCoopSlack more than k
// stand there, each one's rank among them is counted: the k best stay, in
// order, and the k-th is the new bound -- that of all the primitives the
// workgroup has met.  The bound is a whole key, distance and index: by its
// distance alone, every primitive at the k-th distance would stand there again
// and again (1e6 equal points, 1000 queries: 25 ms that way, 10 this way).
// The lower child goes on top, so that indices which only their order in the
// tree separates come in ascending order, the best first.  At the end the same
// step leaves the row.
// What bounds it: the latency of a step (one node load and two barriers) for a
// single query; for many, the cache lines of their nodes, which neighbouring
// queries no longer share.
// (A breadth-first frontier split among 1024 threads, each walking its share
// depth-first with a list and a bound of its own, left 38 % of their time idle
// and took 42 of 105 us a query to grow.  1e7-point shell, k = 10, 38 000
// heavy queries of 1e7: 20.3 ms that way, 7.1 to 10.4 this way; 1e5 queries of
// k = 32 in all: 14.4 ms, now 3.6.)
//
// A step over `take` entries adds at most (A - 1) * take to the stack, so a
// take of (free - kCoopReserve) / A leaves the reserve free, and single ones,
// a depth-first walk, need no more than the reserve (60 levels of three
// siblings, or 120 of one; taller trees are refused).
constexpr int kCoopSlack = 32;
constexpr int kCoopRank = 128;  // candidates ranked at a time, more than any k
constexpr int kCoopReserve = 192;
constexpr int coop_stack(int A, int T) { return (A == 4 ? 14 : 16) * T; }
constexpr int coop_found(int A, int T) { return kMaxRegK + kCoopSlack + A * T; }
// Steps of a small workgroup after which a query goes on to one of
// kCoopLarge threads (from the root again, with the bound reached): the few
// heaviest would end alone.  256 to 2048 measured alike.
constexpr int64_t kCoopSteps = 512;
static_assert(kMaxRegK + kCoopSlack < kCoopRank, "a step's few are ranked at once");

// Order the candidates found so far and drop those beyond the k-th; `bound`
// becomes the k-th key if there are k (every candidate precedes the bound it
// was taken under, so it only ever falls).  More than kCoopRank
// are thinned first, by the k-th of the first kCoopRank.  Called by the whole
// workgroup, after a barrier that makes the candidates visible.
template <int A, int T>
__device__ __forceinline__ void coop_rank(int64_t *cand, uint32_t *found, int64_t *bound,
                                          int64_t *pivot, int k) {
  constexpr int kPer = (coop_found(A, T) + T - 1) / T;
  constexpr int kOne = (kCoopRank + T - 1) / T;
  const int tid = threadIdx.x;
  while (true) {
    const int n = (int)*found, some = min(n, kCoopRank);
    int64_t key[kOne];
    int rank[kOne];
#pragma unroll
    for (int r = 0; r < kOne; ++r) {
      const bool in = r * T + tid < some;
      key[r] = in ? cand[r * T + tid] : 0;
      rank[r] = in ? 0 : kCoopRank;
    }
    if (tid < some) {
#pragma unroll 4
      for (int e = 0; e < some; ++e) {
        const int64_t x = cand[e];
#pragma unroll
        for (int r = 0; r < kOne; ++r) rank[r] += x < key[r] ? 1 : 0;
      }
    }
    if (n <= kCoopRank) {
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kOne; ++r) {
        if (rank[r] < k) cand[rank[r]] = key[r];  // (keys differ: one entry per primitive)
        if (rank[r] == k - 1) *bound = key[r];
      }
      if (tid == 0) *found = (uint32_t)min(n, k);
      __syncthreads();
      return;
    }
    int64_t own[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      const int i = r * T + tid;
      own[r] = i < n ? cand[i] : INT64_MAX;
    }
#pragma unroll
    for (int r = 0; r < kOne; ++r)
      if (rank[r] == k - 1) *pivot = key[r];
    __syncthreads();
    if (tid == 0) *found = 0;
    const int64_t most = *pivot;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPer; ++r)
      if (own[r] <= most) cand[atomicAdd(found, 1u)] = own[r];
    __syncthreads();
  }
}

template <int KIND, int FMT, class Map, int T>
__global__ __launch_bounds__(T) void k_nearest_coop(
    TreeArgs t, Map map, const float *__restrict__ pts, int32_t *__restrict__ indices,
    float *__restrict__ dist, HeavyList heavy,
    HeavyList huge) {
  constexpr int A = FMT == ABX_NODES_Q16W ? 4 : 2;  // children of a node
  constexpr int kCap = coop_stack(A, T);
  static_assert(kHeavyStateEntries + kCoopReserve + A * T <= kCap, "a saved walk fits");
  __shared__ int32_t s_node[kCap];
  __shared__ float s_dist[kCap];
  __shared__ int64_t s_cand[coop_found(A, T)];
  __shared__ int64_t s_pivot, s_bound;
  __shared__ uint32_t s_add[3], s_found, s_h;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const uint32_t total = min(heavy.count[0], heavy.cap);
  // the first query by the workgroup's number (2048 empty workgroups that each
  // drew one took 17 us), the next ones as they come
  uint32_t h = blockIdx.x;
  if (h >= total) return;
  resolve_qframe(t);
  for (bool first = true;; first = false) {
    __syncthreads();  // the previous query's buffers are free again
    if (!first) {
      if (tid == 0) s_h = gridDim.x + atomicAdd(heavy.count + 1, 1u);
      __syncthreads();
      h = s_h;
      if (h >= total) break;
    }
    const int32_t qi = heavy.q[h];
    const QInfo info = map.info(qi, t);
    const int k = info.kk;
    const KnnQuery q{pts[3 * (int64_t)qi], pts[3 * (int64_t)qi + 1], pts[3 * (int64_t)qi + 2]};
    // start from the walk the lane saved (its unexplored subtrees, and its
    // candidates), else from the root
    int size = 1;
    const int32_t *st =
        heavy.state && h < heavy.state_cap ? heavy.state + (int64_t)h * kHeavyStateWords : nullptr;
    int c = st ? min(st[0], kHeavyStateEntries) : -1;
    {
      // every saved node must be an internal node, else restart from the root
      bool bad = false;
      for (int e = tid; e < c; e += T) {
        const int32_t nd = st[2 + 2 * e];
        bad |= nd < 0 || nd >= t.nint;
      }
      if (__syncthreads_or(bad)) c = -1;
    }
    if (tid == 0) {
      s_bound = knn_key(heavy.bound[h], INT32_MAX);  // (no primitive's index)
      s_add[0] = 0;
      s_found = 0;
    }
    __syncthreads();
    if (c >= 1) {
      for (int e = tid; e < c; e += T) {
        s_node[e] = st[2 + 2 * e];
        s_dist[e] = __int_as_float(st[3 + 2 * e]);
      }
      size = c;
      const int64_t *keys = reinterpret_cast<const int64_t *>(st + 2 + 2 * kHeavyStateEntries);
      if (tid < st[1] && keys[tid] >= 0 && keys[tid] != kKeyEmpty)
        s_cand[atomicAdd(&s_found, 1u)] = keys[tid];
    } else if (tid == 0) {
      s_node[0] = info.root;
      s_dist[0] = 0.0f;
    }
    __syncthreads();

    // (without a list to hand on to, the bound on the steps only guarantees the end)
    const int64_t most = huge.q ? kCoopSteps : 4 * t.n + 64;
    int turn = 0, after = 1;  // this step's counter and the next one's, of three
    for (int64_t step = 0; size > 0 && step < most; ++step) {
      const int room = kCap - size;
      const int take = min(size, min(T, max(1, (room - kCoopReserve) / A)));
      const int base = size - take;
      bool ek[A];
      int32_t rk[A];
      float dk[A];
#pragma unroll
      for (int j = 0; j < A; ++j) {
        ek[j] = false;
        rk[j] = 0;
        dk[j] = 0.0f;
      }
      const int64_t kth = s_bound;
      const float bnd = key_dist(kth);
      if (tid < take && s_dist[base + tid] <= bnd) {
        const int32_t node = s_node[base + tid];
        if constexpr (A == 4) {
          Kids4 c4;
          load_kids4<KIND>(t, node, c4);
#pragma unroll
          for (int j = 0; j < A; ++j) {
            rk[j] = c4.ref[j];
            dk[j] = rk[j] == kEmptyRef ? INFINITY
                                       : box_dist2(c4.b[j][0], c4.b[j][1], c4.b[j][2], c4.b[j][3],
                                                   c4.b[j][4], c4.b[j][5], q.x, q.y, q.z);
          }
        } else {
          Kids c2;
          load_kids<KIND, FMT>(t, node, c2);
          rk[0] = c2.lref;
          rk[1] = c2.rref;
          dk[0] = box_dist2(c2.l[0], c2.l[1], c2.l[2], c2.l[3], c2.l[4], c2.l[5], q.x, q.y, q.z);
          dk[1] = box_dist2(c2.r[0], c2.r[1], c2.r[2], c2.r[3], c2.r[4], c2.r[5], q.x, q.y, q.z);
        }
#pragma unroll
        for (int j = 0; j < A; ++j) {
          ek[j] = rk[j] >= 0 && dk[j] <= bnd;
          if (rk[j] < 0 && rk[j] != kEmptyRef && dk[j] <= bnd) {
            float d = dk[j];
            if (!exact_leaf_slots<KIND, FMT>()) {
              float b[6];
              load_leaf_box(t, ~rk[j], b);
              d = box_dist2(b[0], b[1], b[2], b[3], b[4], b[5], q.x, q.y, q.z);
            }
            // (a NaN distance follows every bound)
            const int64_t key = knn_key(d, ~rk[j]);
            if (key < kth) s_cand[atomicAdd(&s_found, 1u)] = key;
          }
        }
      }
      // the counter of the next step: last read two barriers ago
      if (tid == 0) s_add[after] = 0;
      __syncthreads();  // the entries taken have been read, the candidates written
      const int found = (int)s_found;
      // wave-level compaction, one LDS reservation per wave; a lane's children
      // follow the lower lanes' ones, the first child last
      int cnt = 0, at = base;
#pragma unroll
      for (int j = 0; j < A; ++j) {
        const uint64_t bk = __ballot(ek[j]);
        cnt += __popcll(bk);
        at += __popcll(bk & lt);
      }
      uint32_t o = 0;
      if (lane == 0 && cnt > 0) o = atomicAdd(&s_add[turn], (uint32_t)cnt);
      at += (int)__shfl(o, 0, kWave);
#pragma unroll
      for (int j = A - 1; j >= 0; --j) {
        if (ek[j]) {
          s_node[at] = rk[j];
          s_dist[at] = dk[j];
          ++at;
        }
      }
      __syncthreads();
      size = base + (int)s_add[turn];
      turn = after;
      after = after == 2 ? 0 : after + 1;
      if (found > k + kCoopSlack) coop_rank<A, T>(s_cand, &s_found, &s_bound, &s_pivot, k);
    }

    coop_rank<A, T>(s_cand, &s_found, &s_bound, &s_pivot, k);
    if (size > 0 && huge.q) {
      if (tid == 0) {
        const uint32_t e = atomicAdd(huge.count, 1u);
        huge.q[e] = qi;
        huge.bound[e] = key_dist(s_bound);
      }
      continue;
    }
    if (tid < k) {
      const int64_t key = tid < (int)s_found ? s_cand[tid] : kKeyEmpty;
      indices[info.out + tid] = key_index(key) - info.base;
      dist[info.out + tid] = sqrtf(key_dist(key));
    }
  }
}

// Threads a query: as many as one CU holds while there is a CU for each query
// (1e7-point shell, 100 queries, k = 10: 117 us against 142 with 128), fewer
// for more queries, which fill the GPU with less of the barriers between (4000
// queries: 247 us with 256, 508 with 1024; 1e5 of k = 32: 3.4 ms with 128,
// 4.5 with 256, 4.0 with 64).
constexpr int kCoopLarge = 1024;
constexpr int kCoopMiddle = 256;
constexpr int kCoopSmall = 128;

int device_cus();

// The heavy queries of a batch of m (the grids hold as many workgroups as fit
// a CU at once: about 150 B of LDS a thread).
template <int KIND, int FMT, class Map>
abx_status launch_coop(const char *name, const TreeArgs &t, const Map &map, const float *pts, int64_t m,
                       int32_t *idx, float *dist, const HeavyList &heavy, const HeavyList &huge,
                       hipStream_t s) {
  const int cus = device_cus();
  if (m <= cus)
    return launch(name, s, [&] {
      k_nearest_coop<KIND, FMT, Map, kCoopLarge>
          <<<(unsigned)m, kCoopLarge, 0, s>>>(t, map, pts, idx, dist, heavy, HeavyList{});
    });
  return launch(name, s, [&] {  // (one timed launch: the pair)
    if (m <= 16 * (int64_t)cus)
      k_nearest_coop<KIND, FMT, Map, kCoopMiddle>
          <<<(unsigned)(cus * 4), kCoopMiddle, 0, s>>>(t, map, pts, idx, dist, heavy, huge);
    else
      k_nearest_coop<KIND, FMT, Map, kCoopSmall>
          <<<(unsigned)(cus * 8), kCoopSmall, 0, s>>>(t, map, pts, idx, dist, heavy, huge);
    k_nearest_coop<KIND, FMT, Map, kCoopLarge>
        <<<(unsigned)cus, kCoopLarge, 0, s>>>(t, map, pts, idx, dist, huge, HeavyList{});
  });
}

}  // namespace abx
