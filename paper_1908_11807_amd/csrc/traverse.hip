// Tree traversal kernels (ArborX paper, section 2.2).
//
// Batched mode: one lane per query, queries in Morton order so that the 64
// lanes of a wavefront walk nearly the same nodes (section 2.2 "Query
// ordering"); the blockIdx -> query-tile map keeps consecutive tiles on one
// XCD so that they share that XCD's L2.
//
// Spatial (section 2.2 "Traversal for spatial queries"): iterative, with a
// stack of deferred nodes.  A visited node holds both children's boxes; each
// child passing the predicate is emitted (leaf) or descended into (internal,
// the second one deferred on the stack).  Count pass and fill pass (2P).
//
// Nearest (section 2.2 "Traversal for nearest queries"): the same stack walk
// where one child is visited first and the other deferred with its box
// distance (the paper puts the nearer box first; here the child whose box
// centre is nearer goes first, which fills the list sooner); a node is
// pruned when its box is strictly farther than the
// current k-th candidate, which is how the walk stops once the remaining
// candidates cannot improve the result.  The k best candidates are kept
// sorted in registers by (squared distance, index).
//
// Stack: the top entries of each lane live in a circular LDS window (column
// per lane, so a wavefront's pushes hit distinct banks); deeper entries go to
// the lane's private memory.  Trees deeper than kMaxDepth are refused on the
// host.
#include <algorithm>

#include "traverse_common.h"

namespace abx {

// ------------------------------------------------------------------ spatial
template <int PRED>
struct SpatialQuery {
  float a[3], b[3];  // WITHIN: a = point, b[0] = r^2 ; INTERSECTS: a = lo, b = hi
  __device__ __forceinline__ bool test(const float *x) const {
    if (PRED == ABX_PRED_WITHIN)
      return box_dist2(x[0], x[1], x[2], x[3], x[4], x[5], a[0], a[1], a[2]) <= b[0];
    return box_overlap(x[0], x[1], x[2], x[3], x[4], x[5], a[0], a[1], a[2], b[0], b[1], b[2]);
  }
};

// One wavefront per workgroup, as in the nearest pass (keeping pass over 1e6
// cube points 386 -> 376 us, over 1e7 shell points 533 -> 503 us, against four).
constexpr int kSpatialBlock = kWave;

template <int KIND, int PRED, int FMT, int MODE>
__global__ __launch_bounds__(kSpatialBlock) void k_spatial(TreeArgs t, QueryArgs qa,
                                                        int32_t *__restrict__ out_counts,
                                                        const int32_t *__restrict__ offsets,
                                                        int32_t *__restrict__ indices) {
  // passes that hold hits: half the window, the other half holds them
  constexpr bool kHolds = MODE == MODE_KEEP || MODE == MODE_STORE;
  constexpr int kWin = kHolds ? kLdsDepthSpatial / 2 : kLdsDepthSpatial;
  __shared__ int32_t s_stack[kWin * kSpatialBlock];
  __shared__ int32_t s_held[kHolds ? 8 * kSpatialBlock : 1];
  // keeping pass: chunks that the wavefront's rows have asked for, its blocks
  __shared__ int32_t s_taken, s_block[MODE == MODE_KEEP ? kKeptBlocks : 1];
  static_assert(kSpatialBlock == kWave, "a workgroup's chunks are one wavefront's");
  static_assert(kKeptChunks < 4 && kWave * kKeptChunks < 256, "three bytes number a row's chunks");
  if (MODE == MODE_KEEP) {
    s_taken = 0;
    if (threadIdx.x < kKeptBlocks) s_block[threadIdx.x] = 0;
  }
  const int64_t tq = xcd_tile(blockIdx.x, gridDim.x) * kSpatialBlock + threadIdx.x;
  if (tq >= qa.m) return;
  // the fill pass of the one-pass scheme runs only after an overflow, and
  // only when the caller's index buffer holds every hit
  if (MODE == MODE_FILL && qa.flag && (qa.flag[0] == 0 || *qa.total > qa.capacity)) return;
  // after a keeping pass only the rows that it did not keep whole are filled
  if (MODE == MODE_FILL && qa.kept.counts && qa.kept.whole(tq)) return;
  const int64_t qi = qa.order ? qa.order[tq] : tq;
  SpatialQuery<PRED> q;
  if (PRED == ABX_PRED_WITHIN) {
    const float *p = qa.data + 3 * qi;
    q.a[0] = p[0]; q.a[1] = p[1]; q.a[2] = p[2];
    const float r = qa.radii ? qa.radii[qi] : qa.radius;
    q.b[0] = r >= 0.0f ? r * r : -1.0f;
    q.b[1] = q.b[2] = 0.0f;
  } else {
    const float *p = qa.data + 6 * qi;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      q.a[a] = p[a];
      q.b[a] = p[3 + a];
    }
  }
  int32_t *out = MODE == MODE_FILL    ? indices + offsets[qi]
                 : MODE == MODE_STORE ? qa.buf + tq * qa.bufsize
                                      : nullptr;
  const int32_t row_len = MODE == MODE_FILL    ? offsets[qi + 1] - offsets[qi]
                          : MODE == MODE_STORE ? qa.bufsize
                                               : 0;
  int32_t cnt = 0, visited = 0, leaf_reads = 0;

  // Hits collect in LDS and leave eight at a time.  (A store per hit would
  // stand between a visit and the wait for its node, as loads and stores
  // retire in order: 1e6 queries of ten hits on 1e6 points, rows kept, 446 us
  // that way and 386 this way; counting alone takes 346, and the second walk
  // that the kept rows make unnecessary took 404.  The storing pass of the
  // one-pass search, 32 slots a row: 294 -> 270 us.)
  ABX_LDS int32_t *held = (ABX_LDS int32_t *)(s_held) + threadIdx.x;
  bool keeps = MODE == MODE_KEEP;  // the row so far is kept whole
  int32_t ext = 0;                 // its chunks
  int32_t *room = MODE == MODE_KEEP ? qa.kept.buf + tq * kKeptRow : nullptr;
  auto load_block = [&](int32_t b) {
    return __hip_atomic_load(&s_block[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto keep = [&](int32_t at) {  // hits at .. at + 7 of the row
    const int32_t c = at / kKeptRow - 1, in = at % kKeptRow;
    if (in == 0 && at > 0) {
      keeps = c < kKeptChunks;
      if (!keeps) return;
      // the wavefront's chunks, numbered as its lanes ask for them; who opens a
      // block of them takes it from the pool, unless that had run out before
      const int32_t e = atomicAdd(&s_taken, 1), b = e / kKeptBlock;
      if (e % kKeptBlock == 0) {
        int32_t block = -1;
        if (b == 0 || load_block(b - 1) >= 0) {
          const int32_t wave = (int32_t)(tq / kWave), part = wave % qa.kept.parts;
          const uint32_t f = atomicAdd(qa.kept.taken + part * kKeptCounter, 1u);
          if (f < (uint32_t)qa.kept.part_blocks) {
            block = part * qa.kept.part_blocks + (int32_t)f;
            qa.kept.blocks[(int64_t)wave * kKeptBlocks + b] = block;
          }
        }
        __hip_atomic_store(&s_block[b], block, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      // (a wavefront runs as one: the block is stored before any lane reads it)
      __builtin_amdgcn_wave_barrier();
      const int32_t block = load_block(b);
      keeps = block >= 0;
      if (!keeps) return;
      ext |= e << (8 * c);
      room = qa.kept.chunk(block, e);
    }
    int4 *t4 = reinterpret_cast<int4 *>(room + in);
    t4[0] = make_int4(held[0], held[kSpatialBlock], held[2 * kSpatialBlock], held[3 * kSpatialBlock]);
    t4[1] = make_int4(held[4 * kSpatialBlock], held[5 * kSpatialBlock], held[6 * kSpatialBlock], held[7 * kSpatialBlock]);
  };

  auto put = [&](int32_t at) {  // the same hits, in their place in `out`
    // (rows start anywhere: 16 B stores of 4 B alignment)
    typedef int32_t int4u __attribute__((ext_vector_type(4), aligned(4)));
    if (cnt >= at + 8 && at + 8 <= row_len) {
      int4u *to = reinterpret_cast<int4u *>(out + at);
      to[0] = int4u{held[0], held[kSpatialBlock], held[2 * kSpatialBlock], held[3 * kSpatialBlock]};
      to[1] = int4u{held[4 * kSpatialBlock], held[5 * kSpatialBlock], held[6 * kSpatialBlock], held[7 * kSpatialBlock]};
    } else {
      const int32_t end = cnt < row_len ? cnt : row_len;
      for (int j = 0; at + j < end; ++j) out[at + j] = held[j * kSpatialBlock];
    }
  };

  // a leaf child (primitive idx) whose node-stored box passed: confirm where
  // the slot is quantised, and emit
  auto leaf = [&](int32_t idx) {
    if (!exact_leaf_slots<KIND, FMT>()) {
      float b[6];
      load_leaf_box(t, idx, b);
      if (MODE == MODE_STATS) ++leaf_reads;
      if (!q.test(b)) return;
    }
    if (MODE == MODE_FILL && cnt < row_len) out[cnt] = idx;
    if (MODE == MODE_STORE || keeps) held[(cnt & 7) * kSpatialBlock] = idx;
    ++cnt;
    if (kHolds && (cnt & 7) == 0) {
      if (MODE == MODE_STORE) put(cnt - 8);
      else if (keeps) keep(cnt - 8);
    }
  };

  if (t.n == 1) {
    // the scene box of a one-primitive tree is that primitive's box
    if (q.test(t.scene)) leaf(0);
  } else {
    int32_t ovf[kMaxDepth];
    ABX_LDS int32_t *lds = (ABX_LDS int32_t *)(s_stack) + threadIdx.x;
    int sp = 0, nl = 0;
    int32_t node = t.root;
    // a tree has n-1 internal nodes, each visited at most once: the bound
    // only guarantees termination
    for (int64_t it = 0; it < t.n; ++it) {
      if constexpr (FMT == ABX_NODES_Q16W) {
        // 4-wide node: emit the leaf children that pass, descend into the
        // first internal one, defer the others
        Kids4 k;
        load_kids4<KIND>(t, node, k);
        if (MODE == MODE_STATS) ++visited;
        int32_t next = -1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (k.ref[j] == kEmptyRef || !q.test(k.b[j])) continue;
          if (k.ref[j] < 0) leaf(~k.ref[j]);
          else if (next < 0) next = k.ref[j];
          else if (sp < kMaxDepth) stack_push<int32_t, kWin, kSpatialBlock>(lds, ovf, sp, nl, k.ref[j]);
        }
        if (next >= 0) {
          node = next;
        } else {
          if (sp == 0) break;
          node = stack_pop<int32_t, kWin, kSpatialBlock>(lds, ovf, sp, nl);
        }
        continue;
      }
      Kids k;
      load_kids<KIND, FMT>(t, node, k);
      if (MODE == MODE_STATS) ++visited;
      const bool hl = q.test(k.l), hr = q.test(k.r);
      const bool ll = k.lref < 0, lr = k.rref < 0;
      if (hl && ll) leaf(~k.lref);
      if (hr && lr) leaf(~k.rref);
      const bool gl = hl && !ll, gr = hr && !lr;
      if (gl) {
        if (gr && sp < kMaxDepth)
          stack_push<int32_t, kWin, kSpatialBlock>(lds, ovf, sp, nl, k.rref);
        node = k.lref;
      } else if (gr) {
        node = k.rref;
      } else {
        if (sp == 0) break;
        node = stack_pop<int32_t, kWin, kSpatialBlock>(lds, ovf, sp, nl);
      }
    }
  }
  if (MODE == MODE_COUNT || MODE == MODE_STORE || MODE == MODE_KEEP) out_counts[qi] = cnt;
  if (MODE == MODE_STORE && (cnt & 7)) put(cnt & ~7);
  if (MODE == MODE_KEEP) {
    if (keeps && (cnt & 7)) keep(cnt & ~7);
    qa.kept.counts[tq] = cnt;
    if (cnt > kKeptRow) {
      qa.kept.ext[tq] = keeps ? ext : -1;
      if (!keeps && qa.kept.words[1] == 0) qa.kept.words[1] = 1;
    }
  }
  if (MODE == MODE_STORE && cnt > qa.bufsize) atomicOr(qa.flag, 1u);
  if (MODE == MODE_STATS) {
    out_counts[2 * qi] = visited;
    out_counts[2 * qi + 1] = leaf_reads;
  }
}

// ------------------------------------------------------------------ nearest
// One wavefront per workgroup: a walk's length varies, and a workgroup of four
// held its LDS until its longest walk ended; a small batch also spreads over
// four times as many CUs (1000 queries, k = 8, on 1e7 points: 209 -> 177 us a
// call; 1e6 queries on 1e6 points 801 -> 776; workgroups of eight and twelve
// wavefronts 10 % slower than four on the 1e7 shell).
constexpr int kNearestBlock = kWave;

// Pass 1 over one tree: one lane per query, queries in Morton order.
template <int KIND, int FMT, int K, bool STATS>
__global__ __launch_bounds__(kNearestBlock)
__attribute__((amdgpu_waves_per_eu(nearest_waves_per_eu(K, FMT)))) void k_nearest(TreeArgs t, PlainMap map,
                                                        const float *__restrict__ pts, int64_t m,
                                                        const int32_t *__restrict__ order,
                                                        int32_t *__restrict__ indices,
                                                        float *__restrict__ dist,
                                                        int32_t *__restrict__ stats, int64_t budget,
                                                        HeavyList heavy) {
  constexpr int W = lane_window(nearest_waves_per_eu(K, FMT));
  __shared__ int32_t s_node[W * kNearestBlock];
  __shared__ uint16_t s_dist[W * kNearestBlock];
  const int64_t tq = xcd_tile(blockIdx.x, gridDim.x) * kNearestBlock + threadIdx.x;
  if (tq >= m) return;
  const int64_t qi = order ? order[tq] : tq;
  nearest_lane<KIND, FMT, K, STATS, kNearestBlock, W>(
      t, map, pts, qi, (ABX_LDS int32_t *)(s_node) + threadIdx.x,
      (ABX_LDS uint16_t *)(s_dist) + threadIdx.x, indices, dist, stats, budget, heavy);
}

// ------------------------------------------------------------ large k
// k = 65..128 (register lists serve k <= 64: 64 keys take 128 registers, the
// most that leaves two wavefronts per SIMD): each lane keeps its candidates
// in an LDS max-heap (root = the
// current k-th candidate; the heap is the paper's bounded priority list,
// section 2.2), one wavefront per workgroup, entry e of lane l at e * 64 + l
// so that a wavefront's accesses fall in distinct banks.  The walk is the
// one of pass 1 (child with the nearer box centre first, strict pruning by
// the root once the heap is full) with no visit budget.  At the end a heap
// sort leaves the row ascending in place.
constexpr int kHeapLanes = kWave;

__device__ __forceinline__ void heap_push(ABX_LDS int64_t *h, int &size, int64_t x) {
  int i = size++;
  while (i > 0) {
    const int p = (i - 1) >> 1;
    const int64_t vp = h[p * kHeapLanes];
    if (vp >= x) break;
    h[i * kHeapLanes] = vp;
    i = p;
  }
  h[i * kHeapLanes] = x;
}

// x replaces the root of heap [0, size) and sinks to its place
__device__ __forceinline__ void heap_sink(ABX_LDS int64_t *h, int size, int64_t x) {
  int i = 0;
  for (;;) {
    int c = 2 * i + 1;
    if (c >= size) break;
    int64_t vc = h[c * kHeapLanes];
    if (c + 1 < size) {
      const int64_t v2 = h[(c + 1) * kHeapLanes];
      if (v2 > vc) {
        ++c;
        vc = v2;
      }
    }
    if (vc <= x) break;
    h[i * kHeapLanes] = vc;
    i = c;
  }
  h[i * kHeapLanes] = x;
}

// The heap takes 8k bytes of LDS per lane (dynamic, sized to k), which is
// what bounds residency: registers are capped to match (4 waves per SIMD).
template <int KIND, int FMT, bool STATS>
__global__ __launch_bounds__(kHeapLanes) __attribute__((amdgpu_waves_per_eu(4))) void k_nearest_heap(TreeArgs t,
                                                             const float *__restrict__ pts,
                                                             int64_t m,
                                                             const int32_t *__restrict__ order,
                                                             int k, int32_t *__restrict__ indices,
                                                             float *__restrict__ dist,
                                                             int32_t *__restrict__ stats) {
  extern __shared__ int64_t s_heap[];  // k keys per lane, lane-interleaved
  __shared__ int32_t s_node[kLdsDepthNearest * kHeapLanes];
  __shared__ float s_dist[kLdsDepthNearest * kHeapLanes];
  const int64_t tq = xcd_tile(blockIdx.x, gridDim.x) * kHeapLanes + threadIdx.x;
  if (tq >= m) return;
  const int64_t qi = order ? order[tq] : tq;
  const KnnQuery q{pts[3 * qi], pts[3 * qi + 1], pts[3 * qi + 2]};
  ABX_LDS int64_t *h = (ABX_LDS int64_t *)(s_heap) + threadIdx.x;
  ABX_LDS int32_t *lds_n = (ABX_LDS int32_t *)(s_node) + threadIdx.x;
  ABX_LDS float *lds_d = (ABX_LDS float *)(s_dist) + threadIdx.x;
  int size = 0;
  int32_t visited = 0, reads = 0;
  auto kth = [&]() { return size < k ? INFINITY : key_dist(h[0]); };
  auto offer = [&](int64_t x) {
    if (size < k) heap_push(h, size, x);
    else if (x < h[0]) heap_sink(h, k, x);
  };
  // a leaf child whose node-stored box is at squared distance dbox
  auto leaf = [&](int32_t idx, float dbox) {
    if (!(dbox <= kth())) return;
    if (exact_leaf_slots<KIND, FMT>()) {
      offer(knn_key(dbox, idx));
    } else {
      ++reads;
      float b[6];
      load_leaf_box(t, idx, b);
      const float d = box_dist2(b[0], b[1], b[2], b[3], b[4], b[5], q.x, q.y, q.z);
      if (d <= kth()) offer(knn_key(d, idx));
    }
  };
  if (t.n == 1) {
    const float *b = t.scene;
    leaf(0, box_dist2(b[0], b[1], b[2], b[3], b[4], b[5], q.x, q.y, q.z));
  } else {
    int32_t ovf_n[kMaxDepth];
    float ovf_d[kMaxDepth];
    int sp = 0, nl = 0;
    int32_t node = t.root;
    for (int64_t it = 0; it < 2 * t.n; ++it) {
      if (STATS) ++visited;
      if constexpr (FMT == ABX_NODES_Q16W) {
        // 4-wide node, as knn_visit_w: leaves offered, the qualifying
        // internal children visited nearest box centre first
        Kids4 c;
        load_kids4<KIND>(t, node, c);
        float d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          d[j] = c.ref[j] == kEmptyRef ? INFINITY
                                       : box_dist2(c.b[j][0], c.b[j][1], c.b[j][2], c.b[j][3],
                                                   c.b[j][4], c.b[j][5], q.x, q.y, q.z);
          if (c.ref[j] < 0 && c.ref[j] != kEmptyRef) leaf(~c.ref[j], d[j]);
        }
        const float thr = kth();
        float key[4];
        int32_t r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool g = c.ref[j] >= 0 && d[j] <= thr;
          float cc = 0.0f;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const float qa = a == 0 ? q.x : (a == 1 ? q.y : q.z);
            const float mm = (c.b[j][a] - qa) - (qa - c.b[j][3 + a]);
            cc = __fmaf_rn(mm, mm, cc);
          }
          key[j] = g ? cc : INFINITY;
          r[j] = g ? c.ref[j] : -1;
        }
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
          if (r[j] >= 0 && sp < kMaxDepth)
            stack_push2<kLdsDepthNearest, kHeapLanes>(lds_n, lds_d, ovf_n, ovf_d, sp, nl, r[j], d[j]);
        node = r[0];
        if (node < 0) node = knn_pop<kHeapLanes>(kth(), lds_n, lds_d, ovf_n, ovf_d, sp, nl);
        if (node < 0) break;
        continue;
      }
      Kids c;
      load_kids<KIND, FMT>(t, node, c);
      const float dl = box_dist2(c.l[0], c.l[1], c.l[2], c.l[3], c.l[4], c.l[5], q.x, q.y, q.z);
      const float dr = box_dist2(c.r[0], c.r[1], c.r[2], c.r[3], c.r[4], c.r[5], q.x, q.y, q.z);
      const bool ll = c.lref < 0, lr = c.rref < 0;
      if (ll) leaf(~c.lref, dl);
      if (lr) leaf(~c.rref, dr);
      const float thr = kth();
      const bool gl = !ll && dl <= thr, gr = !lr && dr <= thr;
      node = -1;
      if (gl && gr) {
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
          stack_push2<kLdsDepthNearest, kHeapLanes>(lds_n, lds_d, ovf_n, ovf_d, sp, nl,
                                                    left_first ? c.rref : c.lref,
                                                    left_first ? dr : dl);
        node = left_first ? c.lref : c.rref;
      } else if (gl) {
        node = c.lref;
      } else if (gr) {
        node = c.rref;
      }
      if (node < 0) node = knn_pop<kHeapLanes>(kth(), lds_n, lds_d, ovf_n, ovf_d, sp, nl);
      if (node < 0) break;
    }
  }
  if (STATS) {
    stats[2 * qi] = visited;
    stats[2 * qi + 1] = reads;
    return;
  }
  // heap sort: the largest goes to the back, the rest sinks again
  for (int e = size - 1; e > 0; --e) {
    const int64_t top = h[0];
    const int64_t last = h[e * kHeapLanes];
    h[e * kHeapLanes] = top;
    heap_sink(h, e, last);
  }
  int32_t *oi = indices + qi * k;
  float *od = dist + qi * k;
  for (int j = 0; j < size; ++j) {
    const int64_t x = h[j * kHeapLanes];
    oi[j] = key_index(x);
    od[j] = sqrtf(key_dist(x));
  }
}


// ------------------------------------------------------------ query codes
// 30-bit Morton code of each query's centroid against the tree's scene box
// (clamped), for the query ordering of section 2.2.
__device__ __forceinline__ uint32_t spread10q(uint32_t x) {
  x &= 0x3ffu;
  x = (x | (x << 16)) & 0x030000ffu;
  x = (x | (x << 8)) & 0x0300f00fu;
  x = (x | (x << 4)) & 0x030c30c3u;
  x = (x | (x << 2)) & 0x09249249u;
  return x;
}

// `words`: the spatial search's state words, set to (mark, 0); `taken`: the
// counters of its kept rows' pool (null: it keeps none).
template <int W>
__global__ __launch_bounds__(kTravBlock) void k_query_codes(const float *__restrict__ q, int64_t m,
                                                            TreeArgs t, uint32_t *__restrict__ codes,
                                                            uint32_t *__restrict__ words,
                                                            uint32_t mark, uint32_t *__restrict__ taken) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (taken && i < kKeptParts) taken[i * kKeptCounter] = 0;
  if (i == 0) {
    words[0] = mark;
    words[1] = 0;
  }
  if (i >= m) return;
  uint32_t c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float x = W == 3 ? q[3 * i + a] : 0.5f * (q[6 * i + a] + q[6 * i + 3 + a]);
    const float lo = t.scene[a], ext = t.scene[3 + a] - lo;
    const float inv = ext > 0.0f ? 1.0f / ext : 0.0f;
    float u = (x - lo) * inv;
    u = u > 0.0f ? u : 0.0f;
    u = u < 1.0f ? u : 1.0f;
    const uint32_t v = (uint32_t)(u * 1024.0f);
    c[a] = v > 1023u ? 1023u : v;
  }
  codes[i] = (spread10q(c[0]) << 2) | (spread10q(c[1]) << 1) | spread10q(c[2]);
}

// ------------------------------------------------------------ host launchers
TreeArgs tree_args(const abx_bvh *b) {
  TreeArgs t;
  t.nodes = b->nodes();
  t.leaves = b->leaves();
  t.n = b->n;
  t.root = b->root;
  for (int a = 0; a < 6; ++a) t.scene[a] = b->scene[a];
  for (int a = 0; a < 3; ++a) {
    t.qo[a] = b->q_origin[a];
    t.qs[a] = b->q_scale[a];
  }
  t.scene_dev = b->hdr()->scene;
  t.qframe = nullptr;
  t.guard = nullptr;  // the build checked the header before making the handle
  t.nint = b->nint;
  return t;
}

abx_status launch_query_codes(const abx_bvh *b, const float *q, int64_t m, int width,
                              uint32_t *codes, hipStream_t s, uint32_t *words, uint32_t mark,
                              uint32_t *taken) {
  if (m == 0) return ABX_OK;
  const TreeArgs t = tree_args(b);
  const unsigned g = grid_for(m, kTravBlock);
  if (width == 3)
    return launch("query_codes", s, [&] { k_query_codes<3><<<g, kTravBlock, 0, s>>>(q, m, t, codes, words, mark, taken); });
  return launch("query_codes", s, [&] { k_query_codes<6><<<g, kTravBlock, 0, s>>>(q, m, t, codes, words, mark, taken); });
}

template <int KIND, int PRED, int FMT>
abx_status spatial_fmt(const abx_bvh *b, const QueryArgs &qa, int mode, int32_t *counts,
                       const int32_t *offsets, int32_t *indices, hipStream_t s) {
  const TreeArgs t = tree_args(b);
  const unsigned g = grid_for(qa.m, kSpatialBlock);
  const char *name = mode == MODE_COUNT  ? "spatial_count"
                     : mode == MODE_FILL  ? "spatial_fill"
                     : mode == MODE_STORE ? "spatial_store"
                     : mode == MODE_KEEP  ? "spatial_count"
                                          : "spatial_stats";
  return launch(name, s, [&] {
    if (mode == MODE_COUNT)
      k_spatial<KIND, PRED, FMT, MODE_COUNT><<<g, kSpatialBlock, 0, s>>>(t, qa, counts, offsets, indices);
    else if (mode == MODE_KEEP)
      k_spatial<KIND, PRED, FMT, MODE_KEEP><<<g, kSpatialBlock, 0, s>>>(t, qa, counts, offsets, indices);
    else if (mode == MODE_STORE)
      k_spatial<KIND, PRED, FMT, MODE_STORE><<<g, kSpatialBlock, 0, s>>>(t, qa, counts, offsets, indices);
    else if (mode == MODE_FILL)
      k_spatial<KIND, PRED, FMT, MODE_FILL><<<g, kSpatialBlock, 0, s>>>(t, qa, counts, offsets, indices);
    else
      k_spatial<KIND, PRED, FMT, MODE_STATS><<<g, kSpatialBlock, 0, s>>>(t, qa, counts, offsets, indices);
  });
}

template <int KIND, int PRED>
abx_status spatial_pred(const abx_bvh *b, const QueryArgs &qa, int mode, int32_t *counts,
                        const int32_t *offsets, int32_t *indices, hipStream_t s) {
  if (b->format == ABX_NODES_FP32)
    return spatial_fmt<KIND, PRED, ABX_NODES_FP32>(b, qa, mode, counts, offsets, indices, s);
  if (b->format == ABX_NODES_Q16W)
    return spatial_fmt<KIND, PRED, ABX_NODES_Q16W>(b, qa, mode, counts, offsets, indices, s);
  return spatial_fmt<KIND, PRED, ABX_NODES_Q16>(b, qa, mode, counts, offsets, indices, s);
}

abx_status launch_spatial(const abx_bvh *b, int pred, const float *data, int64_t m,
                          const float *radii, float radius, const int32_t *order, int mode,
                          int32_t *counts, const int32_t *offsets, int32_t *indices, hipStream_t s,
                          const OnePass *op, const KeptRows *kept) {
  if (m == 0) return ABX_OK;
  QueryArgs qa{};  // (no kept rows, no one-pass state)
  qa.data = data;
  qa.m = m;
  qa.radii = radii;
  qa.radius = radius;
  qa.order = order;
  if (op) {
    qa.buf = op->buf;
    qa.bufsize = op->bufsize;
    qa.flag = op->flag;
    qa.total = op->total;
    qa.capacity = op->capacity;
  }
  if (kept) qa.kept = *kept;
  if (b->kind == ABX_PRIM_POINTS) {
    if (pred == ABX_PRED_WITHIN)
      return spatial_pred<ABX_PRIM_POINTS, ABX_PRED_WITHIN>(b, qa, mode, counts, offsets, indices, s);
    return spatial_pred<ABX_PRIM_POINTS, ABX_PRED_INTERSECTS_BOX>(b, qa, mode, counts, offsets, indices, s);
  }
  if (pred == ABX_PRED_WITHIN)
    return spatial_pred<ABX_PRIM_BOXES, ABX_PRED_WITHIN>(b, qa, mode, counts, offsets, indices, s);
  return spatial_pred<ABX_PRIM_BOXES, ABX_PRED_INTERSECTS_BOX>(b, qa, mode, counts, offsets, indices, s);
}

// ------------------------------------------------------------ 1P compaction
// After a storing pass with no overflow: the row stored for sorted position
// tq (its first count[q] slots) goes to indices[offsets[q] ...].  A group of
// G lanes (8 or 16) copies one query's hits, G consecutive entries per step:
// reads and writes stay coalesced within the row, and the cost follows the
// results rather than the m * buffer_size slots (a buffer sized for the
// longest row is mostly empty when rows are uneven: hollow case, 2.7 hits
// per row against 259 slots).
__global__ __launch_bounds__(kTravBlock) void k_spatial_compact(const int32_t *__restrict__ buf,
                                                                int32_t bufsize, int64_t m,
                                                                int group_log2,
                                                                const int32_t *__restrict__ order,
                                                                const int32_t *__restrict__ counts,
                                                                const int32_t *__restrict__ offsets,
                                                                int32_t *__restrict__ indices,
                                                                const uint32_t *__restrict__ flag,
                                                                const int64_t *__restrict__ total,
                                                                int64_t capacity) {
  if (flag[0] != 0 || *total > capacity) return;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t tq = id >> group_log2;
  if (tq >= m) return;
  const int32_t g = 1 << group_log2, j0 = (int32_t)(id & (g - 1));
  const int64_t qi = order ? order[tq] : tq;
  const int32_t c = counts[qi];  // <= bufsize: no row overflowed
  const int32_t *row = buf + tq * (int64_t)bufsize;
  int32_t *out = indices + offsets[qi];
  for (int32_t j = j0; j < c; j += g) out[j] = row[j];
}

// ------------------------------------------------------------ kept rows
// The second pass of the two-pass scheme when the first one kept the rows
// (radius search, 1e6 queries of ten hits: 922 -> 600 us a call; box overlaps
// of 1e6 boxes, build included, 1490 -> 1150 us): each is copied to its place
// (those not kept whole are walked again).  Eight lanes a row read 16 B each,
// neighbouring rows one after another; the counts tell an empty row without touching its
// slots.  No more is written of a row than its offsets give it.
__global__ __launch_bounds__(kTravBlock) void k_rows_copy(KeptRows kept, int64_t m,
                                                          const int32_t *__restrict__ order,
                                                          const int32_t *__restrict__ offsets,
                                                          int32_t *__restrict__ indices) {
  constexpr int kLanes = kKeptRow / 4;
  const int64_t id = (int64_t)blockIdx.x * kTravBlock + threadIdx.x;
  const int64_t tq = id / kLanes;
  const int l = (int)(id & (kLanes - 1));
  if (tq >= m) return;
  const int32_t hits = kept.counts[tq];
  if (4 * l >= hits) return;
  int32_t ext = 0;
  if (hits > kKeptRow) {
    ext = kept.ext[tq];
    if (ext < 0) return;
  }
  const int64_t qi = order ? order[tq] : tq;
  const int32_t at = offsets[qi], c = min(hits, offsets[qi + 1] - at);
  if (4 * l >= c) return;
  int32_t *out = indices + at;
  const int4 *from = reinterpret_cast<const int4 *>(kept.buf + tq * kKeptRow);
  for (int32_t e = 4 * l;;) {
    const int4 v = from[l];
    out[e] = v.x;
    if (e + 1 < c) out[e + 1] = v.y;
    if (e + 2 < c) out[e + 2] = v.z;
    if (e + 3 < c) out[e + 3] = v.w;
    e += kKeptRow;
    if (e >= c) break;
    const int32_t n = ext & 255;
    from = reinterpret_cast<const int4 *>(
        kept.chunk(kept.blocks[tq / kWave * kKeptBlocks + n / kKeptBlock], n));
    ext >>= 8;
  }
}

abx_status launch_rows_copy(const KeptRows &kept, int64_t m, const int32_t *order,
                            const int32_t *offsets, int32_t *indices, hipStream_t s) {
  const unsigned g = grid_for(m * (kKeptRow / 4), kTravBlock);
  return launch("spatial_copy", s, [&] {
    k_rows_copy<<<g, kTravBlock, 0, s>>>(kept, m, order, offsets, indices);
  });
}

// info[0] = status, info[1] = traversals made
__global__ void k_spatial_1p_info(const uint32_t *__restrict__ flag, const int64_t *__restrict__ total,
                                  int64_t capacity, int64_t max_count, int32_t *__restrict__ info) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int64_t t = *total;
  const bool fits = t <= capacity;
  info[0] = t >= max_count ? ABX_ERR_OVERFLOW : (fits ? ABX_OK : ABX_ERR_CAPACITY);
  info[1] = flag[0] != 0 && fits ? 2 : 1;
}

abx_status launch_spatial_compact(const OnePass &op, int64_t m, const int32_t *order,
                                  const int32_t *counts, const int32_t *offsets, int32_t *indices,
                                  int32_t *info, int64_t max_count, hipStream_t s) {
  if (m > 0) {
    const int glog = op.bufsize <= 8 ? 3 : 4;  // 8 or 16 lanes per query
    const unsigned g = grid_for(m << glog, kTravBlock);
    ABX_TRY(launch("spatial_compact", s, [&] {
      k_spatial_compact<<<g, kTravBlock, 0, s>>>(op.buf, op.bufsize, m, glog, order, counts,
                                                 offsets, indices, op.flag, op.total, op.capacity);
    }));
  }
  return launch("spatial_1p_info", s, [&] {
    k_spatial_1p_info<<<1, 64, 0, s>>>(op.flag, op.total, op.capacity, max_count, info);
  });
}

struct NearestScratch {
  int32_t *heavy_q;
  float *heavy_bound;
  int32_t *huge_q;  // those the cooperative pass passes on to larger workgroups
  float *huge_bound;
  uint32_t *counters;  // [0] heavy count, [1] next heavy query, [3], [4] the huge ones'
  int64_t budget;
  int32_t *heavy_state;  // saved walks (kHeavyStateWords each), or null
  uint32_t state_cap;
};

int device_cus() {
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess)
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  return cus > 0 ? cus : 256;
}

// Queries of a batch that may leave their lanes: all of them, but on a tree of
// no more than m / 24 primitives one in 64, or as many as the cooperative pass
// answers at once.  Such a tree stands in the caches,
// and a lane's visit to it costs less than a workgroup's; what pays there is to
// take the few long walks out of their wavefronts (30 000 points on a shell,
// 1e6 queries, k = 10: 0.5 % handed over, 1.8 ms against 12.7 with none).
// Where they are many, all walks are long (equal points, where no node can be
// skipped; 1e5 queries of k = 1 on 300 points: 265 us in their lanes, 1380 all
// handed over, 290 this way; 1e6 on 10 000 points 27 ms, 52 and 26).
uint32_t heavy_cap(int64_t n, int64_t m) {
  return n <= m / 24 ? (uint32_t)std::max<int64_t>(m / 64, 8 * device_cus()) : UINT32_MAX;
}

template <int KIND, int FMT, int K>
abx_status nearest_k(const abx_bvh *b, const float *pts, int64_t m, const int32_t *order, int k,
                     int32_t *idx, float *dist, int32_t *stats, const NearestScratch &ns,
                     hipStream_t s) {
  const TreeArgs t = tree_args(b);
  const PlainMap map{k};
  const HeavyList heavy{ns.heavy_q, ns.heavy_bound, ns.counters,
                        saves_walk(K) ? ns.heavy_state : nullptr, ns.state_cap,
                        heavy_cap(b->n, m)};
  const unsigned g = grid_for(m, kNearestBlock);
  if (stats)
    return launch("nearest_stats", s, [&] {
      k_nearest<KIND, FMT, K, true><<<g, kNearestBlock, 0, s>>>(t, map, pts, m, order, idx, dist,
                                                             stats, INT64_MAX, heavy);
    });
  ABX_TRY(fill_u32(ns.counters, 0, 5, s));
  ABX_TRY(launch("nearest", s, [&] {
    k_nearest<KIND, FMT, K, false><<<g, kNearestBlock, 0, s>>>(t, map, pts, m, order, idx, dist,
                                                            stats, ns.budget, heavy);
  }));
  const HeavyList huge{ns.huge_q, ns.huge_bound, ns.counters + 3};
  return launch_coop<KIND, FMT>("nearest_coop", t, map, pts, m, idx, dist, heavy, huge, s);
}

template <int KIND, int FMT, bool STATS>
abx_status launch_heap(const TreeArgs &t, const float *pts, int64_t m, const int32_t *order, int k,
                       int32_t *idx, float *dist, int32_t *stats, hipStream_t s) {
  const size_t heap_bytes = (size_t)k * kHeapLanes * sizeof(int64_t);
  // above 64 KB a kernel must be allowed the larger dynamic LDS explicitly
  // (on the current device; cheap, so done at every launch)
  const hipError_t allowed = hipFuncSetAttribute(
      reinterpret_cast<const void *>(&k_nearest_heap<KIND, FMT, STATS>),
      hipFuncAttributeMaxDynamicSharedMemorySize, (int)heap_bytes);
  if (allowed != hipSuccess) return hip_fail(allowed);
  const unsigned g = grid_for(m, kHeapLanes);
  return launch(STATS ? "nearest_stats" : "nearest", s, [&] {
    k_nearest_heap<KIND, FMT, STATS><<<g, kHeapLanes, heap_bytes, s>>>(t, pts, m, order, k, idx, dist,
                                                                      stats);
  });
}

template <int KIND, int FMT>
abx_status nearest_heap(const abx_bvh *b, const float *pts, int64_t m, const int32_t *order, int k,
                        int32_t *idx, float *dist, int32_t *stats, hipStream_t s) {
  const TreeArgs t = tree_args(b);
  if (stats) return launch_heap<KIND, FMT, true>(t, pts, m, order, k, idx, dist, stats, s);
  return launch_heap<KIND, FMT, false>(t, pts, m, order, k, idx, dist, stats, s);
}

template <int KIND, int FMT>
abx_status nearest_fmt(const abx_bvh *b, const float *pts, int64_t m, const int32_t *order, int k,
                       int32_t *idx, float *dist, int32_t *stats, const NearestScratch &ns,
                       hipStream_t s) {
  if (k <= 1) return nearest_k<KIND, FMT, 1>(b, pts, m, order, k, idx, dist, stats, ns, s);
  if (k <= 2) return nearest_k<KIND, FMT, 2>(b, pts, m, order, k, idx, dist, stats, ns, s);
  if (k <= 4) return nearest_k<KIND, FMT, 4>(b, pts, m, order, k, idx, dist, stats, ns, s);
  if (k <= 8) return nearest_k<KIND, FMT, 8>(b, pts, m, order, k, idx, dist, stats, ns, s);
  if (k <= 10) return nearest_k<KIND, FMT, 10>(b, pts, m, order, k, idx, dist, stats, ns, s);
  if (k <= 16) return nearest_k<KIND, FMT, 16>(b, pts, m, order, k, idx, dist, stats, ns, s);
  if (k <= 32) return nearest_k<KIND, FMT, 32>(b, pts, m, order, k, idx, dist, stats, ns, s);
  if (k <= 48) return nearest_k<KIND, FMT, 48>(b, pts, m, order, k, idx, dist, stats, ns, s);
  return nearest_k<KIND, FMT, kMaxRegK>(b, pts, m, order, k, idx, dist, stats, ns, s);
}

// Visits after which a query of a batch of m leaves its lane for a workgroup.
// A node costs the cooperative pass about as much as the one-lane pass of a
// full GPU, so what decides is how many queries the other lanes and CUs wait
// for, and how many short walks would pay for a hand-off they do not need.
//   36 + k     the least: a bound needs k leaves.  With fewer visits the
//              workgroup starts without one (1e7 points, 1000 queries, k = 32:
//              165 us with 64 visits, 495 with 48).
//   the next   up to what nearly all walks among evenly spread points take
//              (8k + 100), in step with the batch: up to some 1e4 queries the
//              GPU has room for workgroups (1e6 points, 1000 queries, k = 10:
//              132 us against 233 with 512 visits); with 1e5, all of them
//              handed over at 100 visits took 1150 us instead of 770 (k = 64).
//   m / 1024   longer walks, as the one-lane pass fills the GPU for longer
//              (1e7-point shell, k = 10: 1e6 queries 5.7 ms with 1200 to 1800
//              visits, 9.3 with 8192; 1e7 queries 119 ms with 4096 to 12288,
//              125 with 22528: up to 8192).
// A 4-wide walk makes about half as many visits, so its upper limits are half.
// A caller who asks for no limit (INT64_MAX) gets none.
int64_t effective_budget(int64_t budget, int64_t m, int k, bool wide) {
  if (budget == INT64_MAX) return budget;
  if (wide) budget = std::max<int64_t>(1, budget / 2);
  const int64_t usual = std::min<int64_t>(m * (10 + k) / 6400, 100 + 8 * k);
  return std::min(budget, 36 + k + usual + std::min<int64_t>(m / 1024, wide ? 4096 : 8192));
}

abx_status launch_nearest(const abx_bvh *b, const float *pts, int64_t m, const int32_t *order,
                          int k, int32_t *idx, float *dist, int32_t *stats, int32_t *heavy_q,
                          float *heavy_bound, int32_t *huge_q, float *huge_bound,
                          uint32_t *counters, int32_t *heavy_state,
                          int64_t state_cap, int64_t budget, hipStream_t s) {
  if (m == 0 || k == 0) return ABX_OK;
  if (k > kMaxHeapK) return ABX_ERR_UNSUPPORTED;
#define ABX_BY_FORMAT(CALL, KD)                                      \
  do {                                                               \
    if (b->format == ABX_NODES_FP32) return CALL(KD, ABX_NODES_FP32); \
    if (b->format == ABX_NODES_Q16W) return CALL(KD, ABX_NODES_Q16W); \
    return CALL(KD, ABX_NODES_Q16);                                  \
  } while (0)
  if (k > kMaxRegK) {
#define ABX_HEAP(KD, FM) nearest_heap<KD, FM>(b, pts, m, order, k, idx, dist, stats, s)
    if (b->kind == ABX_PRIM_POINTS) ABX_BY_FORMAT(ABX_HEAP, ABX_PRIM_POINTS);
    ABX_BY_FORMAT(ABX_HEAP, ABX_PRIM_BOXES);
#undef ABX_HEAP
  }
  const NearestScratch ns{heavy_q, heavy_bound, huge_q, huge_bound, counters,
                          effective_budget(budget, m, k, b->format == ABX_NODES_Q16W), heavy_state,
                          (uint32_t)std::min<int64_t>(state_cap, kMaxSavedHeavy)};
#define ABX_FMT(KD, FM) nearest_fmt<KD, FM>(b, pts, m, order, k, idx, dist, stats, ns, s)
  if (b->kind == ABX_PRIM_POINTS) ABX_BY_FORMAT(ABX_FMT, ABX_PRIM_POINTS);
  ABX_BY_FORMAT(ABX_FMT, ABX_PRIM_BOXES);
#undef ABX_FMT
#undef ABX_BY_FORMAT
}

int max_tree_depth() { return kMaxDepth; }

}  // namespace abx
