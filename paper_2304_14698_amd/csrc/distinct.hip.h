// Distinct nodes of a batch, level by level. The candidates of a state are local rewrites of its current
// graph, so most of their nodes have, for the first rounds, exactly the history of a node of another
// graph: the same operator, attributes and incoming edge attributes (level 0), and at level l + 1 the
// same level-l class and, edge by edge in the batch's receiver order, senders of the same level-l
// classes; the first two in-edges of a node count in either order, since every sum over a node's
// in-edges adds these two to each other before anything else. Nodes of one class at level l have the same state after l rounds, bit for bit, so a round
// is computed once per class, on the graph of one representative per class (its smallest node) and
// the representatives' in-edges.
//
// Classes are found by hashing a node's key into an open-addressing table (36-bit tag, smallest node
// that has it) and then comparing the key itself with that node's, word by word: a node whose tag
// is another key's too becomes a class of its own, so equality never rests on the hash.
// The search for a tag begins at a slot that the tag alone decides, so nodes of one tag share one slot
// whatever order the hardware ran in, and with it the classes. (A slot chosen by other bits of the hash
// would let two keys of one tag meet or miss each other by the order of insertion.) Class numbers
// ascend with their representatives.
//
// What it saves, a kept minibatch's update step, whole / reduced / with the first two in-edges in either order: 4.3 M nodes,
// H = 256: 88.0 / 11.0 / 3.42 ms (13, then 2.5 % of the edges left over five rounds); 354 k nodes, H = 128: 4.3 / 1.11 / 0.82 ms (24, 10 %);
// 73 k nodes re-evaluated in fp32: 1.19 / 0.35 / 0.23 ms (36, 6 %). The attention rounds keep to the whole batch: their backward gathers per sender, and a
// sender shared by thousands of graphs made that pass 8 times slower than what the rest gained.
//
// Bound by gathers of 4-byte class numbers and by table probes: one pass of each over the nodes and
// edges per level, against two matrix products per edge and node and round for what it saves.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "segsum.hip.h"

constexpr int kMaxLevels = 16;            // levels 0 .. rounds
constexpr unsigned long long kEmptySlot = ~0ull;
constexpr int kNodeBits = 28;             // of a table slot; the others are the tag (a batch has fewer than 2^28 - 1 nodes)
constexpr int kScanItems = 1024;          // nodes per block of the class kernels (four per thread)

struct ClassArgs {
  int64_t N;
  const int32_t *in_ptr, *in_src, *node_op;
  const uint32_t *edge_feat, *node_dense;  // bit patterns
  int De, Dd;
  const uint8_t *swapped;                  // [N] 1: the first two in-edges change places (see first_two_kernel)
  const int32_t *prev;                     // class of each node one level below; nullptr: level 0
  unsigned long long *table;               // [mask + 1] tag << kNodeBits | smallest node, kEmptySlot
  uint32_t mask;
  const int32_t *state_graph_ptr, *graph_node_ptr;
  int32_t *slot;                           // [N] table slot, then (representatives) the class number
  int32_t *rep;                            // [N]
  int2 *block_sum;                         // [blocks] classes and their in-edges, then exclusive sums
  int32_t *totals;                         // [2] classes and in-edges of the level
  int32_t *receivers;                      // [1] set to zero for level_fill_kernel
  int32_t *reps;                           // [classes] representative of each class
  int32_t *ptr;                            // [classes + 1] in-edges of the representatives
  int32_t *cls;                            // [N] class of each node
};

__device__ __forceinline__ uint64_t mix64(uint64_t h, uint64_t v) {   // (order-sensitive)
  h = (h ^ v) * 0x9E3779B97F4A7C15ull;
  return h ^ (h >> 29);
}

__global__ __launch_bounds__(256) void class_clear_kernel(unsigned long long *table, uint32_t n) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < n) table[i] = kEmptySlot;
}

// The graphs of a state list their edges in different orders, so the first two in-edges of a node and of its
// copies in other graphs often come swapped, and what is downstream of them would be distinct (the sums are the
// same bits: x + y = y + x). Where a node's two come is therefore decided by the attributes' bit patterns, then the senders'
// operators, attributes and in-degrees: pairs alike in all of these stay as given, which may cost a class,
// never a wrong one. (The third and further in-edges keep their places: another order would be other sums.)
// Edges left, rounds 1-5: 4.3 M nodes of 16 transformer states 1.7, 2.9, 6, 18, 37 % -> 1.3, 1.9, 2.4, 3.0, 3.8; one such
// state 7, 17, 36, 53, 70 % -> 3, 5, 6, 7, 8; 16 residual networks' states 7, 11, 20, 34, 49 % -> 5, 7, 10, 13, 17.
__global__ __launch_bounds__(256) void first_two_kernel(const ClassArgs a, uint8_t *swapped) {
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (n >= a.N) return;
  const int e0 = a.in_ptr[n];
  int order = 0;                           // 1: the second comes first, -1: as given
  if (a.in_ptr[n + 1] - e0 >= 2) {
    auto differ = [&](uint32_t x, uint32_t y) {
      if (order == 0 && x != y) order = y < x ? 1 : -1;
    };
    const size_t f = (size_t)e0 * a.De;
    for (int w = 0; w < a.De && order == 0; ++w) differ(a.edge_feat[f + w], a.edge_feat[f + a.De + w]);
    if (order == 0) {
      const int32_t s = a.in_src[e0], t = a.in_src[e0 + 1];
      differ((uint32_t)a.node_op[s], (uint32_t)a.node_op[t]);
      for (int k = 0; k < a.Dd && order == 0; ++k) differ(a.node_dense[(size_t)s * a.Dd + k], a.node_dense[(size_t)t * a.Dd + k]);
      differ((uint32_t)(a.in_ptr[s + 1] - a.in_ptr[s]), (uint32_t)(a.in_ptr[t + 1] - a.in_ptr[t]));
    }
  }
  swapped[n] = order > 0;
}
// the k-th in-edge of a node whose first is e0
__device__ __forceinline__ int in_edge(int e0, int k, int swapped) { return e0 + (k < 2 ? k ^ swapped : k); }

// Key of a node, its in-edges four at a time: a loop over single edges waits for each by itself (once_insert_kernel,
// 305 k nodes: 22.8 us, so 19.0).
constexpr int kEdgesAtOnce = 4;
typedef uint32_t u32x4k __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void key_edges(int e0, int d, int sw, int k0, int *e) {     // (past the last: the last again)
#pragma unroll
  for (int i = 0; i < kEdgesAtOnce; ++i) e[i] = in_edge(e0, k0 + i < d ? k0 + i : d - 1, d > 1 ? sw : 0);
}
__device__ __forceinline__ void sender_classes(const ClassArgs &a, const int *e, int *p) {
#pragma unroll
  for (int i = 0; i < kEdgesAtOnce; ++i) p[i] = a.in_src[e[i]];
#pragma unroll
  for (int i = 0; i < kEdgesAtOnce; ++i) p[i] = a.prev[p[i]];
}
__device__ __forceinline__ void edge_words(const ClassArgs &a, const int *e, int q, u32x4k *x) {
#pragma unroll
  for (int i = 0; i < kEdgesAtOnce; ++i) x[i] = ((const u32x4k *)(a.edge_feat + (size_t)e[i] * a.De))[q];   // (De is a multiple of 4)
}
__device__ __forceinline__ uint64_t class_hash(const ClassArgs &a, int64_t n) {
  const int e0 = a.in_ptr[n], d = a.in_ptr[n + 1] - e0, sw = a.swapped[n];
  uint64_t h;
  if (a.prev) {
    h = mix64(0x51ED270B27B4F3CFull, (uint32_t)a.prev[n]);
  } else {
    h = mix64((uint32_t)a.node_op[n], (uint32_t)d);
    for (int k = 0; k < a.Dd; ++k) h = mix64(h, a.node_dense[(size_t)n * a.Dd + k]);
  }
  for (int k0 = 0; k0 < d; k0 += kEdgesAtOnce) {
    int e[kEdgesAtOnce];
    key_edges(e0, d, sw, k0, e);
    if (a.prev) {
      int p[kEdgesAtOnce];
      sender_classes(a, e, p);
#pragma unroll
      for (int i = 0; i < kEdgesAtOnce; ++i)
        if (k0 + i < d) h = mix64(h, (uint32_t)p[i]);
    } else {
      for (int q = 0; q < a.De / 4; ++q) {
        u32x4k x[kEdgesAtOnce];
        edge_words(a, e, q, x);
#pragma unroll
        for (int i = 0; i < kEdgesAtOnce; ++i)
          if (k0 + i < d) h = mix64(mix64(h, x[i][0] | (uint64_t)x[i][1] << 32), x[i][2] | (uint64_t)x[i][3] << 32);
      }
    }
  }
  return mix64(h, h >> 32);
}
__device__ __forceinline__ void class_insert(const ClassArgs &a, int64_t n) {
  const uint64_t h = class_hash(a, n);
  const unsigned long long tag = h >> kNodeBits, mine = tag << kNodeBits | (uint32_t)n;
  uint32_t s = (uint32_t)tag & a.mask;
  for (uint32_t i = 0; i <= a.mask; ++i, s = (s + 1) & a.mask) {      // (the table has more slots than there are nodes)
    // (a slot's tag is written once and its node only falls: most nodes find themselves above it)
    unsigned long long w = __hip_atomic_load(a.table + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (w == kEmptySlot) {
      w = atomicCAS(a.table + s, kEmptySlot, mine);
      if (w == kEmptySlot) w = mine;
    }
    if (w >> kNodeBits != tag) continue;
    if (w > mine) atomicMin(a.table + s, mine);
    a.slot[n] = (int32_t)s;
    break;
  }
}
// The nodes of every state's first graph, a block each, before all nodes: they are the smallest of most
// classes, so the others find their class in place and leave the table alone (all at once, thousands
// of nodes would go for the same slots: 98 us per level at 703 k nodes of 2080 graphs, against 9 for these and
// then 30 for all).
__global__ __launch_bounds__(256) void class_insert_first_kernel(const ClassArgs a) {
  touch_args(a);
  const int g = a.state_graph_ptr[blockIdx.x], n1 = a.graph_node_ptr[g + 1];
  for (int n = a.graph_node_ptr[g] + threadIdx.x; n < n1; n += 256) class_insert(a, n);
}
__global__ __launch_bounds__(256) void class_insert_kernel(const ClassArgs a) {
  touch_args(a);
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (n < a.N) class_insert(a, n);
}

__device__ __forceinline__ bool same_key(const ClassArgs &a, int64_t n, int64_t r) {
  const int e0 = a.in_ptr[n], d = a.in_ptr[n + 1] - e0, sn = a.swapped[n];
  const int f0 = a.in_ptr[r], dr = a.in_ptr[r + 1] - f0, sr = a.swapped[r];
  bool same = d == dr;
  if (a.prev) {
    same &= a.prev[n] == a.prev[r];
  } else {
    same &= a.node_op[n] == a.node_op[r];
    for (int k = 0; k < a.Dd; ++k) same &= a.node_dense[(size_t)n * a.Dd + k] == a.node_dense[(size_t)r * a.Dd + k];
  }
  if (!same) return false;
  for (int k0 = 0; k0 < d; k0 += kEdgesAtOnce) {
    int e[kEdgesAtOnce], f[kEdgesAtOnce];
    key_edges(e0, d, sn, k0, e);
    key_edges(f0, d, sr, k0, f);
    if (a.prev) {
      int p[kEdgesAtOnce], q[kEdgesAtOnce];
      sender_classes(a, e, p);
      sender_classes(a, f, q);
#pragma unroll
      for (int i = 0; i < kEdgesAtOnce; ++i) same &= p[i] == q[i];
    } else {
      for (int w = 0; w < a.De / 4; ++w) {
        u32x4k x[kEdgesAtOnce], y[kEdgesAtOnce];
        edge_words(a, e, w, x);
        edge_words(a, f, w, y);
#pragma unroll
        for (int i = 0; i < kEdgesAtOnce; ++i) same &= x[i][0] == y[i][0] && x[i][1] == y[i][1] && x[i][2] == y[i][2] && x[i][3] == y[i][3];
      }
    }
  }
  return same;
}

// exclusive sums over the 256 threads of a block; total of all in `sum`
__device__ __forceinline__ int2 block_scan_pair(int2 v, int2 *wave_sum, int2 &sum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int2 x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const int px = __shfl_up(x.x, o), py = __shfl_up(x.y, o);
    if (lane >= o) { x.x += px; x.y += py; }
  }
  if (lane == 63) wave_sum[w] = x;
  __syncthreads();
  int2 before = make_int2(0, 0);
  sum = make_int2(0, 0);
  for (int k = 0; k < (int)blockDim.x / 64; ++k) {
    if (k < w) { before.x += wave_sum[k].x; before.y += wave_sum[k].y; }
    sum.x += wave_sum[k].x; sum.y += wave_sum[k].y;
  }
  __syncthreads();
  return make_int2(before.x + x.x - v.x, before.y + x.y - v.y);
}

__global__ __launch_bounds__(256) void class_verify_kernel(const ClassArgs a) {
  touch_args(a);
  __shared__ int2 ws[4];
  int2 v = make_int2(0, 0), sum;
  for (int i = 0; i < kScanItems / 256; ++i) {
    const int64_t n = (int64_t)blockIdx.x * kScanItems + i * 256 + threadIdx.x;
    if (n >= a.N) break;
    int32_t r = (int32_t)(a.table[a.slot[n]] & ((1u << kNodeBits) - 1));
    if (r != (int32_t)n && !same_key(a, n, r)) r = (int32_t)n;
    a.rep[n] = r;
    if (r == (int32_t)n) { ++v.x; v.y += a.in_ptr[n + 1] - a.in_ptr[n]; }
  }
  (void)block_scan_pair(v, ws, sum);
  if (threadIdx.x == 0) a.block_sum[blockIdx.x] = sum;
}

__global__ __launch_bounds__(256) void class_scan_kernel(const ClassArgs a, int n_blocks) {
  __shared__ int2 ws[4];
  int2 base = make_int2(0, 0);
  for (int i0 = 0; i0 < n_blocks; i0 += 256) {
    const int i = i0 + threadIdx.x;
    const int2 v = i < n_blocks ? a.block_sum[i] : make_int2(0, 0);
    int2 sum;
    const int2 x = block_scan_pair(v, ws, sum);
    if (i < n_blocks) a.block_sum[i] = make_int2(base.x + x.x, base.y + x.y);
    base.x += sum.x; base.y += sum.y;
  }
  if (threadIdx.x == 0) {
    a.totals[0] = base.x;
    a.totals[1] = base.y;
    *a.receivers = 0;
    a.ptr[base.x] = base.y;
  }
}

__global__ __launch_bounds__(256) void class_number_kernel(const ClassArgs a) {
  __shared__ int2 ws[4];
  int2 base = a.block_sum[blockIdx.x];
  for (int i = 0; i < kScanItems / 256; ++i) {
    const int64_t n = (int64_t)blockIdx.x * kScanItems + i * 256 + threadIdx.x;
    const bool is_rep = n < a.N && a.rep[n] == (int32_t)n;
    const int2 v = is_rep ? make_int2(1, a.in_ptr[n + 1] - a.in_ptr[n]) : make_int2(0, 0);
    int2 sum;
    const int2 x = block_scan_pair(v, ws, sum);
    if (is_rep) {
      a.slot[n] = base.x + x.x;
      a.reps[base.x + x.x] = (int32_t)n;
      a.ptr[base.x + x.x] = base.y + x.y;
    }
    base.x += sum.x; base.y += sum.y;
  }
}

__global__ __launch_bounds__(256) void class_of_kernel(const ClassArgs a) {
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (n < a.N) a.cls[n] = a.slot[a.rep[n]];
}

// The graph of a level's representatives: receiver-order arrays like the batch's own.
struct LevelFillArgs {
  int64_t n_cls;
  const int32_t *reps, *ptr, *cls, *prev;   // classes of this level and of the one below (nullptr: level 0)
  const int32_t *in_ptr, *in_src, *node_op;
  const float *edge_feat, *node_dense;
  int De, Dd;
  int32_t *o_ptr, *o_src, *o_dst, *o_agg_src, *o_self, *o_op;
  int32_t *o_below_src, *o_below_dst;       // nullable
  float *o_feat, *o_dense;
  int32_t *receivers;                       // classes with in-edges, counted
};
__global__ __launch_bounds__(256) void level_fill_kernel(const LevelFillArgs a) {
  touch_args(a);
  const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (c >= a.n_cls) return;
  const int32_t r = a.reps[c], e0 = a.in_ptr[r], d = a.in_ptr[r + 1] - e0, p0 = a.ptr[c];
  const unsigned long long with = __ballot(d > 0);
  if ((threadIdx.x & 63) == 0 && with) atomicAdd(a.receivers, __popcll(with));
  a.o_ptr[c] = p0;
  if (c == a.n_cls - 1) a.o_ptr[a.n_cls] = p0 + d;
  a.o_agg_src[c] = d > 0 ? (int32_t)c : -1;
  if (a.prev) {
    a.o_self[c] = a.prev[r];
    for (int k = 0; k < d; ++k) {
      a.o_src[p0 + k] = a.cls[a.in_src[e0 + k]];
      a.o_dst[p0 + k] = (int32_t)c;
      if (a.o_below_src) {
        a.o_below_src[p0 + k] = a.prev[a.in_src[e0 + k]];
        a.o_below_dst[p0 + k] = a.prev[r];
      }
    }
  } else {
    a.o_op[c] = a.node_op[r];
    for (int k = 0; k < a.Dd; ++k) a.o_dense[(size_t)c * a.Dd + k] = a.node_dense[(size_t)r * a.Dd + k];
  }
  const f32x4 *src = (const f32x4 *)(a.edge_feat + (size_t)e0 * a.De);      // (De is a multiple of 4)
  f32x4 *dst = (f32x4 *)(a.o_feat + (size_t)p0 * a.De);
  for (int k = 0; k < d * (a.De / 4); ++k) dst[k] = src[k];
}

// ---- Reduced for one encode. A batch that is encoded once, forward only, cannot pay for the waits, nor for what a
// backward pass needs of the levels: its levels are made one at a time in front of the round that runs on them, in the
// same memory, and their sizes never leave the device (the kernels of a round read them, with a grid that fills the
// chip). A node is compared where it finds its tag taken, with the node that took the slot, which stays its
// class's representative: whichever node of a class comes first, so class numbers differ from run to run, states do not.
// A block of once_fill_kernel numbers the representatives among its nodes, cuts their in-edges into tiles by
// itself (one unfilled tile a block) and takes its place among classes, edges and tiles in one atomic addition, so that
// all three stay contiguous in one order. The round's kernels read the states of the level below through
// `self` and the senders' classes there: no copy of the states in between.
// Bound by chains of gathers (nine dependent ones in once_insert_kernel), so all loads of a node's first four in-edges are in
// flight at once. 305 k nodes of 257 graphs, a level: first graphs 6 us, insert 19, fill 16, classes 6, in place of 285 us a
// round of the whole batch at H = 256 where 14 to 73 % of the edges are left; an encode 1.42 -> 0.84 ms of GPU time.
constexpr int kOnceNodes = 512;           // nodes per block of once_fill_kernel
constexpr int kOnceDegree = 32;           // in-edges of a node at most
constexpr int64_t kOnceMax = (int64_t)1 << (kCountBits - 1);   // nodes and edges of such a batch
struct OnceArgs {
  ClassArgs k;                            // (slot, table, prev, cls and the batch; no rep, block_sum, totals, reps, ptr)
  int32_t *num;                           // [slots] class number
  unsigned long long *counts;             // of this level
  int32_t *o_ptr, *o_src, *o_dst, *o_agg_src, *o_self, *o_hrow, *o_op, *o_tile;
  float *o_feat, *o_dense;
};
__global__ __launch_bounds__(256) void once_clear_kernel(unsigned long long *table, uint32_t slots, unsigned long long *counts) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < slots) table[i] = kEmptySlot;
  if (i < (uint32_t)kMaxLevels) counts[i] = 0;
}
__device__ __forceinline__ void once_insert(const ClassArgs &a, int64_t n) {
  const unsigned long long tag = class_hash(a, n) >> kNodeBits, mine = tag << kNodeBits | (uint32_t)n;
  uint32_t s = (uint32_t)tag & a.mask;
  for (uint32_t i = 0; i <= a.mask; ++i, s = (s + 1) & a.mask) {      // (the table has more slots than there are nodes)
    unsigned long long w = __hip_atomic_load(a.table + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (w == kEmptySlot) {
      w = atomicCAS(a.table + s, kEmptySlot, mine);
      if (w == kEmptySlot) w = mine;
    }
    if (w >> kNodeBits != tag) continue;
    const int64_t r = (int64_t)(w & ((1u << kNodeBits) - 1));
    if (r != n && !same_key(a, n, r)) continue;
    a.slot[n] = (int32_t)s;
    break;
  }
}
// the nodes of every state's first graph ahead of the others (see class_insert_first_kernel)
__global__ __launch_bounds__(256) void once_insert_first_kernel(const ClassArgs a, int blocks_per_graph) {
  touch_args(a);
  const int g = a.state_graph_ptr[blockIdx.x / blocks_per_graph];
  const int n = a.graph_node_ptr[g] + (int)(blockIdx.x % blocks_per_graph) * 256 + (int)threadIdx.x;
  if (n < a.graph_node_ptr[g + 1]) once_insert(a, n);
}
__global__ __launch_bounds__(256) void once_insert_kernel(const ClassArgs a) {
  touch_args(a);
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (n < a.N) once_insert(a, n);
}
__global__ __launch_bounds__(256) void once_fill_kernel(const OnceArgs o) {
  constexpr int PER = kOnceNodes / 256, kCuts = 2 * (kOnceNodes * kOnceDegree + 32) / 33 + 2;
  __shared__ uint16_t owner[kOnceNodes * kOnceDegree];   // the block's j-th edge: its receiver among the block's representatives
  __shared__ uint16_t cut[kCuts + 1];
  __shared__ int first[kOnceNodes], given[kOnceNodes], below[kOnceNodes];   // a representative's first edge here and in the batch, its class below
  __shared__ int2 ws[4];
  __shared__ int n_cuts;
  __shared__ unsigned long long place;
  const ClassArgs &a = o.k;
  const int64_t n0 = (int64_t)blockIdx.x * kOnceNodes + PER * (int)threadIdx.x;
  int slot[PER], f0[PER], deg[PER], self[PER];
  unsigned long long w[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int64_t n = n0 + i < a.N ? n0 + i : a.N - 1;
    slot[i] = a.slot[n];
    f0[i] = a.in_ptr[n];
    deg[i] = a.in_ptr[n + 1] - f0[i];
    self[i] = a.prev ? a.prev[n] : 0;
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) w[i] = a.table[slot[i]] & ((1u << kNodeBits) - 1);
  int2 mine = make_int2(0, 0), sum;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (n0 + i >= a.N || w[i] != (unsigned long long)(n0 + i)) slot[i] = -1;
    if (slot[i] >= 0) { ++mine.x; mine.y += deg[i]; }
  }
  const int2 before = block_scan_pair(mine, ws, sum);
  if (sum.x == 0) return;                                // (the whole block)
  int2 at = before;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (slot[i] < 0) continue;
    first[at.x] = at.y;
    given[at.x] = f0[i];
    below[at.x] = self[i];
    for (int k = 0; k < deg[i]; ++k) owner[at.y + k] = (uint16_t)at.x;
    ++at.x; at.y += deg[i];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int c = 0;
    for (int s = 0; s < sum.y && c < kCuts;) {
      cut[c++] = (uint16_t)s;
      s = s + 32 >= sum.y ? sum.y : first[owner[s + 32]];   // (after s: in-degrees <= 32)
    }
    n_cuts = c;
    place = atomicAdd(o.counts, (unsigned long long)sum.x | (unsigned long long)sum.y << kCountBits | (unsigned long long)c << 2 * kCountBits);
  }
  __syncthreads();
  const int c0 = level_classes(place), e0 = level_edges(place), t0 = level_tiles(place);
  for (int i = threadIdx.x; i <= n_cuts; i += 256) o.o_tile[t0 + i] = e0 + (i < n_cuts ? cut[i] : sum.y);
  if (threadIdx.x == 0) o.o_ptr[c0 + sum.x] = e0 + sum.y;         // (the next block's first, or the end)
  at = before;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (slot[i] < 0) continue;
    const int c = c0 + at.x;
    o.num[slot[i]] = c;
    o.o_ptr[c] = e0 + at.y;
    o.o_agg_src[c] = deg[i] > 0 ? c : -1;
    if (a.prev) {
      o.o_self[c] = self[i];
    } else {
      o.o_op[c] = a.node_op[n0 + i];
      for (int k = 0; k < a.Dd; ++k) o.o_dense[(size_t)c * a.Dd + k] = __uint_as_float(a.node_dense[(size_t)(n0 + i) * a.Dd + k]);
    }
    ++at.x; at.y += deg[i];
  }
  if (a.prev)
    for (int j = threadIdx.x; j < sum.y; j += 256) {
      const int v = owner[j];
      o.o_src[e0 + j] = a.prev[a.in_src[given[v] + j - first[v]]];
      o.o_dst[e0 + j] = c0 + v;
      o.o_hrow[e0 + j] = below[v];
    }
  const int P = a.De / 4;                                          // (De is a multiple of 4)
  for (int x = threadIdx.x; x < sum.y * P; x += 256) {
    const int j = x / P, q = x - j * P, v = owner[j];
    ((u32x4k *)(o.o_feat + (size_t)(e0 + j) * a.De))[q] = ((const u32x4k *)(a.edge_feat + (size_t)(given[v] + j - first[v]) * a.De))[q];
  }
}
// the nodes' classes; and the table empty for the next level
__global__ __launch_bounds__(256) void once_class_kernel(const ClassArgs a, const int32_t *num) {
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (n < a.N) a.cls[n] = num[a.slot[n]];
  for (int64_t i = n; i <= (int64_t)a.mask; i += (int64_t)gridDim.x * 256) a.table[i] = kEmptySlot;
}

// Edge tiles of the levels 1 .. rounds: at most 32 edges, cut at receiver boundaries (no receiver of such a
// batch has more than 32). The cut starts afresh every kTileChunk edges, so a block cuts a chunk by
// itself: at one unfilled tile in about 66, where a cut of the whole level is one serial chain.
constexpr int kTileChunk = 2048, kTileChunkMax = 2 * (kTileChunk + 32) / 33 + 2;   // tiles of a chunk at most
struct TileLevels {
  int n_levels;                             // entries below
  int chunk0[kMaxLevels + 1];               // first chunk of each level
  int32_t n_edges[kMaxLevels];
  const int32_t *ptr[kMaxLevels], *dst[kMaxLevels];
  int32_t *tile_ptr[kMaxLevels];
  int32_t *cuts;                            // [chunks][kTileChunkMax]
  int32_t *count;                           // [chunks] tiles, then the first tile of each chunk
  int32_t *totals;                          // [n_levels] tiles of each level
};
__device__ __forceinline__ int tile_level(const TileLevels &a, int chunk) {
  int l = 0;
  while (l + 1 < a.n_levels && chunk >= a.chunk0[l + 1]) ++l;
  return l;
}
__global__ __launch_bounds__(256) void tile_cut_kernel(const TileLevels a) {
  __shared__ int32_t start[kTileChunk + 64];   // first edge of the receiver of edge e0 + j, less e0
  const int l = tile_level(a, blockIdx.x);
  const int32_t E = a.n_edges[l], k = (int)blockIdx.x - a.chunk0[l];
  const int32_t *ptr = a.ptr[l], *dst = a.dst[l];
  // the chunk: from the first receiver boundary at or after k * kTileChunk to the next chunk's
  auto boundary = [&](int64_t e) -> int32_t {
    if (e >= E) return E;
    const int32_t r = dst[e];
    return ptr[r] == (int32_t)e ? (int32_t)e : ptr[r + 1];
  };
  const int32_t e0 = boundary((int64_t)k * kTileChunk), e1 = boundary((int64_t)(k + 1) * kTileChunk);
  const int32_t n = e1 - e0;                   // <= kTileChunk + 31
  for (int j = threadIdx.x; j < n; j += 256) start[j] = ptr[dst[e0 + j]] - e0;
  __syncthreads();
  if (threadIdx.x != 0) return;
  int32_t *cuts = a.cuts + (size_t)blockIdx.x * kTileChunkMax;
  int c = 0;
  for (int s = 0; s < n && c < kTileChunkMax;) {
    cuts[c++] = e0 + s;
    s = s + 32 >= n ? n : start[s + 32];       // the receiver of edge s + 32 starts the next tile (after s: in-degrees <= 32)
  }
  a.count[blockIdx.x] = c;
}
__global__ __launch_bounds__(256) void tile_scan_kernel(const TileLevels a) {
  __shared__ int2 ws[4];
  const int l = blockIdx.x, c0 = a.chunk0[l], c1 = a.chunk0[l + 1];
  int base = 0;
  for (int i0 = c0; i0 < c1; i0 += 256) {
    const int i = i0 + threadIdx.x;
    const int2 v = make_int2(i < c1 ? a.count[i] : 0, 0);
    int2 sum;
    const int2 x = block_scan_pair(v, ws, sum);
    if (i < c1) a.count[i] = base + x.x;
    base += sum.x;
  }
  if (threadIdx.x == 0) {
    a.totals[l] = base;
    a.tile_ptr[l][base] = a.n_edges[l];
  }
}
__global__ __launch_bounds__(256) void tile_write_kernel(const TileLevels a) {
  const int l = tile_level(a, blockIdx.x);
  const int32_t first = a.count[blockIdx.x];
  const int32_t last = (int)blockIdx.x + 1 < a.chunk0[l + 1] ? a.count[blockIdx.x + 1] : a.totals[l];
  for (int i = threadIdx.x; i < last - first; i += 256)
    a.tile_ptr[l][first + i] = a.cuts[(size_t)blockIdx.x * kTileChunkMax + i];
}

// ---- groupings for the backward pass. What a class receives from the level above: the gradients of the
// level's edges whose sender's class it is, those of the level's classes that split it, and what these
// received, rows of one list [edges as senders | classes | received]; and the classes of the last
// level, the pool's gradient for each of their nodes. The three are summed in one fp32 sum and rounded
// once, like a node's gradient in a batch that is not reduced. Received: per class, summed by the
// edge kernel (a class without in-edges has no such row: value -1, a row of zeros), or per edge.
// All groupings are made in one stable radix sort: each owns a range of items and a
// range of keys, in the same order. (A sender may have thousands of edges here, one from every
// graph it is shared by: a sum per segment cut into 16-row pieces, not a loop per node.)
constexpr int kMaxGroupings = kMaxLevels;
struct GroupArgs {
  int n;                                       // groupings
  int64_t item0[kMaxGroupings + 1];            // first item of each
  uint32_t key0[kMaxGroupings + 1];            // first key of each
  int64_t n_edges[kMaxGroupings];              // level groupings: the first items, edges as senders ...
  int64_t n_cls[kMaxGroupings];                // ... then classes, then received rows (members: nodes only)
  const int32_t *src[kMaxGroupings];           // level groupings: senders of the edges
  const int32_t *dst[kMaxGroupings];           // ... their receivers; nullptr: received rows are per class
  const int32_t *agg_src[kMaxGroupings];       // ... -1 for a class without in-edges
  const int32_t *key[kMaxGroupings];           // key of each class, or (members) of each node
  const int32_t *val[kMaxGroupings];           // value of each item; nullptr: the item's index
  int32_t *ptr[kMaxGroupings];                 // [keys + 1] out: first sorted item of each key
  int32_t *seg[kMaxGroupings];                 // [items] out: key of each sorted item
  int32_t *out[kMaxGroupings];                 // [items] out: sorted values
};
__device__ __forceinline__ int grouping_of(const GroupArgs &a, int64_t i) {
  int lo = 0, hi = a.n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a.item0[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}
__global__ __launch_bounds__(256) void group_items_kernel(const GroupArgs a, uint2 *items) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.item0[a.n]) return;
  const int g = grouping_of(a, i);
  const int64_t j = i - a.item0[g];
  const int64_t k = j - a.n_edges[g], q = k - a.n_cls[g];
  const int64_t c = k < 0 ? a.src[g][j] : q < 0 ? k : a.dst[g] ? a.dst[g][q] : q;
  int32_t v = a.val[g] ? a.val[g][j] : (int32_t)j;
  if (q >= 0 && !a.dst[g] && a.agg_src[g][c] < 0) v = -1;
  items[i] = make_uint2(a.key0[g] + (uint32_t)a.key[g][c], (uint32_t)v);
}
constexpr int kSortItems = 4096;               // items per block: four waves of 1024 consecutive ones
__global__ __launch_bounds__(256) void sort_count_kernel(const uint2 *items, int64_t n, int shift, int32_t *hist, int n_blocks) {
  __shared__ int cnt[256];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * kSortItems;
  for (int k = threadIdx.x; k < kSortItems; k += 256)
    if (i0 + k < n) atomicAdd(&cnt[(items[i0 + k].x >> shift) & 255], 1);
  __syncthreads();
  hist[(size_t)threadIdx.x * n_blocks + blockIdx.x] = cnt[threadIdx.x];
}
// one block per digit: exclusive sums over the blocks, the digit's total to digit_total
__global__ __launch_bounds__(256) void sort_scan_kernel(int32_t *hist, int n_blocks, int32_t *digit_total) {
  __shared__ int2 ws[4];
  int32_t *h = hist + (size_t)blockIdx.x * n_blocks;
  int base = 0;
  for (int i0 = 0; i0 < n_blocks; i0 += 256) {
    const int i = i0 + threadIdx.x;
    int2 sum;
    const int2 x = block_scan_pair(make_int2(i < n_blocks ? h[i] : 0, 0), ws, sum);
    if (i < n_blocks) h[i] = base + x.x;
    base += sum.x;
  }
  if (threadIdx.x == 0) digit_total[blockIdx.x] = base;
}
__global__ __launch_bounds__(256) void sort_scatter_kernel(const uint2 *items, int64_t n, int shift, const int32_t *hist,
                                                           int n_blocks, const int32_t *digit_total, uint2 *out) {
  __shared__ int off[4][256];
  __shared__ int2 ws[4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  for (int k = 0; k < 4; ++k) off[k][t] = 0;
  __syncthreads();
  const int64_t w0 = (int64_t)blockIdx.x * kSortItems + w * (kSortItems / 4);
  for (int k = lane; k < kSortItems / 4; k += 64)
    if (w0 + k < n) atomicAdd(&off[w][(items[w0 + k].x >> shift) & 255], 1);
  __syncthreads();
  int2 sum;
  int base = block_scan_pair(make_int2(digit_total[t], 0), ws, sum).x + hist[(size_t)t * n_blocks + blockIdx.x];
  for (int k = 0; k < 4; ++k) {                // thread t: digit t's first place for each wave
    const int c = off[k][t];
    off[k][t] = base;
    base += c;
  }
  __syncthreads();
  volatile int *mine = off[w];
  for (int k = 0; k < kSortItems / 4; k += 64) {
    const int64_t i = w0 + k + lane;
    const bool in = i < n;
    const uint2 x = in ? items[i] : make_uint2(0, 0);
    const int d = (x.x >> shift) & 255;
    unsigned long long same = __ballot(in);
    for (int b = 0; b < 8; ++b) {
      const unsigned long long m = __ballot((d >> b) & 1);
      same &= (d >> b) & 1 ? m : ~m;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1));
    const int place = mine[d] + rank;
    __builtin_amdgcn_wave_barrier();
    if (in && rank == 0) mine[d] = place + __popcll(same);
    __builtin_amdgcn_wave_barrier();
    if (in) out[place] = x;
  }
}
__global__ __launch_bounds__(256) void group_write_kernel(const GroupArgs a, const uint2 *items) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.item0[a.n]) return;
  const int g = grouping_of(a, i);
  const int64_t j = i - a.item0[g];
  const int32_t k = (int32_t)(items[i].x - a.key0[g]);
  const int32_t before = j > 0 ? (int32_t)(items[i - 1].x - a.key0[g]) : -1;
  for (int32_t q = before + 1; q <= k; ++q) a.ptr[g][q] = (int32_t)j;
  if (i + 1 == a.item0[g + 1])
    for (int32_t q = k + 1; q <= (int32_t)(a.key0[g + 1] - a.key0[g]); ++q) a.ptr[g][q] = (int32_t)j + 1;
  a.seg[g][j] = k;
  a.out[g][j] = (int32_t)items[i].y;
}

// out[c, :] = in[from[c], :], rows of `pieces` 16-byte pieces: the states of a level's classes, which
// split the classes of the level below
__global__ __launch_bounds__(256) void expand_states_kernel(const f32x4 *in, const int32_t *from, int64_t n, int pieces,
                                                            f32x4 *out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n * pieces) return;
  const int64_t c = i / pieces;
  out[i] = in[(size_t)from[c] * pieces + (i - c * pieces)];
}

// Sums of rows per class in fp32 and, rounded once, their store in the operand type; with ymask (bf16) multiplied
// by the ReLU mask of the layer that produced the classes' states (see node_grad_gather_kernel). The
// rows are listed class by class (perm, -1 = a row of zeros; seg the class of each place; every class has
// one), and H / VEC lanes take STEPS times sixteen places: a step's indices, then all its rows and the mask words of the classes
// that end there, are requested at once, so a step waits twice whatever classes it holds. A class
// that lies inside the group is stored at once; the pieces of others go to carry[group][begun before, goes on], 8 H bytes a
// group and back again. One step leaves most lanes to hide the gathers with, four the fewest pieces. us of this kernel and the next at 1 / 2 / 4 steps, H = 256:
// 4.36 M rows of the pool's table 493 / 456 / 409, 3.5 M rows 535 / 492 / 458, 582 k rows 125 / 111 / 110, 162 k rows 36 / 32 / 35; H = 128: 368 k rows
// 42.8 / 38.8 / 45.1, 251 k 30.8 / 27.2 / 31.0, 143 k 22.5 / 22.8 / 28.7.
// Bound by the gather of the rows. H = 256, 3.4 M rows of 512 bytes into 400 k classes: 423 us (4.6 TB/s) and 99 for
// the classes in several pieces; a walk that read a segment's end when it reached it, an fp32 array of
// the sums and a pass that masked it took 815 + 90 + 108. The pool's gradient, 4.3 M rows of a 4.7 MB table:
// 379 + 123 us, 609 + 124 + 216 before.
// A table that every class gathers from and that no XCD's L2 holds is taken by column slices: block b belongs to slice b % 8,
// which the round-robin deal of blocks puts on one XCD, and an eighth of the table's columns fits its L2 (the indices are read
// eight times). The pool's gradient, H = 256, 15.9 M rows of a 17.3 MB table into 244 k classes: 1571 -> 979 us; 4.36 M rows of a
// 4.7 MB table 285 -> 275.
constexpr int kSumRows = 16;
struct ClassSumArgs {
  const void *vals, *zero_row;
  const int32_t *perm, *seg, *ptr;   // [n_rows] (readable up to the next multiple of sixteen), [classes + 1]
  int64_t n_rows;
  int D;
  const uint16_t *ymask;
  void *out;                         // [classes, D]
  float *carry;                      // [n_rows / group, rounded up][2][D]
  int group;                         // places a group of lanes takes
  int slices;                        // column slices, one after the other over the blocks: 1, or 8 (an XCD each)
};
// the mask bits of columns c .. c + 3 of row n (c a multiple of 4), lowest first
__device__ __forceinline__ unsigned mask_word(const uint16_t *ymask, int64_t n, int D, int c) {
  return ymask[((size_t)(n / 32) * (D / 32) + c / 32) * 64 + (size_t)(n % 32) + 8 * (c & 4)];
}
template <typename TOut>
__device__ __forceinline__ void store_masked4(TOut *p, float *v, bool masked, unsigned word, int c) {
  const unsigned bits = masked ? word >> (4 * (c % 32 / 8)) : 0xfu;
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = (bits >> j) & 1u ? v[j] : 0.f;
  store4<TOut>(p, v);
}
template <typename TIn, typename TOut, int VEC, int STEPS>
__global__ __launch_bounds__(256) void class_sum_kernel(const ClassSumArgs a) {
  touch_args(a);
  constexpr int NR = kSumRows, NQ = VEC / 4;
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const int lpr = a.D / VEC / a.slices;                    // lanes of a group
  const int64_t gt = (int64_t)(blockIdx.x / a.slices) * 256 + threadIdx.x;
  constexpr int GROUP = STEPS * NR;
  const int64_t st = gt / lpr, r_end = (st + 1) * GROUP < a.n_rows ? (st + 1) * GROUP : a.n_rows;
  int64_t r0 = st * GROUP;
  if (r0 >= a.n_rows) return;
  const int c = ((int)(blockIdx.x % a.slices) * lpr + (int)(gt - st * lpr)) * VEC;
  const bool masked = a.ymask != nullptr;
  const int before = r0 > 0 ? a.seg[r0 - 1] : -1;
  bool begun = false;
  float acc[VEC];
#pragma unroll
  for (int j = 0; j < VEC; ++j) acc[j] = 0.f;
  for (;;) {
    const int nv = r_end - r0 < NR ? (int)(r_end - r0) : NR;
    const bool last = STEPS == 1 || r0 + NR >= r_end;
    i32x4 row4[NR / 4], seg4[NR / 4];
#pragma unroll
    for (int i = 0; i < NR / 4; ++i) {
      row4[i] = ((const i32x4 *)(a.perm + r0))[i];
      seg4[i] = ((const i32x4 *)(a.seg + r0))[i];
    }
    const int after = r0 + NR < a.n_rows ? a.seg[r0 + NR] : -1;
    float v[NR][VEC];
    int seg[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int r = i < nv ? row4[i / 4][i % 4] : -1;      // (places past the last: zeros of the last one's class)
      seg[i] = i < nv ? seg4[i / 4][i % 4] : seg[i - 1 > 0 ? i - 1 : 0];
      RowVec<TIn, VEC>::load((r < 0 ? (const TIn *)a.zero_row : (const TIn *)a.vals + (size_t)r * a.D) + c, v[i]);
    }
    unsigned word[NR][NQ];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int q = 0; q < NQ; ++q) word[i][q] = 0;
    if (masked) {
#pragma unroll
      for (int i = 0; i < NR; ++i)
        if (i == NR - 1 || seg[i + 1 < NR ? i + 1 : i] != seg[i]) {
#pragma unroll
          for (int q = 0; q < NQ; ++q) word[i][q] = mask_word(a.ymask, seg[i], a.D, c + 4 * q);
        }
    }
    if (r0 == st * GROUP) begun = seg[0] == before;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
#pragma unroll
      for (int j = 0; j < VEC; ++j) acc[j] += v[i][j];
      const bool ends = (i == NR - 1 ? after : seg[i + 1 < NR ? i + 1 : i]) != seg[i];
      if (ends || (i == NR - 1 && last)) {
        if (begun || !ends) {
          float *p = a.carry + ((size_t)st * 2 + (begun ? 0 : 1)) * a.D + c;
#pragma unroll
          for (int q = 0; q < NQ; ++q) store4<float>(p + 4 * q, acc + 4 * q);
        } else {
#pragma unroll
          for (int q = 0; q < NQ; ++q) store_masked4<TOut>((TOut *)a.out + (size_t)seg[i] * a.D + c + 4 * q, acc + 4 * q, masked, word[i][q], c + 4 * q);
        }
        begun = false;
#pragma unroll
        for (int j = 0; j < VEC; ++j) acc[j] = 0.f;
      }
    }
    if (last) break;
    r0 += NR;
  }
}
// The pool's gradient per class: the same sums, of rows of a [G, H] fp32 table that are read by far more often than there are rows. A
// class's places are in the order of their graphs, and most classes lie in every graph of their state, once; so the table is
// made three times, row g of window w the sum of rows g .. g + w - 1 (w = 1, 4, 16), and a run of consecutive graphs is read sixteen
// of them at a time, four or one: 11 reads for 64 places of 16 transformer states, 16 of as many residual networks'. A wave takes 64
// places, a row's columns over its lanes, so that what it reads next is the same for all of them; eight reads are in flight. us of
// class_sum_kernel / of this kernel and the tables, H = 256: 4.35 M places 282 / 151 + 9, 15.9 M 979 / 857 + 14 (the classes of an
// episode's states are shared, and the tables of 8 states are more than an XCD's L2); H = 128, 351 k places 22 / 28 + 7: below
// 4096 places a compute unit a wave's chain of reads is the longer way. 4.35 M places are bound by the instructions of a read, 15.9 M by
// the 6 GB that come from behind the L2. For H = 256 alone, where a row is 16 bytes a lane. There short runs cost nothing, us of a backward pass
// of one round by class sums / by windows, graphs alike in runs of 1, 4, 16: 1.1 M places 245 / 239, 245 / 205, 246 / 197, 4.3 M 493 / 445,
// 490 / 325, 489 / 306, 7.7 M 868 / 765, 867 / 548, 863 / 504. Of narrower rows a wave reads half and a quarter as much at a time: H = 128, 4.3 M
// places in runs of 1, 7, 16 246 / 313, 245 / 245, 243 / 167, in a minibatch's own runs, five rounds, 845 / 842, 632 / 625, 809 / 809; H = 64
// 158 / 281, 157 / 214, 156 / 135 and 523 / 542, 411 / 435, 510 / 529. (256 places a wave 202 in place of 155, an XCD to consecutive places 215: the states' shares differ.
// The columns in two slices, on four XCDs each, 236 and 833, in four 440 and 1602, though the 6 GB become 2: a read costs
// the same instructions for fewer columns.)
constexpr int kWindows = 3;                    // of 1, 4 and 16 graphs
constexpr int kWindowStrip = 8;                // rows a thread makes, of four columns
// rows[w][g, :] = sum of dx[g .. g + 4^w - 1, :], each divided by its graph's node count for the mean readout (rows past the
// last graph count as zeros: no run reads such a sum)
__global__ __launch_bounds__(256) void pool_windows_kernel(const float *dx, const int32_t *graph_node_ptr, int mean, int64_t G, int H, float *rows) {
  constexpr int N = kWindowStrip + 15;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, strip = i / (H / 4), g0 = strip * kWindowStrip;
  const int c = (int)(i - strip * (H / 4)) * 4;
  if (g0 >= G) return;
  f32x4 x[N];
#pragma unroll
  for (int k = 0; k < N; ++k) x[k] = *(const f32x4 *)(dx + (size_t)(g0 + k < G ? g0 + k : G - 1) * H + c);
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int64_t g = g0 + k < G ? g0 + k : G - 1;
    if (mean) {
      const int n = graph_node_ptr[g + 1] - graph_node_ptr[g];
      const float d = (float)(n > 1 ? n : 1);
#pragma unroll
      for (int j = 0; j < 4; ++j) x[k][j] /= d;
    }
    if (g0 + k >= G) x[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const size_t table = (size_t)G * H;
#pragma unroll
  for (int k = 0; k < kWindowStrip; ++k)
    if (g0 + k < G) *(f32x4 *)(rows + (size_t)(g0 + k) * H + c) = x[k];
#pragma unroll
  for (int k = 0; k + 3 < N; ++k) x[k] = (x[k] + x[k + 1]) + (x[k + 2] + x[k + 3]);
#pragma unroll
  for (int k = 0; k < kWindowStrip; ++k) {
    if (g0 + k >= G) break;
    *(f32x4 *)(rows + table + (size_t)(g0 + k) * H + c) = x[k];
    *(f32x4 *)(rows + 2 * table + (size_t)(g0 + k) * H + c) = (x[k] + x[k + 4]) + (x[k + 8] + x[k + 12]);
  }
}
// a.vals: the window tables, a.perm: the places' graphs; a.group: kPoolPlaces
constexpr int kPoolPlaces = 64;                // places a wave takes, one a lane
constexpr int kPoolWidth = 256;                // columns of a row, four a lane
template <typename TOut>
__global__ __launch_bounds__(256) void pool_class_sum_kernel(const ClassSumArgs a, const int64_t G) {
  constexpr int H = kPoolWidth, FLY = 8;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t st = (int64_t)blockIdx.x * 4 + wave;
  const int64_t p0 = st * kPoolPlaces;
  if (p0 >= a.n_rows) return;
  const int n = a.n_rows - p0 < kPoolPlaces ? (int)(a.n_rows - p0) : kPoolPlaces;
  const int c = lane * 4;
  const float *table = (const float *)a.vals + c;
  const bool masked = a.ymask != nullptr;
  const int64_t place = p0 + (lane < n ? lane : n - 1);
  const int g = a.perm[place], s = a.seg[place];
  const int seg_before = a.seg[p0 > 0 ? p0 - 1 : 0], seg_behind = a.seg[p0 + n < a.n_rows ? p0 + n : a.n_rows - 1];
  const int before = p0 > 0 ? seg_before : -1, behind = p0 + n < a.n_rows ? seg_behind : -1;
  bool begun = __builtin_amdgcn_readfirstlane(s) == before;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int gl = __shfl_up(g, 1), sl = __shfl_up(s, 1);
  const unsigned long long in = n < 64 ? (1ull << n) - 1 : ~0ull;
  const unsigned long long starts = __ballot(lane == 0 || s != sl || g != gl + 1) & in;
  // the lane's run [first, end), what of it goes by sixteen, by four, by one, and whether this place begins such a read
  const unsigned long long upto = lane < 63 ? (2ull << lane) - 1 : ~0ull;
  const int first = 63 - __builtin_clzll((starts & upto) | 1ull);
  const unsigned long long later = starts & ~upto;
  const int end = later ? __builtin_ctzll(later) : n, len = end - first, o = lane - first;
  const int n16 = len & ~15, n4 = n16 + ((len - n16) & ~3);
  const int w = o < n16 ? 2 : o < n4 ? 1 : 0;
  const bool head = lane < n && (w == 2 ? (o & 15) == 0 : w == 1 ? ((o - n16) & 3) == 0 : true);
  const unsigned row = (unsigned)(w * G) + (unsigned)g;        // of the three tables, one behind the other
  // (a read is its class's last one where the place behind it is another class's)
  const int next = __shfl_down(s, 1), of_next = lane + 1 < n ? next : behind;
  const unsigned long long ends = __ballot(lane < n && s != of_next);
  unsigned long long todo = __ballot(head);
  int l = 0;
  while (todo) {
    f32x4 v[FLY];
    unsigned word[FLY], r[FLY];
    int of[FLY];
    const int m = __popcll(todo) < FLY ? __popcll(todo) : FLY;
    unsigned last = 0;                           // bit i: read i is its class's last
#pragma unroll
    for (int i = 0; i < FLY; ++i) {              // (past the end the last read again, left out of the sums)
      l = todo ? __builtin_ctzll(todo) : l;
      todo &= todo - 1;
      r[i] = (unsigned)__builtin_amdgcn_readlane((int)row, l);
      of[i] = __builtin_amdgcn_readlane(s, l);
      const int stop = todo ? __builtin_ctzll(todo) : n;       // the read's places: l .. stop - 1
      last |= (unsigned)((ends >> (stop - 1)) & 1) << i;
    }
    // (the mask bits before the rows: loads return in order, so no wait for them later stands behind a class's store)
    if (masked) {
#pragma unroll
      for (int i = 0; i < FLY; ++i)
        if ((last >> i) & 1) word[i] = mask_word(a.ymask, of[i], H, c);
    }
#pragma unroll
    for (int i = 0; i < FLY; ++i) v[i] = *(const f32x4 *)(table + (size_t)r[i] * H);
#pragma unroll
    for (int i = 0; i < FLY; ++i) {
      if (i >= m) break;
      acc += v[i];
      const bool complete = (last >> i) & 1, group_ends = i == m - 1 && !todo;
      if (complete || group_ends) {
        if (begun || !complete) {
          *(f32x4 *)(a.carry + ((size_t)st * 2 + (begun ? 0 : 1)) * H + c) = acc;
        } else {
          float y[4] = {acc[0], acc[1], acc[2], acc[3]};
          store_masked4<TOut>((TOut *)a.out + (size_t)of[i] * H + c, y, masked, masked ? word[i] : 0u, c);
        }
        begun = false;
        acc = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
}
// The classes in several pieces. A wave looks at kCarryGroups groups of places, one per lane, and for those
// whose last class begins there and goes on adds up its pieces, one class after the other (of 64 groups: 70 us
// however small the level): D / 4 lanes a piece, the wave's
// 256 / D lane groups every 256 / D-th of them, eight in flight each, added in group order. A class of more than two such rounds
// -- a sender that many graphs share, with edges to many receivers -- is added up by the block's four waves together, in wave order:
// fp32, H = 128, 125 k nodes of 110 inception networks, where one wave took 44 us of each launch, 16.
constexpr int kCarryGroups = 4, kCarryFly = 8;
template <typename TOut>
__global__ __launch_bounds__(256) void class_sum_carried_kernel(const ClassSumArgs a) {
  touch_args(a);
  __shared__ int wide_seg[4 * kCarryGroups], wide_group[4 * kCarryGroups], n_wide;
  __shared__ __align__(16) f32x4 wide_sum[4][64];
  const int NR = a.group;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t block0 = (int64_t)blockIdx.x * 4 * kCarryGroups, st0 = block0 + wave * kCarryGroups, mine = st0 + lane;
  if (threadIdx.x == 0) n_wide = 0;
  int seg = -1;
  bool starts = false;
  if (lane < kCarryGroups && (mine + 1) * NR < a.n_rows) {
    seg = a.seg[mine * NR + NR - 1];
    starts = a.seg[(mine + 1) * NR] == seg && a.ptr[seg] >= mine * NR;
  }
  __syncthreads();
  const int lpr = a.D / 4, parts = 64 / lpr, c = (lane % lpr) * 4, part = lane / lpr;
  // pieces first, first + step, .. of the class that begins in group st: this group's last, then first ones
  auto pieces = [&](int64_t st, int64_t n, int first, int step) {
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int64_t t = first; t < n; t += kCarryFly * step) {
      f32x4 v[kCarryFly];
#pragma unroll
      for (int i = 0; i < kCarryFly; ++i) {
        const int64_t ti = t + i * step < n ? t + i * step : t;
        v[i] = *(const f32x4 *)(a.carry + ((size_t)(st + ti) * 2 + (ti == 0 ? 1 : 0)) * a.D + c);
      }
#pragma unroll
      for (int i = 0; i < kCarryFly; ++i)
        if (t + i * step < n) sum += v[i];
    }
    f32x4 y;                                     // in the lanes of part 0
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      y[j] = sum[j];
      for (int p = 1; p < parts; ++p) y[j] += __shfl(sum[j], (lane + p * lpr) & 63);
    }
    return y;
  };
  auto put = [&](int s, f32x4 sum) {
    float y[4] = {sum[0], sum[1], sum[2], sum[3]};
    store_masked4<TOut>((TOut *)a.out + (size_t)s * a.D + c, y, a.ymask != nullptr, a.ymask ? mask_word(a.ymask, s, a.D, c) : 0u, c);
  };
  for (unsigned long long todo = __ballot(starts); todo; todo &= todo - 1) {
    const int l = __builtin_ctzll(todo);
    const int s = __shfl(seg, l);
    const int64_t st = st0 + l, n = ((int64_t)a.ptr[s + 1] + NR - 1) / NR - st;
    if (n > 2 * kCarryFly * parts) {
      if (lane == 0) {
        const int k = atomicAdd(&n_wide, 1);
        wide_seg[k] = s;
        wide_group[k] = (int)(st - block0);
      }
      continue;
    }
    const f32x4 y = pieces(st, n, part, parts);
    if (part == 0) put(s, y);
  }
  __syncthreads();
  for (int k = 0; k < n_wide; ++k) {
    const int s = wide_seg[k];
    const int64_t st = block0 + wide_group[k], n = ((int64_t)a.ptr[s + 1] + NR - 1) / NR - st;
    const f32x4 y = pieces(st, n, wave * parts + part, 4 * parts);
    if (part == 0) wide_sum[wave][lane] = y;
    __syncthreads();
    if (wave == 0 && part == 0) put(s, (wide_sum[0][lane] + wide_sum[1][lane]) + (wide_sum[2][lane] + wide_sum[3][lane]));
    __syncthreads();
  }
}
