// Fused two-layer ReLU MLP over a tile of rows, both layers on the matrix cores, the hidden
// activation never leaving the block. One kernel template serves the three learned transforms of
// the encoder (Section 3.4):
//   EMBED  rows = nodes,  x = [sum of incoming edge attrs | one-hot op | dense attrs]   -> h0
//          (the sum over the node's in-edges is formed in the prologue)
//   EDGE   rows = edges in receiver order, x = [h_sender | h_receiver | edge attrs]
//          -> ReLU MLP -> summed per receiver (the message-passing sum)                 -> agg
//   NODE   rows = nodes,  x = [h | agg]                                                 -> h'
//
// A tile is 32 rows: one wave's (mlp2_wave_tile, the one-launch encoders) or, split by output features, that
// of a block of H / 32 waves (mlp2_split_kernel). Both layers are computed transposed (features x rows: the weights are
// the A operand, the gathered input rows the B operand), so layer 1's accumulator layout (lane = row, registers = features) is, after ReLU
// and conversion, the B-operand layout of layer 2; layer 2's accumulators have lane = row as
// well, so a row leaves as register quads and the per-receiver sum runs across adjacent lanes.
// Weights are pre-arranged in the per-lane fragment order (arrange_weights_kernel in the
// runtime), so every weight fragment is one coalesced 1 KB load per wave.
#pragma once
#include "mma.hip.h"
#include "segsum.hip.h"

enum { KIND_EMBED = 0, KIND_EDGE = 1, KIND_NODE = 2 };

struct Mlp2Args {
  int64_t n_rows;
  int64_t n_blocks;        // number of tiles
  const void *W1s, *W2s;   // fragment-ordered weights, operand type (mlp2_split3_kernel: their parts)
  const float *W1, *W2;    // the same as they are given, [in, H] (mlp2_split3_kernel alone)
  const float *b1, *b2;    // [H]
  int nslab1;              // slabs of layer 1's (zero-padded) input width
  const void *h;           // [N, H] operand type            (EDGE, NODE)
  const void *agg;         // [N, H] operand type            (NODE)
  const int32_t *agg_src;  // [N] NODE: the row of agg that holds a node's received sum, -1 for a node without
                           //   in-edges (the message kernels never write its row: zeros are read in its place);
                           //   nullptr: every node reads its own row
  const int32_t *in_ptr;   // [N + 1]                        (all kinds)
  const int32_t *in_src;   // [E]                            (EDGE)
  const int32_t *in_dst;   // [E]                            (EDGE)
  const float *edge_feat;  // [E, De] receiver order         (EDGE, EMBED)
  const int32_t *node_op;  // [N]                            (EMBED)
  const float *node_dense; // [N, Dd]                        (EMBED)
  int De, Tn, Dd;
  const void *W1x;         // EMBED: fragment-ordered fp32 rows of W1 for [edge-attr sum | dense attrs]
  int nslabx;              // EMBED: its slabs
  const float *table;      // EMBED: [Tn, H] fp32 rows of W1 for the one-hot op type
  const void *zero_row;    // 1 KB of zeros (source of rows that are absent)
  void *agg0;              // EMBED: first of n_agg received-sum buffers [N, H], agg_stride bytes apart;
  size_t agg_stride;       //        the embed kernel zeroes their rows of nodes without in-edges, which
  int n_agg;               //        the message kernels never write (0 when the readers go by agg_src)
  void *out;               // [N, H] operand type
  void *z1;                // kernels instantiated to keep the forward for the backward pass: the hidden
  uint16_t *z1mask;        //   activation relu(z1) [rows, H] operand type (an operand of the weight gradient)
  uint16_t *ymask;         //   and the ReLU masks of z1 and of y, which is all the backward through the MLP
                           //   needs of the forward: [tiles][H / 32][64 lanes] words, bit r of lane l =
                           //   accumulator register r of that lane (its row, its feature block) > 0. Tiles are
                           //   the kernel's wave tiles: edge tiles, or 32 consecutive nodes
  float *carry;            // [n_tiles, 2, H]                (EDGE)
  const int32_t *tile_ptr; // [n_tiles + 1] first edge of each edge tile (EDGE)
  int64_t n_tiles;         //                                (EDGE)
  // kernels instantiated for a level whose size the host does not know: its counts on the device, and the row
  // of h of each edge's receiver (EDGE; in_src: of its sender) or of each node (NODE)
  const unsigned long long *level_counts;
  const int32_t *h_row;    // (the split kernels: nullptr, or the same of a level whose rows of h are the classes below)
};
// Counts of a level in one word (what the blocks that make it take at once from one counter)
constexpr int kCountBits = 21;
__device__ __forceinline__ int32_t level_classes(unsigned long long v) { return (int32_t)(v & ((1u << kCountBits) - 1)); }
__device__ __forceinline__ int32_t level_edges(unsigned long long v) { return (int32_t)(v >> kCountBits & ((1u << kCountBits) - 1)); }
__device__ __forceinline__ int32_t level_tiles(unsigned long long v) { return (int32_t)(v >> 2 * kCountBits); }
template <bool LEVEL, bool EDGES>
__device__ __forceinline__ Mlp2Args of_level(Mlp2Args a) {
  if constexpr (LEVEL) {
    const unsigned long long v = *a.level_counts;
    a.n_rows = __builtin_amdgcn_readfirstlane(EDGES ? level_edges(v) : level_classes(v));
    a.n_tiles = __builtin_amdgcn_readfirstlane(level_tiles(v));
  }
  return a;
}

// Raw (fp32) piece of one row's trailing attributes that lane group g feeds to slab `ts` of the
// tail: columns [ts*2V + g*V, +V) of a row of `width` floats (width a multiple of 4), zeros
// beyond. The loads are unconditional (out-of-range pieces re-read the row's first columns and
// are zeroed afterwards) so that no branch or early wait separates them from other loads.
template <int V>
struct TailRaw {
  f32x4 q[V / 4];
};
// (the two halves -- request, then zeroing at the point of use -- are separate so that a caller
// can request a tile ahead without the zeroing's wait landing next to the request)
template <int V>
__device__ __forceinline__ TailRaw<V> request_tail(const float *rowp, int width, int ts, int g) {
  TailRaw<V> r;
#pragma unroll
  for (int i = 0; i < V / 4; ++i) {
    const int k = ts * 2 * V + g * V + 4 * i;
    r.q[i] = *(const f32x4 *)(rowp + (k + 4 <= width ? k : 0));
  }
  return r;
}
template <int V>
__device__ __forceinline__ TailRaw<V> zero_tail_beyond(TailRaw<V> r, int width, int ts, int g) {
#pragma unroll
  for (int i = 0; i < V / 4; ++i)
    if (ts * 2 * V + g * V + 4 * i + 4 > width) r.q[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  return r;
}
template <int V>
__device__ __forceinline__ TailRaw<V> load_tail(const float *rowp, int width, int ts, int g) {
  return zero_tail_beyond<V>(request_tail<V>(rowp, width, ts, g), width, ts, g);
}
template <typename T>
__device__ __forceinline__ typename Operand<T>::vec tail_to_operand(const TailRaw<Operand<T>::V> &r);
template <>
__device__ __forceinline__ f32x4 tail_to_operand<float>(const TailRaw<4> &r) { return r.q[0]; }
template <>
__device__ __forceinline__ bf16x8 tail_to_operand<bf16_t>(const TailRaw<8> &r) {
  return pack_bf16x8(r.q[0][0], r.q[0][1], r.q[0][2], r.q[0][3], r.q[1][0], r.q[1][1], r.q[1][2], r.q[1][3]);
}

template <typename T, int H>
__device__ __forceinline__ void mma_slab(const typename Operand<T>::vec *wp,
                                         const typename Operand<T>::vec &x, f32x16 *acc) {
#pragma unroll
  for (int mb = 0; mb < H / 32; ++mb) {
    typename Operand<T>::vec w = wp[mb * 64];
    Operand<T>::mma(w, x, acc[mb]);
  }
}

// Receivers of the edges of a wave tile (edges [e0, e0 + nv), nv <= 32, from the packer's tile
// table), plus those of the edges just outside it.
struct EdgeTileMeta {
  int dst;      // receiver of this lane's edge (lanes 32..63 mirror 0..31; lanes past the tile's
                // last edge repeat it)
  int prev_d;   // receiver of the edge before the tile, -1 if there is none
  int next_d;   // receiver of the edge after the tile, -1 if there is none
};
__device__ __forceinline__ EdgeTileMeta load_edge_meta(const int32_t *in_dst, int64_t n_rows, int64_t e0, int nv,
                                                       int l32) {
  EdgeTileMeta m;
  m.dst = in_dst[e0 + (l32 < nv ? l32 : nv - 1)];
  m.prev_d = e0 > 0 ? in_dst[e0 - 1] : -1;
  m.next_d = e0 + nv < n_rows ? in_dst[e0 + nv] : -1;
  return m;
}

// The mask bits (value > 0) of this lane's 16 registers of one accumulator block.
__device__ __forceinline__ uint16_t lane_mask_bits(const f32x16 &acc) {
  uint32_t m = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) m |= (acc[r] > 0.f ? 1u : 0u) << r;
  return (uint16_t)m;
}

// Per-receiver sum of a wave tile of messages held as features x rows accumulators (lane = edge,
// registers = features; edges are in receiver order, so a receiver's edges are adjacent lanes).
// ReLU, then a segmented suffix sum across lanes by doubling: after the step of distance d a lane
// holds the sum of its own and the next 2d - 1 edges of its receiver, so the first lane of every
// receiver ends with the receiver's total after ceil(log2(longest run)) steps (none at all when
// every receiver of the tile has one in-edge, one when none has more than two). The order of
// the additions is fixed by the positions in the tile alone. The total held by the first lane of
// each run then goes to out[receiver] (whole rows, through the staging buffer) when the run lies
// inside the tile, to
// carry[wt][0] when it began before the tile, to carry[wt][1] when it goes on after it (a run
// covering the whole tile and open on both sides counts as begun before); segsum_fixup adds the
// carried pieces in tile order.
struct EdgeRoute {
  int dsel;             // row this lane's total goes to, -1 = none
  bool to_c0, to_c1;    // ... or the carry it goes to
};
template <int NB>
__device__ __forceinline__ EdgeRoute edge_run_sums(f32x16 (&acc)[NB], const EdgeTileMeta &m, int nv, int lane) {
  const int l32 = lane & 31;
  const bool valid = l32 < nv;                                  // nv >= 1
  const int up = __shfl_up(m.dst, 1);                           // lane 32 reads lane 31, but is a head anyway
  const bool head = valid && (l32 == 0 || up != m.dst);
  const uint64_t heads = ((uint64_t)(uint32_t)__ballot(head)) | ((uint64_t)1 << nv);
  // number of edges after this one that have the same receiver and lie in the tile
  const int rem = valid ? __builtin_ctzll(heads >> (l32 + 1)) : 0;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nb][r] = relu_f32(acc[nb][r]);
  // (the lane's partner value enters through a product with 0 or 1: one fused multiply-add per
  // register instead of a select and an add; the values are finite sums of ReLU outputs)
  if (__any(rem >= 1)) {
    // first step, the only one for in-degrees up to 2: the neighbouring lane's value by a
    // wave-wide shift (no LDS traffic)
    const float takef = rem >= 1 ? 1.f : 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        // (a copy first: bit-casting the vector-element lvalue itself reads element 0)
        const float v = acc[nb][r];
        const float t = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, false));
        acc[nb][r] = fmaf(t, takef, v);
      }
  }
  for (int d = 2; __any(rem >= d); d <<= 1) {
    const float takef = rem >= d ? 1.f : 0.f;
    const int from = ((lane + d) & 63) << 2;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float v = acc[nb][r];
        const float t = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(v)));
        acc[nb][r] = fmaf(t, takef, v);
      }
      // one block's exchanges at a time: all of them in flight at once would hold 16 * NB more
      // registers than the callers that keep a next tile's rows in flight can spare
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const bool ends_tile = l32 + rem == nv - 1;
  EdgeRoute e;
  e.to_c0 = head && l32 == 0 && m.prev_d == m.dst;
  e.to_c1 = head && !e.to_c0 && ends_tile && m.next_d == m.dst;
  e.dsel = (head && !e.to_c0 && !e.to_c1) ? m.dst : -1;
  return e;
}
template <typename T, int H>
__device__ __forceinline__ void edge_tile_sum(f32x16 (&acc)[H / 32], const EdgeTileMeta &m, int64_t wt, int nv,
                                               int lane, T *out, float *carry, char *stage) {
  const EdgeRoute e = edge_run_sums<H / 32>(acc, m, nv, lane);
  store_rows_via_lds<T, H, false>(acc, stage, lane, [&](int r) -> T * {
    const int d = __shfl(e.dsel, r);
    return d >= 0 ? out + (size_t)d * H : nullptr;
  });
  if (e.to_c0 || e.to_c1) {
    const int64_t crow = wt * 2 + (e.to_c1 ? 1 : 0);
#pragma unroll
    for (int nb = 0; nb < H / 32; ++nb) store_tile_rows<float, H>(carry, crow, true, nb, lane >> 5, acc[nb]);
  }
}

// Node-update layer input (Section 3.4) of one node, without its one-hot block: column k of
// [sum of the node's incoming edge attributes (De) | dense attributes (Dd)], zero beyond. The
// in-edges are the node's contiguous receiver-order range [e0, e1) and are added in that order;
// the first two are requested together (most nodes of a computation graph have one or two).
struct EmbedRow {
  int op, e0, e1;
  const float *dense;
};
__device__ __forceinline__ EmbedRow load_embed_row(const int32_t *node_op, const int32_t *in_ptr,
                                                   const float *node_dense, int Dd, int64_t row) {
  EmbedRow r;
  r.op = node_op[row];
  r.e0 = in_ptr[row];
  r.e1 = in_ptr[row + 1];
  r.dense = node_dense + (size_t)row * Dd;
  return r;
}
// four consecutive columns k0 .. k0+3 (k0 a multiple of 4, as are De and the row stride)
__device__ __forceinline__ f32x4 embed_columns(const EmbedRow &r, const float *edge_feat, int De, int Dd, int k0) {
  f32x4 x = {0.f, 0.f, 0.f, 0.f};
  if (k0 < De) {
    const int n = r.e1 - r.e0;
    const float *p = edge_feat + (size_t)r.e0 * De + k0;
    f32x4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = v0;
    if (n > 0) v0 = *(const f32x4 *)p;
    if (n > 1) v1 = *(const f32x4 *)(p + De);
    x = v0;
    if (n > 1) x += v1;
    for (int e = 2; e < n; ++e) x += *(const f32x4 *)(p + (size_t)e * De);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (k0 + j < De + Dd) x[j] = r.dense[k0 + j - De];
  }
  return x;
}

// The same four columns with every load under no condition (an absent edge, a column of the other
// kind or past the last one reads a row of zeros through the load address; up to four in-edges,
// the rest in a loop), so that no load waits for another. Sums in the order of embed_columns
// (adding the zeros changes nothing).
__device__ __forceinline__ f32x4 embed_columns_ahead(const EmbedRow &r, const float *edge_feat, const float *zeros,
                                                     int De, int Dd, int k0) {
  const int n = k0 < De ? r.e1 - r.e0 : 0;
  const float *p = edge_feat + (size_t)r.e0 * De + k0;
  f32x4 v[4], d;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = *(const f32x4 *)(e < n ? p + (size_t)e * De : zeros);
#pragma unroll
  for (int j = 0; j < 4; ++j) d[j] = *(k0 >= De && k0 + j < De + Dd ? r.dense + (k0 + j - De) : zeros);
  f32x4 x = v[0];
#pragma unroll
  for (int e = 1; e < 4; ++e) x += v[e];
  for (int e = 4; e < n; ++e) x += *(const f32x4 *)(p + (size_t)e * De);
  x += d;
  return x;
}

// EMBED: zero rows of the received-sum buffers for the tile's nodes without in-edges (`no_in`:
// this lane's node, lane = row l % 32), whole rows, 16 bytes per lane.
template <typename T, int H>
__device__ __forceinline__ void zero_source_rows(const Mlp2Args &a, int64_t row0, int nv, bool no_in, int lane) {
  constexpr int LPR = H * (int)sizeof(T) / 16, RPI = 64 / LPR;
  if (a.n_agg == 0 || !__any(no_in)) return;
  const int flag = no_in ? 1 : 0;
#pragma unroll
  for (int k = 0; k < 32 / RPI; ++k) {
    const int r = k * RPI + lane / LPR;
    const bool z = __shfl(flag, r) != 0 && r < nv;
    if (z)
      for (int i = 0; i < a.n_agg; ++i)
        *(f32x4 *)((char *)a.agg0 + i * a.agg_stride + ((size_t)(row0 + r) * H) * sizeof(T) + (lane % LPR) * 16) =
            f32x4{0.f, 0.f, 0.f, 0.f};
  }
}

// One wave tile: rows [row0, row0 + nv) (nv in 1..32; for EDGE the edges of tile `wt` of the
// tile table in use), on one wave (the one-launch encoders), staged out through `stage` (RowStage<T, H>::BYTES, private to the wave).
// T1 = operand type of layer 1 (its input rows and W1), T = operand type of layer 2 and of the
// stored activations. They differ only for EMBED in bf16 mode, whose first layer stays in fp32:
// its inputs (log2 shape attributes up to 12, sums of edge attributes) are large enough for bf16
// weight rounding to dominate the error of the whole encoder.
template <typename T1, typename T, int H, int KIND>
__device__ __forceinline__ void mlp2_wave_tile(const Mlp2Args &a, const int64_t row0, const int nv, const int64_t wt,
                                               char *stage, const int lane) {
  using Opd = Operand<T>;
  using vec = typename Opd::vec;
  constexpr int V = Opd::V, SL = 2 * V, MB = H / 32, HS = H / SL;
  using Opd1 = Operand<T1>;
  using vec1 = typename Opd1::vec;
  constexpr int V1 = Opd1::V, SL1 = 2 * V1;
  static_assert(KIND == KIND_EMBED || sizeof(T1) == sizeof(T), "only EMBED mixes operand types");
  const int l32 = lane & 31, g = lane >> 5;
  const int64_t row = row0 + (l32 < nv ? l32 : nv - 1);          // clamp loads; stores are guarded

  // ---------------- layer 1: acc1[mb] = (W1^T x^T) tile, features x rows, bias pre-loaded
  f32x16 acc1[MB];
  if constexpr (KIND != KIND_EMBED) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc1[mb][r] = a.b1[32 * mb + acc_row(r, g)];
  }
  const vec1 *W1 = (const vec1 *)(KIND == KIND_EMBED ? a.W1x : a.W1s) + lane;

  if constexpr (KIND == KIND_EDGE || KIND == KIND_NODE) {
    // both H-wide parts of the input row are requested up front (one exposed latency instead
    // of one per slab); the weight fragments are requested one slab ahead of their MFMAs
    const T *pa, *pb;
    if constexpr (KIND == KIND_EDGE) {
      pa = (const T *)a.h + (size_t)a.in_src[row] * H + g * V;
      pb = (const T *)a.h + (size_t)a.in_dst[row] * H + g * V;
    } else {
      pa = (const T *)a.h + (size_t)row * H + g * V;
      const int64_t ar = a.agg_src ? (int64_t)a.agg_src[row] : row;
      pb = ar < 0 ? (const T *)a.zero_row + g * V : (const T *)a.agg + (size_t)ar * H + g * V;
    }
    vec xa[HS], xb[HS];
#pragma unroll
    for (int s = 0; s < HS; ++s) xa[s] = *(const vec *)(pa + s * SL);
#pragma unroll
    for (int s = 0; s < HS; ++s) xb[s] = *(const vec *)(pb + s * SL);
    [[maybe_unused]] TailRaw<V> xt;
    if constexpr (KIND == KIND_EDGE) xt = load_tail<V>(a.edge_feat + (size_t)row * a.De, a.De, 0, g);
    vec wc[MB], wn[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) wc[mb] = W1[mb * 64];
#pragma unroll
    for (int s = 0; s < 2 * HS; ++s) {
      if (s + 1 < a.nslab1) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) wn[mb] = W1[((size_t)(s + 1) * MB + mb) * 64];
      }
      const vec x = s < HS ? xa[s < HS ? s : 0] : xb[s < HS ? 0 : s - HS];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) Opd::mma(wc[mb], x, acc1[mb]);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) wc[mb] = wn[mb];
    }
    if constexpr (KIND == KIND_EDGE) {
      const float *xe = a.edge_feat + (size_t)row * a.De;
      for (int s = 2 * HS; s < a.nslab1; ++s) {                 // edge attributes
        const vec x = tail_to_operand<T>(s == 2 * HS ? xt : load_tail<V>(xe, a.De, s - 2 * HS, g));
        if (s > 2 * HS) {
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) wc[mb] = W1[((size_t)s * MB + mb) * 64];
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) Opd::mma(wc[mb], x, acc1[mb]);
      }
    }
  } else {
    // The one-hot block of the input selects one row of W1: that row (plus the bias) is the
    // accumulators' starting value, read as four consecutive features per load, and only the
    // remaining [edge-attr sum | dense attrs] columns go through the matrix cores (in fp32).
    const EmbedRow er = load_embed_row(a.node_op, a.in_ptr, a.node_dense, a.Dd, row);
    const float *trow = a.table + (size_t)er.op * H + 4 * g;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 t = *(const f32x4 *)(trow + 32 * mb + 8 * q);
        const f32x4 b = *(const f32x4 *)(a.b1 + 32 * mb + 8 * q + 4 * g);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc1[mb][4 * q + j] = t[j] + b[j];
      }
    static_assert(V1 == 4, "the embed MLP's first layer uses fp32 operands");
    for (int s = 0; s < a.nslabx; ++s) {
      const vec1 x = embed_columns(er, a.edge_feat, a.De, a.Dd, s * SL1 + g * V1);
      mma_slab<T1, H>(W1 + (size_t)s * MB * 64, x, acc1);
    }
  }

  // ---------------- layer 2, transposed as well: acc2[nb] = (W2^T relu(z1)^T) tile, features x
  // rows, bias pre-loaded. Lane = row, and a lane's register quads are four consecutive features
  // of its row: 8- or 16-byte stores, and for EDGE a per-receiver sum across adjacent lanes.
  f32x16 acc2[MB];
#pragma unroll
  for (int nb = 0; nb < MB; ++nb) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc2[nb][r] = a.b2[32 * nb + acc_row(r, g)];
  }
  const vec *W2 = (const vec *)a.W2s + lane;
  {
    constexpr int QB = 32 / SL, NC2 = MB * QB;
    vec wc[MB], wn[MB];
#pragma unroll
    for (int nb = 0; nb < MB; ++nb) wc[nb] = W2[nb * 64];
#pragma unroll
    for (int c = 0; c < NC2; ++c) {
      if (c + 1 < NC2) {
#pragma unroll
        for (int nb = 0; nb < MB; ++nb) wn[nb] = W2[((size_t)(c + 1) * MB + nb) * 64];
      }
      const vec z = relu_operand<T>(acc1[c / QB], c % QB);
#pragma unroll
      for (int nb = 0; nb < MB; ++nb) Opd::mma(wc[nb], z, acc2[nb]);
#pragma unroll
      for (int nb = 0; nb < MB; ++nb) wc[nb] = wn[nb];
    }
  }

  // ---------------- epilogue
  T *out = (T *)a.out;
  if constexpr (KIND != KIND_EDGE) {
    store_rows_via_lds<T, H, true>(acc2, stage, lane, [&](int r) -> T * {
      return r < nv ? out + (size_t)(row0 + r) * H : nullptr;
    });
    if constexpr (KIND == KIND_EMBED) zero_source_rows<T, H>(a, row0, nv, a.in_ptr[row + 1] == a.in_ptr[row], lane);
  } else {
    const EdgeTileMeta m = load_edge_meta(a.in_dst, a.n_rows, row0, nv, l32);
    edge_tile_sum<T, H>(acc2, m, wt, nv, lane, out, a.carry, stage);
  }
}

// Split form, one launch per layer where the persistent kernels do not apply (fp32; small batches in bf16, save
// the levels of a reduced batch that is saved for the backward pass): a block of H / 32 waves takes one
// tile, wave w the 32 output features of block w in both layers. The tile's input rows are gathered
// once, as operand fragments, each wave its share, and shared through LDS, as is relu(z1); a wave
// streams only its own slices of the weights, eight fragments ahead. A tile's chain of dependent
// matrix instructions is H / 32 times shorter: with a wave per tile a launch took 37 us and more in fp32
// at H = 128 however few tiles there were (768 matrix instructions of 64 cycles are 23 us by
// themselves). Same operations in the same order per output: the same bits. Edge kernel, us, a wave
// per tile / split: fp32 H = 128: 158 tiles 39.7 / 14.1, 2278 105 / 88, 13.7 k 479 / 458; H = 256: 158 tiles
// 171 / 35, 2278 514 / 275; H = 64: 200 tiles 16.4 / 12.6, 2278 35.2 / 35.0; bf16 H = 256: 158 tiles 40.8 / 11.6.
// The requests keep their distance only behind scheduling barriers (see the loops): without, fp32 H = 256 edge 971 tiles 111.1 us, with
// 108.6, node 119.5 / 107.7, 1916 tiles 213 / 209 and 202 / 184; H = 64 1915 tiles 25.7 / 23.4 and 23.2 / 21.4; bf16 H = 256 179 tiles 11.8 / 10.7.
template <typename T, int H>
struct SplitTile {
  static constexpr int V = Operand<T>::V, HS = H / (2 * V), MB = H / 32, QB = 32 / (2 * V);
  static constexpr int XBYTES = 2 * HS * 1024, ZBYTES = MB * QB * 1024, SBYTES = MB * BlockStage<T>::BYTES;
  // input fragments; then, in their place, relu(z1) and behind it the waves' output staging
  static constexpr int BYTES = XBYTES > ZBYTES + SBYTES ? XBYTES : ZBYTES + SBYTES;
};
template <typename T1, typename T, int H, int KIND>
__global__ __launch_bounds__(2 * H) void mlp2_split_kernel(const Mlp2Args a) {
  touch_args(a);
  using S = SplitTile<T, H>;
  using Opd = Operand<T>;
  using vec = typename Opd::vec;
  constexpr int V = Opd::V, SL = 2 * V, HS = S::HS, MB = S::MB, QB = S::QB, NC2 = MB * QB;
  constexpr int RING = 8;                                       // weight fragments in flight
  extern __shared__ __align__(16) char smem[];
  const int64_t n_tiles = a.n_blocks, per_xcd = (n_tiles + 7) / 8;
  // consecutive tiles stay on one XCD (blocks are dealt round-robin to the 8 XCDs), so the rows a tile
  // gathers are mostly in that XCD's L2 already
  const int64_t wt = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if ((int64_t)(blockIdx.x / 8) >= per_xcd || wt >= n_tiles) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int64_t row0 = wt * 32;
  int nv;
  if constexpr (KIND == KIND_EDGE) {
    row0 = a.tile_ptr[wt];
    nv = a.tile_ptr[wt + 1] - (int)row0;
  } else {
    nv = a.n_rows - row0 < 32 ? (int)(a.n_rows - row0) : 32;
  }
  const int64_t row = row0 + (l32 < nv ? l32 : nv - 1);         // clamp loads; stores are guarded
  f32x16 acc, b2;                                               // (all loads in front of the barriers: one behind is waited for by itself)
  [[maybe_unused]] EdgeTileMeta meta;
  // ---------------- layer 1
  if constexpr (KIND != KIND_EMBED) {
    const vec *W1 = (const vec *)a.W1s + (size_t)w * 64 + lane;
    const T *pa, *pb;
    if constexpr (KIND == KIND_EDGE) {
      meta = load_edge_meta(a.in_dst, a.n_rows, row0, nv, l32);
      const int32_t *recv = a.h_row ? a.h_row : a.in_dst;
      pa = (const T *)a.h + (size_t)a.in_src[row] * H + g * V;
      pb = (const T *)a.h + (size_t)recv[row] * H + g * V;
    } else {
      pa = (const T *)a.h + (size_t)(a.h_row ? a.h_row[row] : row) * H + g * V;
      const int64_t ar = a.agg_src ? (int64_t)a.agg_src[row] : row;
      pb = ar < 0 ? (const T *)a.zero_row + g * V : (const T *)a.agg + (size_t)ar * H + g * V;
    }
    vec wq[RING];
#pragma unroll
    for (int s = 0; s < RING; ++s) wq[s] = W1[(size_t)s * MB * 64];
    constexpr int MINE = 2 * HS / MB;                           // consecutive slabs of the row this wave fetches
    static_assert(MINE * MB == 2 * HS && HS % MINE == 0 && 2 * HS >= RING, "");
    const int s0 = w * MINE;
    const T *px = s0 < HS ? pa + s0 * SL : pb + (s0 - HS) * SL;
    vec x[MINE];
#pragma unroll
    for (int i = 0; i < MINE; ++i) x[i] = *(const vec *)(px + i * SL);
    [[maybe_unused]] TailRaw<V> xt;
    if constexpr (KIND == KIND_EDGE) xt = load_tail<V>(a.edge_feat + (size_t)row * a.De, a.De, 0, g);
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[r] = a.b1[32 * w + acc_row(r, g)]; b2[r] = a.b2[32 * w + acc_row(r, g)]; }
    vec *xs = (vec *)smem;                                      // [2 HS][64]
#pragma unroll
    for (int i = 0; i < MINE; ++i) xs[(s0 + i) * 64 + lane] = x[i];
    __syncthreads();
    vec x0 = xs[lane];
#pragma unroll
    for (int s = 0; s < 2 * HS; ++s) {
      const vec x1 = xs[(s + 1 < 2 * HS ? s + 1 : 0) * 64 + lane];
      Opd::mma(wq[s % RING], x0, acc);
      if (s + RING < 2 * HS || (KIND == KIND_EDGE && s + RING == 2 * HS)) wq[s % RING] = W1[(size_t)(s + RING) * MB * 64];
      x0 = x1;
      // the compiler otherwise moves every request down to its use, to save registers, and each is waited for by itself
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (KIND == KIND_EDGE) {
      const float *xe = a.edge_feat + (size_t)row * a.De;
      for (int s = 2 * HS; s < a.nslab1; ++s) {                 // edge attributes
        const vec xv = tail_to_operand<T>(s == 2 * HS ? xt : load_tail<V>(xe, a.De, s - 2 * HS, g));
        const vec wv = s == 2 * HS ? wq[(2 * HS) % RING] : W1[(size_t)s * MB * 64];
        Opd::mma(wv, xv, acc);
      }
    }
  } else {
    // (see mlp2_wave_tile: the op type's row of W1 and the bias, then the fp32 columns)
    const f32x4 *W1 = (const f32x4 *)a.W1x + (size_t)w * 64 + lane;
    const EmbedRow er = load_embed_row(a.node_op, a.in_ptr, a.node_dense, a.Dd, row);
    const float *trow = a.table + (size_t)er.op * H + 32 * w + 4 * g;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 t = *(const f32x4 *)(trow + 8 * q);
      const f32x4 b = *(const f32x4 *)(a.b1 + 32 * w + 8 * q + 4 * g), c = *(const f32x4 *)(a.b2 + 32 * w + 8 * q + 4 * g);
#pragma unroll
      for (int j = 0; j < 4; ++j) { acc[4 * q + j] = t[j] + b[j]; b2[4 * q + j] = c[j]; }
    }
    for (int s = 0; s < a.nslabx; ++s) {
      const f32x4 xv = embed_columns(er, a.edge_feat, a.De, a.Dd, s * 8 + g * 4);
      Operand<float>::mma(W1[(size_t)s * MB * 64], xv, acc);
    }
  }
  // ---------------- layer 2
  const vec *W2 = (const vec *)a.W2s + (size_t)w * 64 + lane;
  constexpr int RING2 = NC2 < RING ? NC2 : RING;
  vec wq[RING2];
#pragma unroll
  for (int c = 0; c < RING2; ++c) wq[c] = W2[(size_t)c * MB * 64];
  vec *zs = (vec *)smem;                                        // [NC2][64]
  if constexpr (KIND != KIND_EMBED) __syncthreads();            // (every wave has read its input fragments)
#pragma unroll
  for (int q = 0; q < QB; ++q) zs[(w * QB + q) * 64 + lane] = relu_operand<T>(acc, q);
  acc = b2;
  __syncthreads();
  vec z0 = zs[lane];
#pragma unroll
  for (int c = 0; c < NC2; ++c) {
    const vec z1 = zs[(c + 1 < NC2 ? c + 1 : 0) * 64 + lane];
    Opd::mma(wq[c % RING2], z0, acc);
    if (c + RING2 < NC2) wq[c % RING2] = W2[(size_t)(c + RING2) * MB * 64];
    z0 = z1;
    __builtin_amdgcn_sched_barrier(0);
  }
  // ---------------- epilogue on this wave's 32 features
  T *out = (T *)a.out;
  char *stage = smem + S::ZBYTES + w * BlockStage<T>::BYTES;
  if constexpr (KIND != KIND_EDGE) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = relu_f32(acc[r]);
    store_block_via_lds<T, H>(out, row0, nv, w, lane, acc, stage);
    if constexpr (KIND == KIND_EMBED)
      if (w == 0) zero_source_rows<T, H>(a, row0, nv, a.in_ptr[row + 1] == a.in_ptr[row], lane);
  } else {
    f32x16 one[1] = {acc};
    const EdgeRoute e = edge_run_sums<1>(one, meta, nv, lane);
    store_block_rows_via_lds<T, H>(out, e.dsel, w, lane, one[0], stage);
    if (e.to_c0 || e.to_c1) store_tile_rows<float, H>(a.carry, wt * 2 + (e.to_c1 ? 1 : 0), true, w, g, one[0]);
  }
}

// The same split form for the fp32 edge and node MLPs of H = 128, whose launches were bound by the matrix cores (12.5 k
// cycles of fp32 matrix instructions per wave and edge tile): operands in three bf16 parts (Split3), 4.8 k cycles of
// bf16 ones. Weights come in parts (arrange_weights_kernel: the three parts of a fragment one behind the other),
// input rows and relu(z1) are cut on their way into LDS. Three blocks share a compute unit, each a chain of indices, rows, products
// and stores; from a few tiles per compute unit on the matrix cores are busy about half of the time (two tiles a block, for half the weights'
// way from L2, gained 5 % at 5000 tiles and lost a third at 300). us, fp32 instructions / parts / parts with the
// weights requested four slabs ahead throughout: edge 179 tiles 15.8 / 14.1 / 11.5, 969 38.0 / 27.7 / 25.0, 1918 62.5 / 47.6 / 43.4; node
// 179 tiles - / 12.8 / 10.1, 969 39.0 / 25.1 / 22.8. Relative error of the embeddings against float64, nine states, geometric mean 1.44e-7 / 1.32e-7;
// of the gradients, five states, 2.82e-7 / 2.54e-7; of the heads' gradients of a state, differences of its slots, 104 states,
// 1.01 +- 0.05 times the fp32 instructions'. Rows with a value that has no parts, or that overflow, are computed once more by
// fp32 multiply-adds (0.3 us a launch to look for them). (H = 256: embeddings 1.95e-7 / 1.83e-7, but the heads' gradients of five
// states came out 1.3 times as far off: left on fp32 instructions. H = 64 is left on them too: in a copy of the library parts
// took 76 us per encode of 0.5 k nodes for 80, 141 for 177 of 34 k, 776 for 1106 of 338 k; its error has not been measured.)
template <int H>
struct Split3Tile {
  static constexpr int HS = H / 16, MB = H / 32, NC2 = 2 * MB;
  static constexpr int XBYTES = 2 * HS * 3 * 1024, ZBYTES = NC2 * 3 * 1024, SBYTES = MB * BlockStage<float>::BYTES;
  static constexpr int BYTES = XBYTES > ZBYTES + SBYTES ? XBYTES : ZBYTES + SBYTES;
};
template <int H, int KIND>
__global__ __launch_bounds__(2 * H) void mlp2_split3_kernel(const Mlp2Args a) {
  touch_args(a);
  using S = Split3Tile<H>;
  using vec = bf16x8;
  constexpr int HS = S::HS, MB = S::MB, NC2 = S::NC2, RING = 4;   // slabs of weights in flight, three fragments each
  static_assert(KIND == KIND_EDGE || KIND == KIND_NODE, "");
  extern __shared__ __align__(16) char smem[];
  const int64_t n_tiles = a.n_blocks, per_xcd = (n_tiles + 7) / 8;
  const int64_t wt = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;      // (see mlp2_split_kernel)
  if ((int64_t)(blockIdx.x / 8) >= per_xcd || wt >= n_tiles) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int64_t row0 = wt * 32;
  int nv;
  if constexpr (KIND == KIND_EDGE) {
    row0 = a.tile_ptr[wt];
    nv = a.tile_ptr[wt + 1] - (int)row0;
  } else {
    nv = a.n_rows - row0 < 32 ? (int)(a.n_rows - row0) : 32;
  }
  const int64_t row = row0 + (l32 < nv ? l32 : nv - 1);         // clamp loads; stores are guarded
  auto weights = [&](const void *W, int s) {                    // slab s of this wave's 32 features
    const vec *p = (const vec *)W + ((size_t)s * MB + w) * 192 + lane;
    return Split3{{p[0], p[64], p[128]}};
  };
  auto shared = [&](int s) {                                    // operand s of the tile, shared through LDS
    const vec *p = (const vec *)smem + s * 192 + lane;
    return Split3{{p[0], p[64], p[128]}};
  };
  auto share = [&](int s, const Split3 &x) {
    vec *p = (vec *)smem + s * 192 + lane;
#pragma unroll
    for (int k = 0; k < 3; ++k) p[k * 64] = x.p[k];
  };
  f32x16 acc, corr, b2;
  // ---------------- layer 1
  const float *pa, *pb;
  [[maybe_unused]] EdgeTileMeta meta;
  if constexpr (KIND == KIND_EDGE) {
    meta = load_edge_meta(a.in_dst, a.n_rows, row0, nv, l32);
    const int32_t *recv = a.h_row ? a.h_row : a.in_dst;
    pa = (const float *)a.h + (size_t)a.in_src[row] * H + g * 8;
    pb = (const float *)a.h + (size_t)recv[row] * H + g * 8;
  } else {
    pa = (const float *)a.h + (size_t)(a.h_row ? a.h_row[row] : row) * H + g * 8;
    const int64_t ar = a.agg_src ? (int64_t)a.agg_src[row] : row;
    pb = ar < 0 ? (const float *)a.zero_row + g * 8 : (const float *)a.agg + (size_t)ar * H + g * 8;
  }
  Split3 wq[RING];
#pragma unroll
  for (int s = 0; s < RING; ++s) wq[s] = weights(a.W1s, s);
  constexpr int MINE = 2 * HS / MB;                             // consecutive slabs of the row this wave fetches and cuts
  static_assert(MINE * MB == 2 * HS && HS % MINE == 0 && 2 * HS >= RING, "");
  const int s0 = w * MINE;
  const float *px = s0 < HS ? pa + s0 * 16 : pb + (s0 - HS) * 16;
  f32x4 x[MINE][2];
#pragma unroll
  for (int i = 0; i < MINE; ++i)
#pragma unroll
    for (int k = 0; k < 2; ++k) x[i][k] = *(const f32x4 *)(px + i * 16 + 4 * k);
  [[maybe_unused]] TailRaw<8> xt;
  if constexpr (KIND == KIND_EDGE) xt = load_tail<8>(a.edge_feat + (size_t)row * a.De, a.De, 0, g);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    acc[r] = a.b1[32 * w + acc_row(r, g)];
    b2[r] = a.b2[32 * w + acc_row(r, g)];
    corr[r] = 0.f;
  }
  auto cut = [](const f32x4 &lo, const f32x4 &hi) {
    const float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return split3(v);
  };
#pragma unroll
  for (int i = 0; i < MINE; ++i) share(s0 + i, cut(x[i][0], x[i][1]));
  __syncthreads();
  Split3 x0 = shared(0);
#pragma unroll
  for (int s = 0; s < 2 * HS; ++s) {
    const Split3 x1 = shared(s + 1 < 2 * HS ? s + 1 : 0);
    mma_split3(wq[s % RING], x0, acc, corr);
    if (s + RING < 2 * HS || (KIND == KIND_EDGE && s + RING == 2 * HS)) wq[s % RING] = weights(a.W1s, s + RING);
    x0 = x1;
    __builtin_amdgcn_sched_barrier(0);                          // (see mlp2_split_kernel)
  }
  if constexpr (KIND == KIND_EDGE) {
    const float *xe = a.edge_feat + (size_t)row * a.De;
    for (int s = 2 * HS; s < a.nslab1; ++s) {                   // edge attributes
      const TailRaw<8> r = s == 2 * HS ? xt : load_tail<8>(xe, a.De, s - 2 * HS, g);
      const Split3 wv = s == 2 * HS ? wq[(2 * HS) % RING] : weights(a.W1s, s);
      mma_split3(wv, cut(r.q[0], r.q[1]), acc, corr);
    }
  }
  // ---------------- layer 2
#pragma unroll
  for (int c = 0; c < RING; ++c) wq[c] = weights(a.W2s, c);
  __syncthreads();                                              // (every wave has read its input fragments)
  float odd = 0.f;                                              // a NaN if one of them is not finite, which then makes the row's every output one
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    acc[r] += corr[r];
    odd = fmaf(acc[r], 0.f, odd);
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float z[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) z[j] = relu_f32(acc[8 * q + j]);
    if (q == 0) z[0] += odd;
    share(2 * w + q, split3(z));
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) { acc[r] = b2[r]; corr[r] = 0.f; }
  __syncthreads();
  x0 = shared(0);
#pragma unroll
  for (int c = 0; c < NC2; ++c) {
    const Split3 x1 = shared(c + 1 < NC2 ? c + 1 : 0);
    mma_split3(wq[c % RING], x0, acc, corr);
    if (c + RING < NC2) wq[c % RING] = weights(a.W2s, c + RING);
    x0 = x1;
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] += corr[r];
  // ---------------- rows with a value that has no parts, or that overflowed: once more, in fp32
  odd = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) odd = fmaf(acc[r], 0.f, odd);
  const unsigned long long lanes = __ballot(odd != 0.f && l32 < nv);
  for (unsigned rows = (unsigned)(lanes | lanes >> 32); rows; rows &= rows - 1) {
    const int r = __builtin_ctz(rows);
    const int64_t ro = row0 + r;
    const int64_t first = KIND == KIND_EDGE ? a.in_src[ro] : a.h_row ? a.h_row[ro] : ro;
    const int64_t second = KIND == KIND_EDGE ? (a.h_row ? a.h_row : a.in_dst)[ro] : a.agg_src ? a.agg_src[ro] : ro;
    const float *xa = (const float *)a.h + (size_t)first * H, *xe = a.edge_feat + (KIND == KIND_EDGE ? (size_t)ro * a.De : 0);
    const float *xb = second < 0 ? (const float *)a.zero_row : (const float *)(KIND == KIND_EDGE ? a.h : a.agg) + (size_t)second * H;
    const int K = KIND == KIND_EDGE ? 2 * H + a.De : 2 * H;
    constexpr int NF = H / 64;                                  // relu(z1) of features lane, lane + 64, ..
    float z[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) z[i] = a.b1[lane + 64 * i];
    for (int k = 0; k < K; ++k) {
      const float x = k < H ? xa[k] : k < 2 * H ? xb[k - H] : xe[k - 2 * H];
#pragma unroll
      for (int i = 0; i < NF; ++i) z[i] = fmaf(x, a.W1[(size_t)k * H + lane + 64 * i], z[i]);
    }
    float y = a.b2[32 * w + l32];                               // feature 32 w + l32, twice
    for (int k = 0; k < 64; ++k)
#pragma unroll
      for (int i = 0; i < NF; ++i) y = fmaf(__shfl(relu_f32(z[i]), k), a.W2[(size_t)(k + 64 * i) * H + 32 * w + l32], y);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float v = __shfl(y, acc_row(i, g));
      acc[i] = l32 == r ? v : acc[i];
    }
  }
  // ---------------- epilogue on this wave's 32 features
  float *out = (float *)a.out;
  char *stage = smem + S::ZBYTES + w * BlockStage<float>::BYTES;
  if constexpr (KIND != KIND_EDGE) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = relu_f32(acc[r]);
    store_block_via_lds<float, H>(out, row0, nv, w, lane, acc, stage);
  } else {
    f32x16 one[1] = {acc};
    const EdgeRoute e = edge_run_sums<1>(one, meta, nv, lane);
    store_block_rows_via_lds<float, H>(out, e.dsel, w, lane, one[0], stage);
    if (e.to_c0 || e.to_c1) store_tile_rows<float, H>(a.carry, wt * 2 + (e.to_c1 ? 1 : 0), true, w, g, one[0]);
  }
}

// A whole message-passing round in one launch, bf16, forward only, for batches of a few tiles per compute unit: a
// node's received sum needs its own in-edges alone, so a block of H / 32 waves that owns some consecutive
// nodes runs the edge MLP on their in-edges, 32 at a time (cut between receivers: no receiver may have
// more), keeps the sums in LDS, as the second half of the node MLP's input fragments, and goes on with
// the node MLP. Same operations in the same order per output as the two split kernels: the same bits.
// Bound by its chain of dependent steps (ranges, indices, rows, four products, stores); a wave requests all its
// weights of an MLP (100 registers) under the steps before. fp32, whose products are four times
// as long, gains nothing. As many nodes a block as give every compute unit one, 16 to 28: their in-edges, about one
// per node, then mostly fit one pass. us per encode of five rounds, two launches a round /
// one, H = 128: 454 nodes 56.5 / 46.4, 5.1 k 60.8 / 49.9, 7.1 k 61.9 / 58.3, 13.8 k 78.0 / 70.6, 20.6 k 96.0 / 96.9; H = 64: 454
// 48.0 / 35.5, 5.1 k 47.6 / 37.9, 13.8 k 54.5 / 48.2, 27.4 k 65.6 / 56.6.
// Two passes over a block's in-edges are the most that gain: same, 1 k nodes of 1 / 2 / 4 / 8 / 30 in-edges, H = 128:
// 63.5 / 49.2, 63.5 / 50.4, 66.1 / 60.5, 69.0 / 88.0, 93.7 / 275.8, H = 64: 53.0 / 39.4, 56.0 / 41.2, 56.3 / 48.8, 58.2 / 66.8, 68.8 / 199.9; three,
// of 28 nodes of 3 in-edges, 88.6 / 85.0 and 63.8 / 59.9, of 6 or more, 28 nodes of 4 in-edges, 90.9 / 98.0 and 62.9 / 67.7.
constexpr int kRoundNodesMin = 16, kRoundNodesMax = 28, kRoundEdges = 72;   // (a receiver that does not fit is left to the next pass)
struct RoundArgs {
  Mlp2Args edge, node;     // node.out: [N, H]; node.agg and edge.out are not used
  int nodes;               // of a block, at most 32
};
template <typename T, int H>
struct RoundTile {
  using S = SplitTile<T, H>;
  static constexpr int STAGE = S::MB * BlockStage<T>::BYTES;
  static constexpr int BYTES = 2 * S::XBYTES + STAGE;          // edge fragments (then relu(z1)), node fragments, staging
  static constexpr bool FITS = sizeof(T) == 2 && H <= 128;
};
// Layers 1 and 2 of a tile whose input fragments lie in `xs`: acc = this wave's 32 output features, bias
// included, before the last ReLU. relu(z1) goes where `zs` points (which may be xs).
template <typename T, int H, int TAIL>
__device__ __forceinline__ void split_layers(const Mlp2Args &a, const typename Operand<T>::vec *xs, typename Operand<T>::vec *zs,
                                             const typename Operand<T>::vec (&w1)[2 * SplitTile<T, H>::HS + 1],
                                             const typename Operand<T>::vec (&w2)[SplitTile<T, H>::MB * SplitTile<T, H>::QB],
                                             const TailRaw<Operand<T>::V> *xt, int64_t row,
                                             int w, int lane, f32x16 &acc) {
  using S = SplitTile<T, H>;
  using Opd = Operand<T>;
  using vec = typename Opd::vec;
  constexpr int V = Opd::V, HS = S::HS, MB = S::MB, QB = S::QB, NC2 = MB * QB;
  const int g = lane >> 5;
#pragma unroll
  for (int s = 0; s < 2 * HS; ++s) Opd::mma(w1[s], xs[s * 64 + lane], acc);
  if constexpr (TAIL) {
    const vec *W1 = (const vec *)a.W1s + (size_t)w * 64 + lane;
    const float *xe = a.edge_feat + (size_t)row * a.De;
    for (int s = 2 * HS; s < a.nslab1; ++s) {                   // edge attributes
      const vec xv = tail_to_operand<T>(s == 2 * HS ? *xt : load_tail<V>(xe, a.De, s - 2 * HS, g));
      const vec wv = s == 2 * HS ? w1[2 * HS] : W1[(size_t)s * MB * 64];
      Opd::mma(wv, xv, acc);
    }
  }
  __syncthreads();                                              // (every wave has read its input fragments)
#pragma unroll
  for (int q = 0; q < QB; ++q) zs[(w * QB + q) * 64 + lane] = relu_operand<T>(acc, q);
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = a.b2[32 * w + acc_row(r, g)];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < NC2; ++c) Opd::mma(w2[c], zs[c * 64 + lane], acc);
}
template <typename T, int H>
__global__ __launch_bounds__(2 * H) void mlp2_round_kernel(const RoundArgs a) {
  touch_args(a);
  using S = SplitTile<T, H>;
  using Opd = Operand<T>;
  using vec = typename Opd::vec;
  constexpr int V = Opd::V, SL = 2 * V, HS = S::HS, MB = S::MB, QB = S::QB, NC2 = MB * QB;
  extern __shared__ __align__(16) char smem[];
  vec *xe = (vec *)smem, *xn = (vec *)(smem + S::XBYTES);       // [2 HS][64] each
  const Mlp2Args &e = a.edge, &n = a.node;
  const int64_t n_tiles = n.n_blocks, per_xcd = (n_tiles + 7) / 8;
  const int64_t wt = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;      // (see mlp2_split_kernel)
  if ((int64_t)(blockIdx.x / 8) >= per_xcd || wt >= n_tiles) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char *stage = smem + 2 * S::XBYTES + w * BlockStage<T>::BYTES;
  // all the edge MLP's weights of this wave first, under the chain of indices
  vec w1[2 * HS + 1], w2[NC2];
  auto weights = [&](const Mlp2Args &m, int n1) {
    const vec *p1 = (const vec *)m.W1s + (size_t)w * 64 + lane, *p2 = (const vec *)m.W2s + (size_t)w * 64 + lane;
#pragma unroll
    for (int s = 0; s < 2 * HS + 1; ++s) w1[s] = p1[(size_t)(s < n1 ? s : 0) * MB * 64];
#pragma unroll
    for (int c = 0; c < NC2; ++c) w2[c] = p2[(size_t)c * MB * 64];
  };
  const int64_t n0 = wt * a.nodes;
  const int nn = n.n_rows - n0 < a.nodes ? (int)(n.n_rows - n0) : a.nodes;
  const int lo = n.in_ptr[n0], hi = n.in_ptr[n0 + (l32 < nn ? l32 + 1 : nn)];   // hi: end of node l32's in-edges
  weights(e, 2 * HS + 1);
  __builtin_amdgcn_sched_barrier(0);
  // ---- the node MLP's own half, and zeros for the sums of nodes without in-edges
  constexpr int MINE = 2 * HS / MB, OWN = HS / MB;              // consecutive slabs this wave fetches of an edge's two rows, of a node's
  static_assert(MINE * MB == 2 * HS && OWN * MB == HS && HS % MINE == 0, "");
  const T *h = (const T *)n.h;
  {
    const T *own = h + (size_t)(n0 + (l32 < nn ? l32 : nn - 1)) * H + g * V;
    vec x[OWN];
#pragma unroll
    for (int i = 0; i < OWN; ++i) x[i] = *(const vec *)(own + (w * OWN + i) * SL);
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
      xn[(w * OWN + i) * 64 + lane] = x[i];
      xn[(HS + w * OWN + i) * 64 + lane] = Opd::zero();
    }
  }
  const int end = __shfl(hi, nn - 1);
  for (int c0 = lo; c0 < end;) {
    // the receivers whose in-edges end within the next 32 (at least one: none has more)
    const int upto = __popcll(__ballot(hi <= c0 + 32 && lane < nn));
    const int c1 = __shfl(hi, upto - 1), nv = c1 - c0;
    const int64_t row = c0 + (l32 < nv ? l32 : nv - 1);
    const int src = e.in_src[row], dst = e.in_dst[row];
    const int s0 = w * MINE;
    const T *px = h + (size_t)(s0 < HS ? src : dst) * H + g * V + (s0 < HS ? s0 : s0 - HS) * SL;
    vec x[MINE];
#pragma unroll
    for (int i = 0; i < MINE; ++i) x[i] = *(const vec *)(px + i * SL);
    const TailRaw<V> xt = load_tail<V>(e.edge_feat + (size_t)row * e.De, e.De, 0, g);
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = e.b1[32 * w + acc_row(r, g)];
    __syncthreads();                                            // (the pass before has read relu(z1))
#pragma unroll
    for (int i = 0; i < MINE; ++i) xe[(s0 + i) * 64 + lane] = x[i];
    __syncthreads();
    split_layers<T, H, 1>(e, xe, xe, w1, w2, &xt, row, w, lane, acc);
    if (c1 >= end) weights(n, 2 * HS);                          // (the node MLP's, under the sums)
    EdgeTileMeta m;
    m.dst = dst; m.prev_d = m.next_d = -1;                      // (a pass holds whole receivers)
    f32x16 one[1] = {acc};
    const EdgeRoute to = edge_run_sums<1>(one, m, nv, lane);
    if (to.dsel >= 0) {
      // as operand fragments: feature f of this wave's 32 is element f % V of slab f / 2V, lane group (f % 2V) / V
      char *p = (char *)(xn + (HS + w * QB) * 64 + (to.dsel - (int)n0));
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float v[4] = {one[0][4 * q], one[0][4 * q + 1], one[0][4 * q + 2], one[0][4 * q + 3]};
        const int slab = sizeof(T) == 2 ? q / 2 : q, half = sizeof(T) == 2 ? q % 2 : g, at = sizeof(T) == 2 ? 8 * g : 0;
        store4<T>((T *)(p + (slab * 64 + half * 32) * 16 + at), v);
      }
    }
    c0 = c1;
  }
  if (lo >= end) weights(n, 2 * HS);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = n.b1[32 * w + acc_row(r, g)];
  __syncthreads();
  split_layers<T, H, 0>(n, xn, xe, w1, w2, nullptr, 0, w, lane, acc);
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = relu_f32(acc[r]);
  store_block_via_lds<T, H>((T *)n.out, n0, nn, w, lane, acc, stage);
}
