// Backward of the fused two-layer ReLU MLPs of the encoder (Section 3.3.4: one back-propagation
// through the GNN of Section 3.4), per tile of 32 rows per wave, all contractions on the matrix
// cores. For y = relu(relu(x W1 + b1) W2 + b2) and upstream dy:
//     dz2 = dy * [y > 0],  dz1 = (dz2 W2^T) * [z1 > 0],  dx = dz1 W1^T.
// Everything is kept transposed (features x rows: lane = row, registers = features), so each
// result is already laid out as the next contraction's B operand:
//     z1^T  = W1^T x^T            (as in the forward kernel)
//     y^T   = W2^T z1^T           (EDGE only: its per-edge output is not stored by the forward)
//     dz1^T = W2 dz2^T            (W2 pre-arranged with the contraction over its columns)
//     dx^T  = W1 dz1^T            (W1 pre-arranged with the contraction over its columns)
// A block of H / 32 waves takes one tile of 32 rows, wave w the 32 output features of block w of z1, y and
// dz1, and blocks w and H / 32 + w of dx; a product's input is shared through LDS as operand fragments, and a wave streams
// its own slices of the weights, eight fragments ahead (mlp2_split_kernel does the forward the same way). What bounds it: few tiles,
// the chain of dependent products, which is H / 32 times shorter than with a wave per tile; many, in fp32, the matrix cores (87 % busy at
// H = 256), in bf16 the weights' way from L2. us per launch, a wave per tile (four of them sharing the weights through LDS in bf16) / this,
// edge: fp32 H = 64: 1.8 k edges 29.0 / 13.1, 20 k 31.0 / 22.6, 158 k 108.7 / 99.4; H = 128: 91.5 / 20.6, 131 / 49.9, 370 / 302; H = 256:
// 371 / 56.7, 534 / 166, 2128 / 1093; bf16: H = 64: 1.8 k 11.0 / 7.1, 39 k 16.0 / 13.4; H = 128: 18.8 / 9.3, 29.5 / 25.3; H = 256: 44.1 / 15.1, 95.9 / 62.8
// (157 k, which only attributes of more than eight columns bring here in bf16, 245 / 251).
// The kernel writes z1, dz1, dz2 as [rows, H] for the weight-gradient kernel, and dx:
//   EDGE: per-edge gradients w.r.t. h_sender and h_receiver ([E, H] each; summed per node later),
//   NODE: d/dh and d/dagg [N, H],   EMBED: nothing (its inputs are data).
// Gradients w.r.t. node states travel between kernels in the operand type: their only readers
// are this kernel's instantiations, which turn them into operands of that type anyway, and the
// per-node gather, which sums in fp32.
#pragma once
#include <type_traits>
#include "mlp2.hip.h"

struct Mlp2BwdArgs {
  int64_t n_rows, n_blocks;
  const void *W1s, *W2s;     // forward fragment order
  const void *W2bt, *W1bt;   // contraction over the weight's columns (SWZ_CHAIN order)
  const float *b1, *b2;
  int nslab1;
  const void *W1x;           // EMBED: see Mlp2Args
  int nslabx;
  const float *table;
  const void *h, *agg;       // forward inputs, operand type
  const int32_t *agg_src;    // NODE: [N] row of agg per node, -1 = none (zeros are read); or nullptr
  const void *zero_row;      // 1 KB of zeros
  const void *y;             // saved forward output [N, H] operand type      (NODE, EMBED)
  const void *dy;            // upstream gradient [N, H], operand type (EDGE: indexed by receiver)
  const int32_t *in_ptr, *in_src, *in_dst;
  const float *edge_feat;
  const int32_t *node_op;
  const float *node_dense;
  int De, Tn, Dd;
  void *z1, *dz1, *dz2;      // [rows, H] operand type
  void *dx_a, *dx_b;         // EDGE: d h_sender, d h_receiver [E, H] operand type;
                             // NODE: d h, d agg [N, H] operand type
};

// Accumulator tile (features x rows) -> the 32 / (2V) operand slabs of its 32 features.
template <typename T>
__device__ __forceinline__ typename Operand<T>::vec acc_slab(const f32x16 &acc, int q);
template <>
__device__ __forceinline__ f32x4 acc_slab<float>(const f32x16 &acc, int q) {
  return f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
}
template <>
__device__ __forceinline__ bf16x8 acc_slab<bf16_t>(const f32x16 &acc, int q) {
  return pack_bf16x8(acc[8 * q], acc[8 * q + 1], acc[8 * q + 2], acc[8 * q + 3], acc[8 * q + 4],
                     acc[8 * q + 5], acc[8 * q + 6], acc[8 * q + 7]);
}

// (Operations in the order of the forward kernel. EMBED: z1 as the forward forms it, from the op type's row of W1 and the fp32 columns.)
template <typename T, int H>
struct BwdTile {
  using S = SplitTile<T, H>;
  static constexpr int EBYTES = S::HS * 1024;                   // an exchange area: [HS][64] fragments; two of them hold the input
  static constexpr int BYTES = 2 * EBYTES + S::MB * BlockStage<T>::BYTES;
};
template <typename T1, typename T, int H, int KIND>
__global__ __launch_bounds__(2 * H) void mlp2_bwd_kernel(const Mlp2BwdArgs a) {
  using S = SplitTile<T, H>;
  using B = BwdTile<T, H>;
  using Opd = Operand<T>;
  using vec = typename Opd::vec;
  constexpr int V = Opd::V, SL = 2 * V, HS = S::HS, MB = S::MB, QB = S::QB;
  constexpr int RING = HS < 8 ? HS : 8;                         // weight fragments in flight
  static_assert(MB * QB == HS, "");
  extern __shared__ __align__(16) char smem[];
  vec *ea = (vec *)smem, *eb = (vec *)(smem + B::EBYTES);
  const int64_t n_tiles = a.n_blocks, per_xcd = (n_tiles + 7) / 8;
  const int64_t wt = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;      // (see mlp2_split_kernel)
  if ((int64_t)(blockIdx.x / 8) >= per_xcd || wt >= n_tiles) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char *stage = smem + 2 * B::EBYTES + w * BlockStage<T>::BYTES;
  const int64_t row0 = wt * 32;
  const int nv = a.n_rows - row0 < 32 ? (int)(a.n_rows - row0) : 32;
  const int64_t row = row0 + (l32 < nv ? l32 : nv - 1);         // clamp loads; stores are guarded

  vec wq[RING];
  // first fragments of a product: block cb of the cbs blocks of W
  auto begin = [&](const void *W, int cb, int cbs) {
    const vec *p = (const vec *)W + (size_t)cb * 64 + lane;
#pragma unroll
    for (int c = 0; c < RING; ++c) wq[c] = p[(size_t)c * cbs * 64];
  };
  // acc += block cb of W times the N fragments of x (LDS); one more fragment of W is left in wq[N % RING] if EXTRA
  auto product = [&](auto n, auto extra, const void *W, int cb, int cbs, const vec *x, f32x16 &acc) {
    constexpr int N = decltype(n)::value, LAST = N + (decltype(extra)::value ? 1 : 0);
    const vec *p = (const vec *)W + (size_t)cb * 64 + lane;
    vec x0 = x[lane];
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const vec x1 = x[(c + 1 < N ? c + 1 : 0) * 64 + lane];
      Opd::mma(wq[c % RING], x0, acc);
      if (c + RING < LAST) wq[c % RING] = p[(size_t)(c + RING) * cbs * 64];
      x0 = x1;
      __builtin_amdgcn_sched_barrier(0);                        // (see mlp2_split_kernel)
    }
  };
  constexpr std::integral_constant<int, HS> one_part{};
  constexpr std::false_type no{};
  auto share = [&](vec *to, const f32x16 &d) {
#pragma unroll
    for (int q = 0; q < QB; ++q) to[(w * QB + q) * 64 + lane] = acc_slab<T>(d, q);
  };

  // ---------------- z1^T = relu(W1^T x^T + b1), exactly as in the forward kernel, and what dz2 is formed of
  f32x16 z1, dy, y;
  auto quads = [&](const T *p, f32x16 &v) {                     // this wave's 32 features of a row
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float t[4];
      load4<T>(p + 32 * w + 8 * q + 4 * g, t);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[4 * q + j] = t[j];
    }
  };
  if constexpr (KIND != KIND_EMBED) {
    const T *pa, *pb;
    int64_t dyr = row;
    if constexpr (KIND == KIND_EDGE) {
      dyr = a.in_dst[row];
      pa = (const T *)a.h + (size_t)a.in_src[row] * H + g * V;
      pb = (const T *)a.h + (size_t)dyr * H + g * V;
    } else {
      pa = (const T *)a.h + (size_t)row * H + g * V;
      const int64_t ar = a.agg_src ? (int64_t)a.agg_src[row] : row;
      pb = ar < 0 ? (const T *)a.zero_row + g * V : (const T *)a.agg + (size_t)ar * H + g * V;
    }
    begin(a.W1s, w, MB);
    constexpr int MINE = 2 * HS / MB;                           // consecutive slabs of the row this wave fetches
    static_assert(MINE * MB == 2 * HS && HS % MINE == 0, "");
    const int s0 = w * MINE;
    const T *px = s0 < HS ? pa + s0 * SL : pb + (s0 - HS) * SL;
    vec x[MINE];
#pragma unroll
    for (int i = 0; i < MINE; ++i) x[i] = *(const vec *)(px + i * SL);
    [[maybe_unused]] TailRaw<V> xt;
    if constexpr (KIND == KIND_EDGE) xt = load_tail<V>(a.edge_feat + (size_t)row * a.De, a.De, 0, g);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      z1[r] = a.b1[32 * w + acc_row(r, g)];
      if constexpr (KIND == KIND_EDGE) y[r] = a.b2[32 * w + acc_row(r, g)];
    }
    quads((const T *)a.dy + (size_t)dyr * H, dy);
    if constexpr (KIND != KIND_EDGE) quads((const T *)a.y + (size_t)row * H, y);
#pragma unroll
    for (int i = 0; i < MINE; ++i) ea[(s0 + i) * 64 + lane] = x[i];
    __syncthreads();
    product(std::integral_constant<int, 2 * HS>(), std::bool_constant<KIND == KIND_EDGE>(), a.W1s, w, MB, ea, z1);
    if constexpr (KIND == KIND_EDGE) {
      const vec *W1 = (const vec *)a.W1s + (size_t)w * 64 + lane;
      for (int s = 2 * HS; s < a.nslab1; ++s) {                 // edge attributes
        const vec xv = tail_to_operand<T>(s == 2 * HS ? xt : load_tail<V>(a.edge_feat + (size_t)row * a.De, a.De, s - 2 * HS, g));
        const vec wv = s == 2 * HS ? wq[(2 * HS) % RING] : W1[(size_t)s * MB * 64];
        Opd::mma(wv, xv, z1);
      }
    }
  } else {
    const EmbedRow er = load_embed_row(a.node_op, a.in_ptr, a.node_dense, a.Dd, row);
    const float *trow = a.table + (size_t)er.op * H + 32 * w + 4 * g;
    quads((const T *)a.dy + (size_t)row * H, dy);
    quads((const T *)a.y + (size_t)row * H, y);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 t = *(const f32x4 *)(trow + 8 * q);
      const f32x4 b = *(const f32x4 *)(a.b1 + 32 * w + 8 * q + 4 * g);
#pragma unroll
      for (int j = 0; j < 4; ++j) z1[4 * q + j] = t[j] + b[j];
    }
    const f32x4 *W1 = (const f32x4 *)a.W1x + (size_t)w * 64 + lane;
    for (int s = 0; s < a.nslabx; ++s) {
      const f32x4 xv = embed_columns(er, a.edge_feat, a.De, a.Dd, s * 8 + g * 4);
      Operand<float>::mma(W1[(size_t)s * MB * 64], xv, z1);
    }
  }
  begin(KIND == KIND_EDGE ? a.W2s : a.W2bt, w, MB);
#pragma unroll
  for (int r = 0; r < 16; ++r) z1[r] = relu_f32(z1[r]);
  __syncthreads();                                              // (every wave has read the input)

  // ---------------- dz2^T = dy^T * [y^T > 0]
  if constexpr (KIND == KIND_EDGE) {
    share(ea, z1);
    store_block_via_lds<T, H>((T *)a.z1, row0, nv, w, lane, z1, stage);
    __syncthreads();
    product(one_part, no, a.W2s, w, MB, ea, y);
    begin(a.W2bt, w, MB);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) dy[r] = y[r] > 0.f ? dy[r] : 0.f;
  share(eb, dy);
  if constexpr (KIND != KIND_EDGE) store_block_via_lds<T, H>((T *)a.z1, row0, nv, w, lane, z1, stage);
  store_block_via_lds<T, H>((T *)a.dz2, row0, nv, w, lane, dy, stage);
  __syncthreads();

  // ---------------- dz1^T = (W2 dz2^T) * [z1^T > 0]
  f32x16 d;
#pragma unroll
  for (int r = 0; r < 16; ++r) d[r] = 0.f;
  product(one_part, no, a.W2bt, w, MB, eb, d);
  if constexpr (KIND != KIND_EMBED) begin(a.W1bt, w, 2 * MB);
#pragma unroll
  for (int r = 0; r < 16; ++r) d[r] = z1[r] > 0.f ? d[r] : 0.f;
  if constexpr (KIND != KIND_EMBED) share(ea, d);
  store_block_via_lds<T, H>((T *)a.dz1, row0, nv, w, lane, d, stage);

  // ---------------- dx^T = W1 dz1^T over the first 2H input columns (h parts only)
  if constexpr (KIND != KIND_EMBED) {
    __syncthreads();
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
      for (int r = 0; r < 16; ++r) d[r] = 0.f;
      product(one_part, no, a.W1bt, part * MB + w, 2 * MB, ea, d);
      if (part == 0) begin(a.W1bt, MB + w, 2 * MB);
      store_block_via_lds<T, H>((T *)(part == 0 ? a.dx_a : a.dx_b), row0, nv, w, lane, d, stage);
    }
  }
}
