// Backward of the fused two-layer ReLU MLPs of the encoder (Section 3.3.4: one back-propagation
// through the GNN of Section 3.4), a tile of 32 rows per block, all contractions on the matrix
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
// (many rows in bf16: mlp2_bwd_wide_kernel).
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
  int De, Dd;
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
template <typename T, int H, int KIND>
__global__ __launch_bounds__(2 * H) void mlp2_bwd_kernel(const Mlp2BwdArgs a) {
  touch_args(a);
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

// Weight fragments for NW waves, UG units of UF fragments per group, through LDS: every wave
// fetches GF / NW of a group's fragments a whole group ahead of their use.
template <int UF, int UG, int NW>
struct WeightGroupsN {
  static constexpr int GF = UF * UG, PW = GF / NW;
  static_assert(GF % NW == 0, "a group is fetched by all waves of the block");
  f32x4 (*buf)[GF][64];
  int p = 0, wave, lane;
  f32x4 r[PW];
  template <typename Idx>
  __device__ __forceinline__ void fetch(const bf16x8 *W, Idx idx) {
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      const int jg = wave * PW + i;
      r[i] = __builtin_bit_cast(f32x4, W[(size_t)idx(jg / UF, jg % UF) * 64]);
    }
  }
  __device__ __forceinline__ void commit(int q) {
#pragma unroll
    for (int i = 0; i < PW; ++i) buf[q][wave * PW + i][lane] = r[i];
  }
  template <typename Idx>
  __device__ __forceinline__ void begin(const bf16x8 *W, Idx idx) {
    fetch(W, idx);
    commit(p);
    __syncthreads();
  }
  __device__ __forceinline__ void next(bool have_next) {
    if (have_next) commit(p ^ 1);
    __syncthreads();
    p ^= 1;
  }
  __device__ __forceinline__ bf16x8 get(int u, int j) const { return __builtin_bit_cast(bf16x8, buf[p][u * UF + j][lane]); }
};

// The same in bf16 for many rows: a wave per tile of 32 rows, four of them a block that walks through the weight matrices in groups of
// fragments, each fetched from L2 once per block, a whole group ahead of its use. Same operations in the same order: the same bits.
// A quarter of the weights' way from L2, but a chain of products H / 32 times as long, so it takes a pass of the chip, whole or
// not, at a time; launch_mlp2_bwd_wide has the rule. us per launch, split / this: edge, H = 64: 85 k edges 20.9 / 18.9, 163 k 32.3 / 29.0, 319 k
// 98.2 / 83.2; H = 128: 64 k 34.4 / 28.8, 117 k 58.2 / 50.2, 163 k 112 / 88, 319 k 219 / 166; H = 256: 163 k 271 / 242, 319 k 510 / 463; node, H = 256,
// 305 k nodes 469 / 421.
template <int H>
struct BwdWide {
  static constexpr int NW = 4, MB = H / 32, QB = 2, UF = MB * QB;   // waves; 32-feature blocks, slabs of one, fragments per unit
  static constexpr int UG = H >= 256 ? 4 : 2;                       // units per group
  static constexpr int BYTES = NW * BlockStage<bf16_t>::BYTES + 2 * UF * UG * 1024;
};
template <int H, int KIND>
__global__ __launch_bounds__(256) void mlp2_bwd_wide_kernel(const Mlp2BwdArgs a) {
  touch_args(a);
  static_assert(KIND != KIND_EMBED, "the embed MLP's backward has two products: the split form is the faster one at any size");
  using T = bf16_t;
  using S = BwdWide<H>;
  using Opd = Operand<T>;
  using vec = bf16x8;
  constexpr int V = Opd::V, SL = 2 * V, MB = S::MB, QB = S::QB, HS = H / SL, UF = S::UF, UG = S::UG;
  constexpr int SPU = UF / MB;                              // layer-1 slabs per unit
  const int64_t per_xcd = (a.n_blocks + 7) / 8;
  const int64_t tile = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (tile >= a.n_blocks) return;                           // (the whole block)
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row0 = (tile * S::NW + wave) * 32, left = a.n_rows - row0;
  const int n_valid = left < 32 ? (left > 0 ? (int)left : 0) : 32;
  const int64_t row = row0 + l32 < a.n_rows ? row0 + l32 : a.n_rows - 1;        // clamp loads; stores are guarded
  extern __shared__ __align__(16) char smem[];
  char *stage = smem + wave * BlockStage<T>::BYTES;
  WeightGroupsN<UF, UG, S::NW> wg;
  wg.buf = reinterpret_cast<f32x4 (*)[UF * UG][64]>(smem + S::NW * BlockStage<T>::BYTES);
  wg.wave = wave; wg.lane = lane;
  // a unit's fragments: all LDS reads in flight together, the products behind them wait for one each
  auto unit = [&](vec *w, int u) {
#pragma unroll
    for (int j = 0; j < UF; ++j) w[j] = wg.get(u, j);
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---------------- z1^T = relu(W1^T x^T + b1)
  f32x16 acc1[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc1[mb][r] = a.b1[32 * mb + acc_row(r, g)];
  int64_t dyr = row;
  {
    // layer 1's fragments are contiguous: unit u = fragments [u UF, u UF + UF) = SPU slabs
    const vec *W1 = (const vec *)a.W1s + lane;
    const int n_frag = a.nslab1 * MB, n_units = (a.nslab1 + SPU - 1) / SPU;
    const T *pa, *pb;
    if constexpr (KIND == KIND_EDGE) {
      dyr = a.in_dst[row];
      pa = (const T *)a.h + (size_t)a.in_src[row] * H + g * V;
      pb = (const T *)a.h + (size_t)dyr * H + g * V;
    } else {
      pa = (const T *)a.h + (size_t)row * H + g * V;
      const int64_t ar = a.agg_src ? (int64_t)a.agg_src[row] : row;
      pb = ar < 0 ? (const T *)a.zero_row + g * V : (const T *)a.agg + (size_t)ar * H + g * V;
    }
    // fragment j of unit u of the group that starts at unit u0 (past the last: the first once more, not used)
    auto idx_from = [&](int u0) {
      return [=](int u, int j) { const int f = (u0 + u) * UF + j; return f < n_frag ? f : 0; };
    };
    wg.begin(W1, idx_from(0));
    // the 2 HS slabs of the two H-wide input parts: gathered rows, requested XQ slabs ahead
    constexpr int NSH = 2 * HS, XQ = 8, NSU = NSH / SPU;
    static_assert(XQ <= NSH && NSU % UG == 0, "the H-wide parts fill whole groups");
    auto load_slab = [&](int s) -> vec { return *(const vec *)(s < HS ? pa + s * SL : pb + (s - HS) * SL); };
    vec xq[XQ];
#pragma unroll
    for (int s = 0; s < XQ; ++s) xq[s] = load_slab(s);
#pragma unroll
    for (int g0 = 0; g0 < NSU; g0 += UG) {
      if (g0 + UG < n_units) wg.fetch(W1, idx_from(g0 + UG));
#pragma unroll
      for (int u = 0; u < UG; ++u) {
        vec w[UF];
        unit(w, u);
#pragma unroll
        for (int j = 0; j < SPU; ++j) {
          const int s = (g0 + u) * SPU + j;
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) Opd::mma(w[j * MB + mb], xq[s % XQ], acc1[mb]);
          if (s + XQ < NSH) xq[s % XQ] = load_slab(s + XQ);
        }
      }
      wg.next(g0 + UG < n_units);
    }
    for (int u0 = NSU; u0 < n_units; u0 += UG) {            // edge attributes
      if (u0 + UG < n_units) wg.fetch(W1, idx_from(u0 + UG));
#pragma unroll
      for (int u = 0; u < UG; ++u)
#pragma unroll
        for (int j = 0; j < SPU; ++j) {
          const int s = (u0 + u) * SPU + j;
          if (s < a.nslab1) {
            const vec x = tail_to_operand<T>(load_tail<V>(a.edge_feat + (size_t)row * a.De, a.De, s - NSH, g));
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) Opd::mma(wg.get(u, j * MB + mb), x, acc1[mb]);
          }
        }
      wg.next(u0 + UG < n_units);
    }
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc1[mb][r] = relu_f32(acc1[mb][r]);
    store_block_via_lds<T, H>((T *)a.z1, row0, n_valid, mb, lane, acc1[mb], stage);
  }

  // ---------------- dz2^T = dy^T * [y^T > 0], stored and kept as operand slabs
  vec dz2s[MB][QB];
  {
    const T *dyrow = (const T *)a.dy + (size_t)dyr * H + 4 * g;
    [[maybe_unused]] const vec *W2 = (const vec *)a.W2s + lane;
    [[maybe_unused]] const T *yrow = KIND == KIND_EDGE ? nullptr : (const T *)a.y + (size_t)row * H + 4 * g;
    // dy (and y where the forward stored it) of block nb + 1 is requested while block nb is worked on: the
    // fences of the staged stores keep the compiler from doing that itself
    auto quads = [&](const T *p, int nb, f32x16 &v) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float t[4];
        load4<T>(p + 32 * nb + 8 * q, t);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[4 * q + j] = t[j];
      }
    };
    f32x16 dyc, yc, dyn, yn;
    quads(dyrow, 0, dyc);
    if constexpr (KIND != KIND_EDGE) quads(yrow, 0, yc);
    // EDGE: y^T block nb needs W2's fragments ((mb, q), nb) for all (mb, q): unit nb
    auto idx_from = [&](int u0) { return [=](int u, int j) { return j * MB + u0 + u; }; };
    if constexpr (KIND == KIND_EDGE) wg.begin(W2, idx_from(0));
#pragma unroll
    for (int nb = 0; nb < MB; ++nb) {
      if (nb + 1 < MB) {
        quads(dyrow, nb + 1, dyn);
        if constexpr (KIND != KIND_EDGE) quads(yrow, nb + 1, yn);
      }
      if constexpr (KIND == KIND_EDGE) {
        const int g0 = nb / UG * UG, u = nb % UG;
        if (u == 0 && g0 + UG < MB) wg.fetch(W2, idx_from(g0 + UG));
        vec w[UF];
        unit(w, u);
#pragma unroll
        for (int r = 0; r < 16; ++r) yc[r] = a.b2[32 * nb + acc_row(r, g)];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int q = 0; q < QB; ++q) Opd::mma(w[mb * QB + q], acc_slab<T>(acc1[mb], q), yc);
        if (u == UG - 1) wg.next(g0 + UG < MB);
      }
      f32x16 d;
#pragma unroll
      for (int r = 0; r < 16; ++r) d[r] = yc[r] > 0.f ? dyc[r] : 0.f;
      store_block_via_lds<T, H>((T *)a.dz2, row0, n_valid, nb, lane, d, stage);
#pragma unroll
      for (int q = 0; q < QB; ++q) dz2s[nb][q] = acc_slab<T>(d, q);
      if (nb + 1 < MB) { dyc = dyn; yc = yn; }
    }
  }

  // ---------------- dz1^T = (W2 dz2^T) * [z1^T > 0]: unit mb = the W2^T fragments of block mb
  vec dz1s[MB][QB];
  {
    const vec *W2b = (const vec *)a.W2bt + lane;
    auto idx_from = [&](int u0) { return [=](int u, int j) { return j * MB + u0 + u; }; };
    wg.begin(W2b, idx_from(0));
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int g0 = mb / UG * UG, u = mb % UG;
      if (u == 0 && g0 + UG < MB) wg.fetch(W2b, idx_from(g0 + UG));
      vec w[UF];
      unit(w, u);
      f32x16 d;
#pragma unroll
      for (int r = 0; r < 16; ++r) d[r] = 0.f;
#pragma unroll
      for (int nb = 0; nb < MB; ++nb)
#pragma unroll
        for (int q = 0; q < QB; ++q) Opd::mma(w[nb * QB + q], dz2s[nb][q], d);
      if (u == UG - 1) wg.next(g0 + UG < MB);
#pragma unroll
      for (int r = 0; r < 16; ++r) d[r] = acc1[mb][r] > 0.f ? d[r] : 0.f;
      store_block_via_lds<T, H>((T *)a.dz1, row0, n_valid, mb, lane, d, stage);
#pragma unroll
      for (int q = 0; q < QB; ++q) dz1s[mb][q] = acc_slab<T>(d, q);
    }
  }

  // ---------------- dx^T = W1 dz1^T over the first 2H input columns (h parts only): unit kb = the W1^T fragments of
  // the 32-column block kb of [part a | part b]
  const vec *W1b = (const vec *)a.W1bt + lane;
  constexpr int KB = 2 * MB;
  auto idx_from = [&](int u0) { return [=](int u, int j) { return j * KB + u0 + u; }; };
  wg.begin(W1b, idx_from(0));
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const int g0 = kb / UG * UG, u = kb % UG;
    if (u == 0 && g0 + UG < KB) wg.fetch(W1b, idx_from(g0 + UG));
    vec w[UF];
    unit(w, u);
    f32x16 d;
#pragma unroll
    for (int r = 0; r < 16; ++r) d[r] = 0.f;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int q = 0; q < QB; ++q) Opd::mma(w[mb * QB + q], dz1s[mb][q], d);
    if (u == UG - 1) wg.next(g0 + UG < KB);
    store_block_via_lds<T, H>((T *)(kb < MB ? a.dx_a : a.dx_b), row0, n_valid, kb % MB, lane, d, stage);
  }
}
