// The graph-attention reading of the message-passing layer (second equation of Section 3.4, which
// cites graph attention for its learned per-edge weighting): per round
//   z = h W;  per edge j -> i: s = LeakyReLU_0.2(a_src . z_j + a_dst . z_i), likewise for a self
//   edge; alpha = softmax of s over i's in-edges plus the self edge;  h'_i = ReLU(sum alpha z_j).
// The dense part on the matrix cores (z and the two per-node scalars a_src . z, a_dst . z, taken from
// the fp32 accumulators), then a gather-bound pass over each receiver's contiguous in-edge
// range: a kernel each, or (gat_round_kernel, smaller batches) the pass of one round and the dense part
// of the next in one launch. The backward pass (further down) is gather-based as well: one
// pass per receiver for the softmax and score gradients, one per sender for dz, then two dense
// products (dh = dz W^T, dW = h^T dz) on the matrix cores.
#pragma once
#include "mlp2.hip.h"

struct GatArgs {
  int64_t n_rows, n_blocks;      // nodes; 128-row tiles
  const void *h;                 // [N, H] operand type
  const void *Ws;                // fragment-ordered W [H, H], operand type
  const float *a_src, *a_dst;    // [H]
  void *z;                       // [N, H] operand type
  float *s_src, *s_dst;          // [N]
  const int32_t *in_ptr, *in_src;
  const void *zero_row;          // 1 KB of zeros
  void *out;                     // [N, H] operand type
};

// z = h W for a tile of 32 rows per wave (features x rows, as the fused MLP's first layer), the
// two attention scalars of each row from the accumulators, z stored as whole rows. W streams from L2: for fp32 at
// H = 256, whose 256 KB fit no LDS.
template <typename T, int H>
__global__ __launch_bounds__(256) void gat_linear_kernel(const GatArgs a) {
  using Opd = Operand<T>;
  using vec = typename Opd::vec;
  constexpr int V = Opd::V, SL = 2 * V, MB = H / 32, HS = H / SL;
  __shared__ __align__(16) char stage[4][RowStage<T, H>::BYTES];
  const int64_t per_xcd = (a.n_blocks + 7) / 8;
  const int64_t tile = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (tile >= a.n_blocks) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, g = lane >> 5;
  const int64_t row0 = (tile * 4 + wave) * 32;
  if (row0 >= a.n_rows) return;
  int64_t row = row0 + l32;
  if (row >= a.n_rows) row = a.n_rows - 1;
  f32x16 acc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[mb][r] = 0.f;
  const vec *W = (const vec *)a.Ws + lane;
  const T *hp = (const T *)a.h + (size_t)row * H + g * V;
  vec x[HS];
#pragma unroll
  for (int s = 0; s < HS; ++s) x[s] = *(const vec *)(hp + s * SL);
#pragma unroll
  for (int s = 0; s < HS; ++s) mma_slab<T, H>(W + (size_t)s * MB * 64, x[s], acc);
  float ps = 0.f, pd = 0.f;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 as = *(const f32x4 *)(a.a_src + 32 * mb + 8 * q + 4 * g);
      const f32x4 ad = *(const f32x4 *)(a.a_dst + 32 * mb + 8 * q + 4 * g);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ps = fmaf(acc[mb][4 * q + j], as[j], ps);
        pd = fmaf(acc[mb][4 * q + j], ad[j], pd);
      }
    }
  ps += __shfl_xor(ps, 32);                                     // the row's other half of the features
  pd += __shfl_xor(pd, 32);
  if (a.s_src && g == 0 && row0 + l32 < a.n_rows) {          // (null for the backward's dh = dz W^T)
    a.s_src[row] = ps;
    a.s_dst[row] = pd;
  }
  T *z = (T *)a.z;
  store_rows_via_lds<T, H, false>(acc, stage[wave], lane, [&](int r) -> T * {
    return row0 + r < a.n_rows ? z + (size_t)(row0 + r) * H : nullptr;
  });
}

// The same product with W held in LDS: persistent blocks of eight waves copy it once and walk over wave tiles, a
// wave's next rows requested once the products have consumed this tile's. Bound by the rows' bytes; with every wave
// streaming W for each of its tiles the launch moved four times them through the L2: 148 k
// nodes, H = 128, bf16 26.0 -> 15.4 us (76 MB at 4.9 TB/s), 45 k nodes 14.0 -> 11.4.
template <typename T, int H>
struct GatLds {
  static constexpr int MB = H / 32, HS = H / (2 * Operand<T>::V);
  static constexpr int NW = HS * MB <= 32 ? 4 : 8;       // (a small W several times per compute unit)
  static constexpr bool BLOCKWISE = H * sizeof(T) > 256 && sizeof(T) == 2;      // staging by 32-feature blocks (W takes most of the LDS)
  static constexpr int WBYTES = HS * MB * 1024, ABYTES = 2 * MB * 2 * 16 * 4;
  static constexpr int STAGE = BLOCKWISE ? BlockStage<T>::BYTES : RowStage<T, H>::BYTES;
  static constexpr int BYTES = WBYTES + ABYTES + NW * STAGE;
  static constexpr bool FITS = BYTES <= 160 * 1024;
  static constexpr int PER_CU = NW == 8 ? 1 : 3;         // (the registers allow three waves per SIMD at H = 128)
};
template <typename T, int H>
__global__ __launch_bounds__((64 * GatLds<T, H>::NW)) void gat_linear_lds_kernel(const GatArgs a) {
  touch_args(a);
  using Opd = Operand<T>;
  using vec = typename Opd::vec;
  using S = GatLds<T, H>;
  constexpr int V = Opd::V, SL = 2 * V, MB = S::MB, HS = S::HS, NT = 64 * S::NW;
  extern __shared__ __align__(16) char smem[];
  vec *Wl = (vec *)smem;                                             // [HS][MB][64]
  float(*al)[MB][2][16] = (float(*)[MB][2][16])(smem + S::WBYTES);   // a_src, a_dst in accumulator order
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  char *stage = smem + S::WBYTES + S::ABYTES + wave * S::STAGE;
  // the wave tiles of one XCD are contiguous; inside it, tile j of a pass goes to wave j / nbx of block j % nbx
  const int nbx = gridDim.x / 8, xcd = blockIdx.x % 8, lid = blockIdx.x / 8;
  const int64_t n_wt = (a.n_rows + 31) / 32, per_xcd = (n_wt + 7) / 8, t_begin = xcd * per_xcd;
  const int64_t t_end = t_begin + per_xcd < n_wt ? t_begin + per_xcd : n_wt, stride = (int64_t)nbx * S::NW;
  int64_t wt = t_begin + (int64_t)wave * nbx + lid;
  vec x[HS];
  auto load_rows = [&](int64_t t) {
    int64_t row = t * 32 + l32;
    if (row >= a.n_rows) row = a.n_rows - 1;
    const T *hp = (const T *)a.h + (size_t)row * H + g * V;
#pragma unroll
    for (int s = 0; s < HS; ++s) x[s] = *(const vec *)(hp + s * SL);
  };
  {
    constexpr int NF = HS * MB * 64, C = (NF + NT - 1) / NT, B = C < 16 ? C : 16;   // in batches of at most 16 loads
    const vec *W = (const vec *)a.Ws;
    for (int c0 = 0; c0 < C; c0 += B) {
      vec t[B];
#pragma unroll
      for (int c = 0; c < B; ++c) t[c] = W[tid + (c0 + c) * NT < NF ? tid + (c0 + c) * NT : 0];
#pragma unroll
      for (int c = 0; c < B; ++c)
        if (tid + (c0 + c) * NT < NF) Wl[tid + (c0 + c) * NT] = t[c];
    }
    if (tid < MB * 32) {
      const int f = 32 * (tid / 32) + acc_row(tid % 16, (tid / 16) % 2);
      al[0][tid / 32][(tid / 16) % 2][tid % 16] = a.a_src[f];
      al[1][tid / 32][(tid / 16) % 2][tid % 16] = a.a_dst[f];
    }
  }
  if (wt < t_end) load_rows(wt);
  __syncthreads();
  for (; wt < t_end; wt += stride) {
    asm volatile("" ::: "memory");                           // (W's fragments are read from LDS in every tile)
    const int64_t row0 = wt * 32;
    f32x16 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mb][r] = 0.f;
#pragma unroll
    for (int s = 0; s < HS; ++s) mma_slab<T, H>(Wl + (size_t)s * MB * 64 + lane, x[s], acc);
    if (wt + stride < t_end) load_rows(wt + stride);
    if (a.s_src) {                                           // (null for the backward's dh = dz W^T)
      float ps = 0.f, pd = 0.f;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          ps = fmaf(acc[mb][r], al[0][mb][g][r], ps);
          pd = fmaf(acc[mb][r], al[1][mb][g][r], pd);
        }
      ps += __shfl_xor(ps, 32);                              // the row's other half of the features
      pd += __shfl_xor(pd, 32);
      if (g == 0 && row0 + l32 < a.n_rows) {
        a.s_src[row0 + l32] = ps;
        a.s_dst[row0 + l32] = pd;
      }
    }
    T *z = (T *)a.z;
    if constexpr (S::BLOCKWISE) {
      const int nv = a.n_rows - row0 < 32 ? (int)(a.n_rows - row0) : 32;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) store_block_via_lds<T, H>(z, row0, nv, mb, lane, acc[mb], stage);
    } else {
      store_rows_via_lds<T, H, false>(acc, stage, lane, [&](int r) -> T * {
        return row0 + r < a.n_rows ? z + (size_t)(row0 + r) * H : nullptr;
      });
    }
  }
}

__device__ __forceinline__ float leaky02(float x) { return x > 0.f ? x : 0.2f * x; }

// The first kGatAhead in-edges of receiver n (most have one or two): senders' scores and rows, requested together and
// under no condition (an absent edge reads the receiver's score and a row of zeros), so that a receiver waits
// for in_ptr, senders, and then scores and rows together, not for each edge in turn: 148 k nodes, H = 128,
// bf16: backward 56.2 -> 38.2 us (190 MB at 5.0 TB/s), forward 28.0 -> 21.8 (115 MB at 5.3 TB/s).
constexpr int kGatAhead = 2;
template <typename T, int VEC>
struct GatAhead {
  float s[kGatAhead], v[kGatAhead][VEC];
  __device__ __forceinline__ void request(const T *z, const T *zero_row, const float *s_src, const int32_t *in_src, int64_t n, int e0, int e1,
                                          int c, int H) {
    int from[kGatAhead];
#pragma unroll
    for (int k = 0; k < kGatAhead; ++k) from[k] = *(e0 + k < e1 ? in_src + e0 + k : (const int32_t *)zero_row);
#pragma unroll
    for (int k = 0; k < kGatAhead; ++k) {
      const bool there = e0 + k < e1;
      s[k] = s_src[there ? (int64_t)from[k] : n];
      RowVec<T, VEC>::load(there ? z + (size_t)from[k] * H + c : zero_row + c, v[k]);
    }
  }
};

// One receiver per group of H * sizeof(T) / 16 lanes, each a 16-byte column slice: softmax
// over the receiver's in-edges (contiguous in receiver order) plus the self edge, weighted sum
// of the gathered z rows, ReLU. Edges are taken in order, so the result is run-to-run identical.
template <typename T, int VEC>
__device__ __forceinline__ void gat_aggregate_row(const GatArgs &a, int H, int64_t n, int c, float *r) {
  const T *z = (const T *)a.z;
  const int e0 = a.in_ptr[n], e1 = a.in_ptr[n + 1];
  GatAhead<T, VEC> ahead;
  ahead.request(z, (const T *)a.zero_row, a.s_src, a.in_src, n, e0, e1, c, H);
  const float sd = a.s_dst[n];
  const float s_self = leaky02(a.s_src[n] + sd);
  float acc[VEC], v[VEC];
  RowVec<T, VEC>::load(z + (size_t)n * H + c, v);
  float u[kGatAhead], mx = s_self;
#pragma unroll
  for (int k = 0; k < kGatAhead; ++k) {
    u[k] = e0 + k < e1 ? leaky02(ahead.s[k] + sd) : -INFINITY;
    mx = fmaxf(mx, u[k]);
  }
  for (int e = e0 + kGatAhead; e < e1; ++e) mx = fmaxf(mx, leaky02(a.s_src[a.in_src[e]] + sd));
  float den = expf(s_self - mx);
#pragma unroll
  for (int j = 0; j < VEC; ++j) acc[j] = den * v[j];
#pragma unroll
  for (int k = 0; k < kGatAhead; ++k) {
    const float w = expf(u[k] - mx);                       // (absent: exactly 0, times a row of zeros)
    den += w;
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc[j] = fmaf(w, ahead.v[k][j], acc[j]);
  }
  for (int e = e0 + kGatAhead; e < e1; ++e) {
    const int s = a.in_src[e];
    const float w = expf(leaky02(a.s_src[s] + sd) - mx);
    den += w;
    RowVec<T, VEC>::load(z + (size_t)s * H + c, v);
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc[j] = fmaf(w, v[j], acc[j]);
  }
  const float inv = 1.f / den;
#pragma unroll
  for (int j = 0; j < VEC; ++j) r[j] = fmaxf(acc[j] * inv, 0.f);
}
template <typename T, int VEC>
__global__ __launch_bounds__(256) void gat_aggregate_kernel(const GatArgs a, int H) {
  touch_args(a);
  const int lpr = H / VEC;
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n = gt / lpr;
  if (n >= a.n_rows) return;
  const int c = (int)(gt - n * lpr) * VEC;
  float r[VEC];
  gat_aggregate_row<T, VEC>(a, H, n, c, r);
  T *o = (T *)a.out + (size_t)n * H + c;
#pragma unroll
  for (int q = 0; q < VEC / 4; ++q) store4<T>(o + 4 * q, r + 4 * q);
}

// A round's aggregation and the product of the next round in one launch: a persistent block of 32 receivers' lane groups
// aggregates a tile of 32 rows into LDS as operand fragments, and one of its waves, each in turn, forms z = h W of the tile from
// there and from W, which the block keeps in LDS, while the others aggregate the next tile (two tile buffers, one
// barrier a tile). h leaves for memory only where it is kept for the backward pass. The arithmetic is that of the two
// kernels above. Bound by the aggregation's three dependent gathers. Encodes of
// five rounds, two kernels a round / this one, us: bf16 H = 128, 1 k nodes 64.3 / 55.8, 18 k 90 / 80, 37 k 135 / 110, 55 k 145 / 128, 145 k 220 / 243;
// H = 64, 1 k 60 / 47, 37 k 86 / 69, 73 k 125 / 96; fp32 H = 64, 1 k 71 / 56, 37 k 136 / 116, 55 k 149 / 143, 73 k 172 / 176. Two blocks a
// compute unit: for three the registers spill (22 us a round of 35 k nodes for 18; two kernels 24).
template <typename T, int H>
struct GatRound {
  static constexpr int MB = H / 32, HS = H / (2 * Operand<T>::V), LPR = H * (int)sizeof(T) / 16;
  static constexpr int NW = 32 * LPR / 64, NT = 64 * NW;                       // lanes for 32 receivers
  static constexpr int SROW = H * (int)sizeof(T) + 16, XBYTES = 32 * SROW;     // a tile as operand fragments, then its rows of z
  static constexpr int WBYTES = HS * MB * 1024, ABYTES = 2 * MB * 2 * 16 * 4;
  static constexpr int BYTES = WBYTES + ABYTES + 2 * XBYTES;
  static constexpr bool FITS = WBYTES <= 32 * 1024;
  static constexpr int PER_CU = 2;
};
struct GatNext {                 // of the next round
  const void *Ws;
  const float *a_src, *a_dst;
  void *z;
  float *s_src, *s_dst;
};
template <typename T, int H>
__global__ __launch_bounds__((GatRound<T, H>::NT), (GatRound<T, H>::PER_CU * GatRound<T, H>::NW / 4)) void gat_round_kernel(const GatArgs a, const GatNext next) {
  touch_args(a);
  using Opd = Operand<T>;
  using vec = typename Opd::vec;
  using S = GatRound<T, H>;
  constexpr int VEC = 16 / (int)sizeof(T), MB = S::MB, HS = S::HS, NT = S::NT;
  extern __shared__ __align__(16) char smem[];
  vec *Wl = (vec *)smem;                                             // [HS][MB][64]
  float(*al)[MB][2][16] = (float(*)[MB][2][16])(smem + S::WBYTES);   // a_src, a_dst in accumulator order
  char *xbuf = smem + S::WBYTES + S::ABYTES;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nbx = gridDim.x / 8, xcd = blockIdx.x % 8, lid = blockIdx.x / 8;
  const int64_t n_wt = (a.n_rows + 31) / 32, per_xcd = (n_wt + 7) / 8, t_begin = xcd * per_xcd;
  const int64_t t_end = t_begin + per_xcd < n_wt ? t_begin + per_xcd : n_wt;
  int64_t wt = t_begin + lid;
  if (wt >= t_end) return;                                           // (the whole block)
  {
    constexpr int NF = HS * MB * 64, C = (NF + NT - 1) / NT;
    const vec *W = (const vec *)next.Ws;
    vec t[C];
#pragma unroll
    for (int c = 0; c < C; ++c) t[c] = W[tid + c * NT < NF ? tid + c * NT : 0];
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (tid + c * NT < NF) Wl[tid + c * NT] = t[c];
    if (tid < MB * 32) {
      const int f = 32 * (tid / 32) + acc_row(tid % 16, (tid / 16) % 2);
      al[0][tid / 32][(tid / 16) % 2][tid % 16] = next.a_src[f];
      al[1][tid / 32][(tid / 16) % 2][tid % 16] = next.a_dst[f];
    }
  }
  const int row = tid / S::LPR, piece = tid % S::LPR, c = piece * VEC;
  int turn = 0, buf = 0;
  for (; wt < t_end; wt += nbx) {
    asm volatile("" ::: "memory");                           // (W's fragments are read from LDS in every tile)
    char *x = xbuf + buf * S::XBYTES;
    const int64_t row0 = wt * 32;
    const int64_t n = row0 + row < a.n_rows ? row0 + row : a.n_rows - 1;
    float r[VEC];
    gat_aggregate_row<T, VEC>(a, H, n, c, r);
    T *f = (T *)(x + ((size_t)(piece / 2) * 64 + (piece & 1) * 32 + row) * 16);   // piece 2 s + g of a row: slab s, lane group g
#pragma unroll
    for (int q = 0; q < VEC / 4; ++q) store4<T>(f + 4 * q, r + 4 * q);
    if (a.out && row0 + row < a.n_rows) {
      T *o = (T *)a.out + (size_t)n * H + c;
#pragma unroll
      for (int q = 0; q < VEC / 4; ++q) store4<T>(o + 4 * q, r + 4 * q);
    }
    __syncthreads();
    if (wave == turn) {
      vec h[HS];
#pragma unroll
      for (int s = 0; s < HS; ++s) h[s] = *(const vec *)(x + ((size_t)s * 64 + lane) * 16);
      wave_lds_fence();
      float ps = 0.f, pd = 0.f;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int s = 0; s < HS; ++s) Opd::mma(Wl[(s * MB + mb) * 64 + lane], h[s], acc);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          ps = fmaf(acc[i], al[0][mb][g][i], ps);
          pd = fmaf(acc[i], al[1][mb][g][i], pd);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[4] = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
          store4<T>((T *)(x + l32 * S::SROW) + 32 * mb + 8 * q + 4 * g, v);
        }
      }
      ps += __shfl_xor(ps, 32);                              // the row's other half of the features
      pd += __shfl_xor(pd, 32);
      if (g == 0 && row0 + l32 < a.n_rows) {
        next.s_src[row0 + l32] = ps;
        next.s_dst[row0 + l32] = pd;
      }
      wave_lds_fence();
      constexpr int RPI = 64 / S::LPR;
#pragma unroll
      for (int i = 0; i < 32 / RPI; ++i) {
        const int rr = i * RPI + lane / S::LPR, p = lane % S::LPR;
        const f32x4 v = *(const f32x4 *)(x + rr * S::SROW + p * 16);
        if (row0 + rr < a.n_rows) *(f32x4 *)((char *)((T *)next.z + (size_t)(row0 + rr) * H) + p * 16) = v;
      }
    }
    turn = turn + 1 == S::NW ? 0 : turn + 1;
    buf ^= 1;
  }
}

// ---------------------------------------------------------------------------------------------
// Backward of the attention round. With dpre = dh' * [h' > 0] and, per receiver i, the softmax
// weights alpha over its in-edges k (sender j_k) and its self edge:
//   d alpha_k = dpre_i . z_{j_k},   sum_m alpha_m d alpha_m = dpre_i . pre_i = dpre_i . h'_i,
//   d u_k = alpha_k (d alpha_k - dpre_i . h'_i) * LeakyReLU'(u_k),   u_k = s_src[j_k] + s_dst[i],
//   dz_j = alpha_self,j dpre_j + sum over j's out-edges of alpha_k dpre_{i_k}
//          + a_src * (d u_self,j + sum over out-edges d u_k) + a_dst * (d u_self,j + sum over in-edges d u_k),
//   d a_src = sum_n d_ss[n] z_n,  d a_dst = sum_n d_sd[n] z_n,  dh = dz W^T,  dW = h^T dz.
struct GatBwdArgs {
  int64_t n_rows;
  const void *z, *hout, *dout;   // [N, H] operand type: saved z and h' of the round, upstream d h'
  const float *s_src, *s_dst;    // [N] saved scores
  const float *a_src, *a_dst;    // [H]
  const int32_t *in_ptr, *in_src, *in_dst, *out_ptr, *out_pos;
  const void *zero_row;          // 1 KB of zeros
  float *alpha_e, *du_e;         // [E], receiver order
  float *alpha_s, *du_s;         // [N] self edge
  float *d_ss, *d_sd;            // [N] d / d s_src[n], d / d s_dst[n]
  void *dpre, *dz;               // [N, H] operand type
};

// sum over the `width` lanes of a lane group (width a power of two, groups aligned)
__device__ __forceinline__ float group_sum(float v, int width) {
  for (int o = width >> 1; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Per receiver (a group of H / VEC lanes, each a 16-byte column slice): dpre, the softmax weights
// of its in-edges and self edge, and the gradients of their scores. Edges in order.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void gat_bwd_scores_kernel(const GatBwdArgs a, int H) {
  touch_args(a);
  const int lpr = H / VEC;
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t n = gt / lpr;
  const bool live = n < a.n_rows;                      // (whole groups; idle groups follow along for the shuffles)
  if (!live) n = a.n_rows - 1;
  const int c = (int)(gt % lpr) * VEC;
  const T *z = (const T *)a.z;
  const int e0 = a.in_ptr[n], e1 = a.in_ptr[n + 1];
  GatAhead<T, VEC> ahead;
  ahead.request(z, (const T *)a.zero_row, a.s_src, a.in_src, n, e0, e1, c, H);
  float dp[VEC], hv[VEC], v[VEC];
  RowVec<T, VEC>::load((const T *)a.dout + (size_t)n * H + c, dp);
  RowVec<T, VEC>::load((const T *)a.hout + (size_t)n * H + c, hv);
  RowVec<T, VEC>::load(z + (size_t)n * H + c, v);
  const float sd = a.s_dst[n];
  const float u_self = a.s_src[n] + sd, s_self = leaky02(u_self);
  float ci = 0.f, da = 0.f, d[kGatAhead];
#pragma unroll
  for (int k = 0; k < kGatAhead; ++k) d[k] = 0.f;
#pragma unroll
  for (int j = 0; j < VEC; ++j) {
    dp[j] = hv[j] > 0.f ? dp[j] : 0.f;
    ci = fmaf(dp[j], hv[j], ci);
    da = fmaf(dp[j], v[j], da);
#pragma unroll
    for (int k = 0; k < kGatAhead; ++k) d[k] = fmaf(dp[j], ahead.v[k][j], d[k]);
  }
  ci = group_sum(ci, lpr);
  da = group_sum(da, lpr);
#pragma unroll
  for (int k = 0; k < kGatAhead; ++k) d[k] = group_sum(d[k], lpr);
  if (live) {
#pragma unroll
    for (int q = 0; q < VEC / 4; ++q) store4<T>((T *)a.dpre + (size_t)n * H + c + 4 * q, dp + 4 * q);
  }
  float u[kGatAhead], mx = s_self;
#pragma unroll
  for (int k = 0; k < kGatAhead; ++k) {
    u[k] = ahead.s[k] + sd;
    mx = e0 + k < e1 ? fmaxf(mx, leaky02(u[k])) : mx;
  }
  for (int e = e0 + kGatAhead; e < e1; ++e) mx = fmaxf(mx, leaky02(a.s_src[a.in_src[e]] + sd));
  float den = expf(s_self - mx);
#pragma unroll
  for (int k = 0; k < kGatAhead; ++k) den += e0 + k < e1 ? expf(leaky02(u[k]) - mx) : 0.f;
  for (int e = e0 + kGatAhead; e < e1; ++e) den += expf(leaky02(a.s_src[a.in_src[e]] + sd) - mx);
  const float inv = 1.f / den;
  // self edge
  const float al_s = expf(s_self - mx) * inv;
  const float du_s = al_s * (da - ci) * (u_self > 0.f ? 1.f : 0.2f);
  float dsd = du_s;
  auto edge = [&](int e, float uk, float dk) {
    const float al = expf(leaky02(uk) - mx) * inv;
    const float du = al * (dk - ci) * (uk > 0.f ? 1.f : 0.2f);
    dsd += du;
    if (live && c == 0) { a.alpha_e[e] = al; a.du_e[e] = du; }
  };
#pragma unroll
  for (int k = 0; k < kGatAhead; ++k)
    if (e0 + k < e1) edge(e0 + k, u[k], d[k]);
  for (int e = e0 + kGatAhead; e < e1; ++e) {
    const int s = a.in_src[e];
    RowVec<T, VEC>::load(z + (size_t)s * H + c, v);
    float dk = 0.f;
#pragma unroll
    for (int j = 0; j < VEC; ++j) dk = fmaf(dp[j], v[j], dk);
    edge(e, a.s_src[s] + sd, group_sum(dk, lpr));
  }
  if (live && c == 0) { a.alpha_s[n] = al_s; a.du_s[n] = du_s; a.d_sd[n] = dsd; }
}

// Per sender j (a group of H / VEC lanes): dz_j from its self edge, its out-edges (receiver-order
// positions out_pos[k], ascending) and the two score gradients; also d_ss[j].
template <typename T, int VEC>
__global__ __launch_bounds__(256) void gat_bwd_dz_kernel(const GatBwdArgs a, int H) {
  touch_args(a);
  const int lpr = H / VEC;
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n = gt / lpr;
  if (n >= a.n_rows) return;
  const int c = (int)(gt - n * lpr) * VEC;
  const T *dpre = (const T *)a.dpre;
  float acc[VEC], v[VEC];
  RowVec<T, VEC>::load(dpre + (size_t)n * H + c, v);
  const float al_s = a.alpha_s[n];
#pragma unroll
  for (int j = 0; j < VEC; ++j) acc[j] = al_s * v[j];
  float dss = a.du_s[n];
  const int k0 = a.out_ptr[n], k1 = a.out_ptr[n + 1];
  for (int k = k0; k < k1; ++k) {
    const int e = a.out_pos[k];
    const float al = a.alpha_e[e];
    dss += a.du_e[e];
    RowVec<T, VEC>::load(dpre + (size_t)a.in_dst[e] * H + c, v);
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc[j] = fmaf(al, v[j], acc[j]);
  }
  const float dsd = a.d_sd[n];
#pragma unroll
  for (int j = 0; j < VEC; ++j) acc[j] += dss * a.a_src[c + j] + dsd * a.a_dst[c + j];
#pragma unroll
  for (int q = 0; q < VEC / 4; ++q) store4<T>((T *)a.dz + (size_t)n * H + c + 4 * q, acc + 4 * q);
  if (c == 0) a.d_ss[n] = dss;
}

// Partial sums of d a_src = sum_n d_ss[n] z_n and d a_dst = sum_n d_sd[n] z_n over a chunk of rows
// per block: partial[chunk][2][H]. Threads = H / VEC column slices x 256 / (H / VEC) row groups;
// a group walks its rows in order and the groups are added in group order (fixed order).
template <typename T, int VEC>
__global__ __launch_bounds__(256) void gat_avec_grad_kernel(const T *z, const float *d_ss, const float *d_sd,
                                                            int64_t n_rows, int rows_per_chunk, int H,
                                                            float *partial) {
  extern __shared__ __align__(16) float sm[];               // [groups][2][H]
  const int lpr = H / VEC, ng = 256 / lpr, t = threadIdx.x, c = (t % lpr) * VEC, q = t / lpr;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_chunk;
  int64_t r1 = r0 + rows_per_chunk;
  if (r1 > n_rows) r1 = n_rows;
  float as[VEC], ad[VEC], v[VEC];
#pragma unroll
  for (int j = 0; j < VEC; ++j) { as[j] = 0.f; ad[j] = 0.f; }
  for (int64_t r = r0 + q; r < r1; r += ng) {
    RowVec<T, VEC>::load(z + (size_t)r * H + c, v);
    const float ws = d_ss[r], wd = d_sd[r];
#pragma unroll
    for (int j = 0; j < VEC; ++j) { as[j] = fmaf(ws, v[j], as[j]); ad[j] = fmaf(wd, v[j], ad[j]); }
  }
#pragma unroll
  for (int j = 0; j < VEC; ++j) { sm[(q * 2) * H + c + j] = as[j]; sm[(q * 2 + 1) * H + c + j] = ad[j]; }
  __syncthreads();
  for (int i = t; i < 2 * H; i += 256) {
    float s = sm[i];
    for (int k = 1; k < ng; ++k) s += sm[(size_t)k * 2 * H + i];
    partial[(size_t)blockIdx.x * 2 * H + i] = s;
  }
}
