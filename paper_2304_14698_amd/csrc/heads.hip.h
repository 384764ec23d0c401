// Small fp32 kernels on per-graph and per-state data: the readout MLP of the global-update layer
// (Section 3.4), the policy and value heads with invalid-action masking (Section 3.3.2), and
// their backward passes. G and S rows only -- latency-bound, plain vector ALU code.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>
#include "segsum.hip.h"

// Up to three affine layers over rows of [in1 | in2]; ReLU after every layer except, when
// relu_last == 0, the last. Optionally stores every layer's output (post-activation) for the
// backward pass: act[l] is [n_rows, d_out[l]].
struct RowMlpArgs {
  int n_layers, relu_last;
  const float *W[3], *b[3];
  int d_in[3], d_out[3];
  const float *in1, *in2;  // in2 nullable
  int w1, w2;              // widths of in1 / in2; w1 + w2 == d_in[0]
  int64_t n_rows;
  float *out;              // [n_rows, d_out[last]]
  float *act[3];           // nullable each
};

// ROWS rows (row .. row + ROWS - 1, those below a.n_rows stored) through the layers of `a`, all 256 threads of the block
// cooperating. These kernels are bound by memory latency and, from about two blocks per compute unit on, by
// every block reading all the weights from L2; so a layer's weights are requested in as few dependent
// rounds as possible, and several rows share them where there are rows enough: with d_out a multiple of 4 (and the
// matrix 16-byte aligned) a thread owns four adjacent outputs and one of 256 / (d_out / 4) slices of the
// contraction, loads its weights 16 bytes at a time, sixteen loads in flight (a remainder as sixteen, eight or
// four, whose missing rows re-read the last one and count as zeros), and the slices' partial sums are added in slice
// order; other layers (a single output, say) split the contraction the same way with scalar loads. A row's
// sums do not depend on ROWS.
// cur holds the input rows (d_in[0] floats each, ld apart) on entry; cur/nxt: >= ROWS * ld floats, ld >= widest layer;
// part: ROWS * 1024 floats, 16-byte aligned. COHERENT_OUT stores a.out with device scope, for a consumer in
// another block of the same launch.
template <typename F>
__device__ __forceinline__ void in_batches(int k0, int k1, F f) {
  for (int k = k0; k < k1;) {
    if (k1 - k > 8) { f(k, std::integral_constant<int, 16>()); k += 16; }
    else if (k1 - k > 4) { f(k, std::integral_constant<int, 8>()); k += 8; }
    else { f(k, std::integral_constant<int, 4>()); k += 4; }
  }
}
template <bool COHERENT_OUT = false>
__device__ __forceinline__ void store_row_out(float *p, float y) {
  if constexpr (COHERENT_OUT) __hip_atomic_store(p, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = y;
}

template <bool COHERENT_OUT = false, int ROWS = 1>
__device__ __forceinline__ void block_row_mlp(const RowMlpArgs &a, float *cur, float *nxt, float *part,
                                              int64_t row, int ld = 0) {
  const int t = threadIdx.x;
  for (int l = 0; l < a.n_layers; ++l) {
    const int din = a.d_in[l], dout = a.d_out[l];
    const bool relu = a.relu_last || (l + 1 < a.n_layers);
    const float *W = a.W[l];
    auto finish = [&](int r, int f, float v) {
      v += a.b[l][f];
      const float y = relu ? fmaxf(v, 0.f) : v;
      nxt[r * ld + f] = y;
      if (ROWS == 1 || row + r < a.n_rows) {
        if (a.act[l]) a.act[l][(row + r) * dout + f] = y;
        if (l + 1 == a.n_layers) store_row_out<COHERENT_OUT>(a.out + (row + r) * dout + f, y);
      }
    };
    if ((dout & 3) == 0 && dout <= 1024 && ((uintptr_t)W & 15) == 0) {
      const int fq = dout >> 2;                           // 16-byte columns
      int KQ = 256 / fq;                                  // slices of the contraction
      if (KQ > din) KQ = din;
      const int kc = (din + KQ - 1) / KQ;
      const int fl = t % fq, kq = t / fq;
      if (kq < KQ) {
        const int k0 = kq * kc, k1 = (k0 + kc) < din ? (k0 + kc) : din;
        float4 acc[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] = make_float4(0.f, 0.f, 0.f, 0.f);
        in_batches(k0, k1, [&](int k, auto batch) {
          constexpr int U = decltype(batch)::value;
          float4 w[U];
#pragma unroll
          for (int i = 0; i < U; ++i) {
            const unsigned at = (unsigned)((k + i < k1 ? k + i : k1 - 1) * fq + fl) * 16u;   // (32 bits: one register each)
            w[i] = *(const float4 *)((const char *)W + at);
            if (k + i >= k1) w[i] = make_float4(0.f, 0.f, 0.f, 0.f);
          }
#pragma unroll
          for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int i = 0; i < U; ++i) {
              const float x = k + i < k1 ? cur[r * ld + k + i] : 0.f;
              acc[r].x = fmaf(x, w[i].x, acc[r].x); acc[r].y = fmaf(x, w[i].y, acc[r].y);
              acc[r].z = fmaf(x, w[i].z, acc[r].z); acc[r].w = fmaf(x, w[i].w, acc[r].w);
            }
        });
#pragma unroll
        for (int r = 0; r < ROWS; ++r) ((float4 *)part)[r * 256 + kq * fq + fl] = acc[r];
      }
      __syncthreads();
      for (int i = t; i < ROWS * dout; i += 256) {
        const int r = i / dout, f = i - r * dout;
        float v = part[r * 1024 + f];
        for (int q = 1; q < KQ; ++q) v += part[r * 1024 + q * dout + f];
        finish(r, f, v);
      }
      __syncthreads();
    } else {
      int fw = 256;                                       // outputs handled per pass
      while (fw / 2 >= dout && 256 / (fw / 2) <= din) fw /= 2;
      const int KQ = 256 / fw;                            // thread groups splitting the contraction
      const int kc = (din + KQ - 1) / KQ;
      const int fl = t % fw, kq = t / fw;
      const int k0 = kq * kc, k1 = (k0 + kc) < din ? (k0 + kc) : din;
      for (int f0 = 0; f0 < dout; f0 += fw) {
        const int f = f0 + fl;
        float acc[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[r] = 0.f;
        if (f < dout)
          in_batches(k0, k1, [&](int k, auto batch) {
            constexpr int U = decltype(batch)::value;
            float w[U];
#pragma unroll
            for (int i = 0; i < U; ++i) {
              w[i] = W[(size_t)(k + i < k1 ? k + i : k1 - 1) * dout + f];
              if (k + i >= k1) w[i] = 0.f;
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
              for (int i = 0; i < U; ++i) acc[r] = fmaf(k + i < k1 ? cur[r * ld + k + i] : 0.f, w[i], acc[r]);
          });
        if (KQ > 1) {
#pragma unroll
          for (int r = 0; r < ROWS; ++r) part[r * 1024 + t] = acc[r];
          __syncthreads();
          for (int i = t; i < ROWS * fw; i += 256) {
            const int r = i / fw, fi = i - r * fw;
            if (f0 + fi >= dout) continue;
            float v = part[r * 1024 + fi];
            for (int q = 1; q < KQ; ++q) v += part[r * 1024 + q * fw + fi];
            finish(r, f0 + fi, v);
          }
          __syncthreads();
        } else if (f < dout) {
#pragma unroll
          for (int r = 0; r < ROWS; ++r) finish(r, f, acc[r]);
        }
      }
      __syncthreads();
    }
    float *tmp = cur; cur = nxt; nxt = tmp;
  }
}

// One, two or four rows per block by block_row_mlp; eight with a thread per output, which is enough from 4096 rows on.
template <int ROWMLP_ROWS>
__global__ __launch_bounds__(256) void rowmlp_kernel(const RowMlpArgs a) {
  // two buffers of ROWMLP_ROWS * dmax floats; up to four rows per block, 1024 floats of partial sums a row first
  extern __shared__ __align__(16) float sm[];
  int dmax = a.d_in[0];
  for (int l = 0; l < a.n_layers; ++l) dmax = a.d_out[l] > dmax ? a.d_out[l] : dmax;
  float *cur = sm + (ROWMLP_ROWS <= 4 ? ROWMLP_ROWS * 1024 : 0), *nxt = cur + ROWMLP_ROWS * dmax;
  const int64_t row0 = (int64_t)blockIdx.x * ROWMLP_ROWS;
  for (int i = threadIdx.x; i < ROWMLP_ROWS * a.d_in[0]; i += blockDim.x) {
    const int r = i / a.d_in[0], k = i - r * a.d_in[0];
    const int64_t row = row0 + r;
    float v = 0.f;
    if (row < a.n_rows) v = k < a.w1 ? a.in1[row * a.w1 + k] : a.in2[row * a.w2 + (k - a.w1)];
    cur[r * dmax + k] = v;
  }
  __syncthreads();
  if constexpr (ROWMLP_ROWS <= 4) {
    block_row_mlp<false, ROWMLP_ROWS>(a, cur, nxt, sm, row0, dmax);
    return;
  }
  for (int l = 0; l < a.n_layers; ++l) {
    const int din = a.d_in[l], dout = a.d_out[l];
    const bool relu = a.relu_last || (l + 1 < a.n_layers);
    for (int f = threadIdx.x; f < dout; f += blockDim.x) {
      float acc[ROWMLP_ROWS];
      const float bv = a.b[l][f];
#pragma unroll
      for (int r = 0; r < ROWMLP_ROWS; ++r) acc[r] = bv;
#pragma unroll 16
      for (int k = 0; k < din; ++k) {
        const float w = a.W[l][(size_t)k * dout + f];
#pragma unroll
        for (int r = 0; r < ROWMLP_ROWS; ++r) acc[r] = fmaf(cur[r * dmax + k], w, acc[r]);
      }
#pragma unroll
      for (int r = 0; r < ROWMLP_ROWS; ++r) {
        const float y = relu ? fmaxf(acc[r], 0.f) : acc[r];
        nxt[r * dmax + f] = y;
        const int64_t row = row0 + r;
        if (row < a.n_rows) {
          if (a.act[l]) a.act[l][row * dout + f] = y;
          if (l + 1 == a.n_layers) a.out[row * dout + f] = y;
        }
      }
    }
    __syncthreads();
    float *t = cur; cur = nxt; nxt = t;
  }
}

// Global-update layer (Section 3.4) for one graph per block: the sum (or mean) of the graph's node
// states, then the readout MLP on [pool | global attrs], without leaving the block. The 256
// threads form 256 / (H / VEC) row groups, each lane owning a 16-byte column slice; a group
// takes every (number of groups)-th node with eight loads in flight, and the groups' partial
// sums are added in group order, so the result does not depend on timing. pool [G, H] is also
// stored (it is an input of the backward pass). Meant for batches of many graphs of moderate
// size; a few huge graphs go through the generic segment-sum kernels instead.
// MAPPED: row_of[n] is the row of h that holds node n's state (else row n).
// (sm: (256 * VEC + 2 * widest layer) floats of LDS; all 256 threads of the block call it together.
// UF = loads a thread keeps in flight: a thread adds its rows in the same order whatever UF is.)
template <typename T, int VEC, int UF = 8, bool MAPPED = false>
__device__ __forceinline__ void graph_readout_block(const T *h, const int n0, const int n1, const int g, int H,
                                                    int mean, float *pool, const RowMlpArgs &mlp, float *sm,
                                                    const int32_t *row_of = nullptr) {
  const int t = threadIdx.x;
  const int tpr = H / VEC, ng = 256 / tpr, c0 = (t % tpr) * VEC, q = t / tpr;
  float acc[VEC];
#pragma unroll
  for (int j = 0; j < VEC; ++j) acc[j] = 0.f;
  int n = n0 + q;
  for (; n + (UF - 1) * ng < n1; n += UF * ng) {
    float v[UF][VEC];
#pragma unroll
    for (int i = 0; i < UF; ++i) {
      const int r = n + i * ng;
      RowVec<T, VEC>::load(h + (size_t)(MAPPED ? row_of[r] : r) * H + c0, v[i]);
    }
#pragma unroll
    for (int i = 0; i < UF; ++i)
#pragma unroll
      for (int j = 0; j < VEC; ++j) acc[j] += v[i][j];
  }
  if (n < n1) {
    // the last, partial round: the same loads in flight (rows past the end re-read the graph's
    // last row and are left out of the sum), not one dependent load after another
    float v[UF][VEC];
#pragma unroll
    for (int i = 0; i < UF; ++i) {
      const int r = n + i * ng;
      const int rc = r < n1 ? r : n1 - 1;
      RowVec<T, VEC>::load(h + (size_t)(MAPPED ? row_of[rc] : rc) * H + c0, v[i]);
    }
#pragma unroll
    for (int i = 0; i < UF; ++i)
#pragma unroll
      for (int j = 0; j < VEC; ++j) acc[j] += n + i * ng < n1 ? v[i][j] : 0.f;
  }
#pragma unroll
  for (int j = 0; j < VEC; ++j) sm[(q * tpr + t % tpr) * VEC + j] = acc[j];
  __syncthreads();
  int dmax = mlp.d_in[0];
  for (int l = 0; l < mlp.n_layers; ++l) dmax = mlp.d_out[l] > dmax ? mlp.d_out[l] : dmax;
  float *cur = sm + 256 * VEC, *nxt = cur + dmax, *part = sm;   // (the partial sums are dead by then)
  const float scale = mean ? 1.f / (float)(n1 - n0 > 1 ? n1 - n0 : 1) : 1.f;
  for (int f = t; f < H; f += 256) {
    float a = sm[f];
    for (int k = 1; k < ng; ++k) a += sm[k * H + f];
    a *= scale;
    pool[(size_t)g * H + f] = a;
    cur[f] = a;
  }
  for (int k = t; k < mlp.w2; k += 256) cur[H + k] = mlp.in2[(size_t)g * mlp.w2 + k];
  __syncthreads();
  block_row_mlp(mlp, cur, nxt, part, g);
}

// (five blocks per compute unit: 1040 graphs take 20.3 us so and 25.8 with four)
template <typename T, int VEC, int UF, bool MAPPED>
__global__ __launch_bounds__(256, 5) void graph_readout_kernel(const T *h, const int32_t *graph_node_ptr, int H,
                                                            int mean, float *pool, const RowMlpArgs mlp,
                                                            const int32_t *row_of) {
  extern __shared__ __align__(16) float sm[];   // [256 * VEC] partial sums, then the MLP's buffers
  const int g = blockIdx.x;
  graph_readout_block<T, VEC, UF, MAPPED>(h, graph_node_ptr[g], graph_node_ptr[g + 1], g, H, mean, pool, mlp, sm, row_of);
}

// pool[g, :] /= max(n_g, 1)  (mean readout)
__global__ void mean_scale_kernel(float *pool, const int32_t *graph_node_ptr, int64_t G, int H,
                                  int inverse_only_grad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= G * H) return;
  const int64_t g = i / H;
  const int n = graph_node_ptr[g + 1] - graph_node_ptr[g];
  pool[i] = pool[i] / (float)(n > 1 ? n : 1);
}

// Block-wide reductions over 256 threads in a fixed order: inside a wave by exchange, then the four waves' in order.
// red: 8 words of LDS (the result is read by all before it is written again).
__device__ __forceinline__ float block_sum(float v, float *red) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const float r = ((red[0] + red[1]) + red[2]) + red[3];
  __syncthreads();
  return r;
}
struct BestSlot {
  float value;
  int index;             // lowest index that has it
};
__device__ __forceinline__ BestSlot better(const BestSlot &a, const BestSlot &b) {
  return b.value > a.value || (b.value == a.value && b.index < a.index) ? b : a;
}
__device__ __forceinline__ BestSlot block_best(BestSlot b, float *red) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const BestSlot other{__shfl_xor(b.value, o), __shfl_xor(b.index, o)};
    b = better(b, other);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[w] = b.value; red[4 + w] = __int_as_float(b.index); }
  __syncthreads();
  for (int k = 0; k < 4; ++k) b = better(b, BestSlot{red[k], __float_as_int(red[4 + k])});
  __syncthreads();
  return b;
}
// A state's masked log-softmax, entropy and first-max action from its slots' logits (ld: reads one).
template <typename Load>
__device__ __forceinline__ float state_softmax(Load ld, const uint8_t *mask, int j0, int j1, float *logp, float *entropy, int32_t *action,
                                               float *red) {
  const int t = threadIdx.x;
  BestSlot best{-INFINITY, 0x7fffffff};
  for (int j = j0 + t; j < j1; j += 256)
    if (mask[j]) best = better(best, BestSlot{ld(j), j});
  best = block_best(best, red);
  float se = 0.f;
  int cnt = 0;
  for (int j = j0 + t; j < j1; j += 256)
    if (mask[j]) { se += expf(ld(j) - best.value); ++cnt; }
  const float lse = best.value + logf(block_sum(se, red));
  const float nvalid = block_sum((float)cnt, red);
  float ent = 0.f;
  for (int j = j0 + t; j < j1; j += 256) {
    if (mask[j]) {
      const float lp = ld(j) - lse;
      logp[j] = lp;
      ent -= expf(lp) * lp;
    } else {
      logp[j] = -INFINITY;
    }
  }
  ent = block_sum(ent, red);
  if (t == 0) { *entropy = ent; *action = best.index - j0; }
  return nvalid;
}

// One block per state: masked log-softmax over the state's slots, entropy, first-max action,
// the mean embedding of the valid slots and, on it, the value head (value.n_layers == 0 skips it).
__global__ __launch_bounds__(256) void state_policy_kernel(
    const float *logit, const uint8_t *mask, const int32_t *state_graph_ptr, const float *emb,
    int H, float *logp, float *entropy, int32_t *action, float *zmean, const RowMlpArgs value) {
  __shared__ float red[8];
  __shared__ __align__(16) float zbuf[1024];                      // partial sums of the mean embedding
  __shared__ __align__(16) float vcur[512], vnxt[512];            // value head: layer input / output
  const int s = blockIdx.x, t = threadIdx.x;
  const int j0 = state_graph_ptr[s], j1 = state_graph_ptr[s + 1];
  const float nvalid = state_softmax([&](int j) { return logit[j]; }, mask, j0, j1, logp, entropy + s, action + s, red);
  // mean embedding of the valid slots: H / 4 threads cover a row with 16-byte loads, the 1024 / H
  // thread groups take every (1024/H)-th slot, eight loads in flight each; the groups' partial
  // sums are combined in group order
  const int tpr = H / 4, ng = 256 / tpr, c4 = (t % tpr) * 4, q = t / tpr;     // H is 64, 128 or 256
  float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int j = j0 + q; j < j1; j += 8 * ng) {
    float4 v[8];
    bool on[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int ji = j + i * ng < j1 ? j + i * ng : j;
      v[i] = *(const float4 *)(emb + (size_t)ji * H + c4);
      on[i] = j + i * ng < j1 && mask[ji];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (on[i]) { p.x += v[i].x; p.y += v[i].y; p.z += v[i].z; p.w += v[i].w; }
  }
  float4 *zp = (float4 *)zbuf;                                   // [ng][H / 4]
  zp[t] = p;
  __syncthreads();
  if (t < tpr) {
    float4 acc = zp[t];
    for (int k = 1; k < ng; ++k) {
      const float4 o = zp[k * tpr + t];
      acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w;
    }
    acc.x /= nvalid; acc.y /= nvalid; acc.z /= nvalid; acc.w /= nvalid;
    *(float4 *)(zmean + (size_t)s * H + c4) = acc;
    *(float4 *)(vcur + c4) = acc;
  }
  __syncthreads();
  // value head on the mean embedding (Section 3.3.2), in the same block
  if (value.n_layers > 0) block_row_mlp(value, vcur, vnxt, zbuf, s);
}

// Both heads in one launch for batches of at most a few thousand slots. The first blocks: the policy
// MLP of ROWS slots, of one or of several states; the block that finishes a state's last slot (a per-state
// counter, which it also resets) does that state's masked log-softmax, entropy and first-max action. The last
// S blocks: the mean embedding of a state's valid slots and the value head on it, independent of
// the policy blocks. Results are the same as rowmlp_kernel<1> followed by state_policy_kernel, for any ROWS.
// Logits cross blocks through device-scope stores and loads (each completed before the block's
// counter increment is issued), so no cache write-back or invalidation is needed. us before ROWS: 1040 slots of H = 128
// 31.6, now 22.6; 2096 slots 48 and 25.
template <int ROWS>
__global__ __launch_bounds__(256) void policy_value_kernel(
    const RowMlpArgs policy, const uint8_t *mask, const int32_t *state_graph_ptr, int G, int S, int H,
    int32_t *counter, float *logp, float *entropy, int32_t *action, float *zmean, const RowMlpArgs value) {
  constexpr int LD = 512;
  __shared__ __align__(16) float part[ROWS * 1024];
  __shared__ __align__(16) float bufa[ROWS * LD], bufb[ROWS * LD];
  __shared__ float red[8];
  __shared__ int redi[256];
  __shared__ int sh_state[ROWS], sh_done[ROWS], sh_n_done;
  const int t = threadIdx.x, policy_blocks = (G + ROWS - 1) / ROWS;
  if ((int)blockIdx.x >= policy_blocks) {
    // ---- value head of state s
    const int s = blockIdx.x - policy_blocks;
    const int j0 = state_graph_ptr[s], j1 = state_graph_ptr[s + 1];
    const float *emb = policy.in1;
    const int tpr = H / 4, ng = 256 / tpr, c4 = (t % tpr) * 4, q = t / tpr;   // H is 64, 128 or 256
    float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
    int cnt = 0;
    for (int j = j0 + q; j < j1; j += 8 * ng) {
      float4 v[8];
      bool on[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int ji = j + i * ng < j1 ? j + i * ng : j;
        v[i] = *(const float4 *)(emb + (size_t)ji * H + c4);
        on[i] = j + i * ng < j1 && mask[ji];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (on[i]) { p.x += v[i].x; p.y += v[i].y; p.z += v[i].z; p.w += v[i].w; ++cnt; }
    }
    ((float4 *)part)[t] = p;                                       // [ng][H / 4]
    redi[t] = cnt;
    __syncthreads();
    if (t < tpr) {
      float4 acc = ((float4 *)part)[t];
      int n = redi[0];
      for (int k = 1; k < ng; ++k) {
        const float4 o = ((float4 *)part)[k * tpr + t];
        acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w;
        n += redi[k * tpr];
      }
      const float nvalid = (float)n;
      acc.x /= nvalid; acc.y /= nvalid; acc.z /= nvalid; acc.w /= nvalid;
      *(float4 *)(zmean + (size_t)s * H + c4) = acc;
      *(float4 *)(bufa + c4) = acc;
    }
    __syncthreads();
    if (value.n_layers > 0) block_row_mlp(value, bufa, bufb, part, s);
    return;
  }
  // ---- policy MLP of the block's slots; meanwhile find their states
  const int slot0 = blockIdx.x * ROWS;
  if (t < ROWS) sh_state[t] = -1;
  for (int i = t; i < ROWS * H; i += 256) {
    const int r = i / H, k = i - r * H;
    bufa[r * LD + k] = slot0 + r < G ? policy.in1[(size_t)(slot0 + r) * H + k] : 0.f;
  }
  __syncthreads();
  for (int s = t; s < S; s += 256) {
    const int a = state_graph_ptr[s], z = state_graph_ptr[s + 1];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
      if (a <= slot0 + r && slot0 + r < z) sh_state[r] = s;
  }
  block_row_mlp<true, ROWS>(policy, bufa, bufb, part, slot0, LD);
  __builtin_amdgcn_s_waitcnt(0x0F70);                              // vmcnt(0): this wave's logit stores have completed
  __syncthreads();
  if (t == 0) {
    int n = 0;
    for (int r = 0; r < ROWS;) {                                   // the block's slots, state by state (-1: past the last slot)
      const int s = sh_state[r];
      int k = 1;
      while (r + k < ROWS && sh_state[r + k] == s) ++k;
      if (s >= 0) {
        const int slots = state_graph_ptr[s + 1] - state_graph_ptr[s];
        if (atomicAdd(&counter[s], k) + k == slots) {
          counter[s] = 0;                                          // ready for the next launch
          sh_done[n++] = s;
        }
      }
      r += k;
    }
    sh_n_done = n;
  }
  __syncthreads();
  const float *logit = policy.out;
  auto ld = [&](int i) { return __hip_atomic_load(logit + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  for (int i = 0; i < sh_n_done; ++i) {
    const int s = sh_done[i];
    (void)state_softmax(ld, mask, state_graph_ptr[s], state_graph_ptr[s + 1], logp, entropy + s, action + s, red);
  }
}

// dJ/dlogit per slot from (dlogp, dentropy) and the forward's logp/entropy; one block per state.
//   dlogit_k = c_k - p_k * sum_valid c  -  dent * p_k * (logp_k + entropy)      (0 when masked)
__global__ __launch_bounds__(256) void state_policy_bwd_kernel(
    const float *logp, const float *entropy, const uint8_t *mask, const int32_t *state_graph_ptr,
    const float *dlogp, const float *dentropy, float *dlogit, float *inv_nvalid) {
  __shared__ float red[8];
  const int s = blockIdx.x, t = threadIdx.x;
  const int j0 = state_graph_ptr[s], j1 = state_graph_ptr[s + 1];
  float cs = 0.f;
  int cnt = 0;
  for (int j = j0 + t; j < j1; j += 256)
    if (mask[j]) { cs += dlogp[j]; ++cnt; }
  cs = block_sum(cs, red);
  const float nvalid = block_sum((float)cnt, red);
  const float de = dentropy[s], ent = entropy[s];
  for (int j = j0 + t; j < j1; j += 256) {
    float d = 0.f;
    if (mask[j]) {
      const float lp = logp[j], p = expf(lp);
      d = dlogp[j] - p * cs - de * p * (lp + ent);
    }
    dlogit[j] = d;
  }
  if (t == 0) inv_nvalid[s] = 1.f / nvalid;
}

// Backward of rowmlp_kernel for up to three layers, a block for ROWMLP_ROWS rows:
// given dout [n_rows, d_out[last]] and the saved post-activation outputs act[l], computes the
// pre-activation gradients dz[l] (stored, for the weight-gradient pass) and dx [n_rows, d_in[0]].
struct RowMlpBwdArgs {
  int n_layers, relu_last;
  const float *W[3];
  int d_in[3], d_out[3];
  const float *act[3];   // saved outputs of each layer
  const float *dout;     // [n_rows, d_out[last]]
  int64_t n_rows;
  float *dz[3];          // [n_rows, d_out[l]]
  float *dx;             // [n_rows, d_in[0]] nullable
};

template <int ROWMLP_ROWS>
__device__ __forceinline__ void rowmlp_bwd_block(const RowMlpBwdArgs &a, int block, float *sm) {
  int dmax = a.d_in[0];
  for (int l = 0; l < a.n_layers; ++l) dmax = a.d_out[l] > dmax ? a.d_out[l] : dmax;
  float *cur = sm, *nxt = sm + ROWMLP_ROWS * dmax;
  const int64_t row0 = (int64_t)block * ROWMLP_ROWS;
  const int L = a.n_layers;
  // dz of the last layer
  {
    const int dout = a.d_out[L - 1];
    for (int i = threadIdx.x; i < ROWMLP_ROWS * dout; i += blockDim.x) {
      const int r = i / dout, f = i - r * dout;
      const int64_t row = row0 + r;
      float v = 0.f;
      if (row < a.n_rows) {
        v = a.dout[row * dout + f];
        if (a.relu_last && !(a.act[L - 1][row * dout + f] > 0.f)) v = 0.f;
        a.dz[L - 1][row * dout + f] = v;
      }
      cur[r * dmax + f] = v;
    }
  }
  __syncthreads();
  for (int l = L - 1; l >= 0; --l) {
    // dy_in[k] = sum_f dz[l][f] W[l][k, f]; then mask by layer l-1's activation
    const int din = a.d_in[l], dout = a.d_out[l];
    if (l == 0 && !a.dx) break;
    for (int k = threadIdx.x; k < din; k += blockDim.x) {
      float acc[ROWMLP_ROWS];
#pragma unroll
      for (int r = 0; r < ROWMLP_ROWS; ++r) acc[r] = 0.f;
      const float *wrow = a.W[l] + (size_t)k * dout;
      // aligned rows by 16-byte pieces, four in flight: us, 1040 rows of H = 128 19.1, now 15.9; 262 rows 15.9 and 13.6
      if ((dout & 15) == 0 && ((uintptr_t)a.W[l] & 15) == 0) {
        for (int f = 0; f < dout; f += 16) {
          f32x4 w[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) w[i] = *(const f32x4 *)(wrow + f + 4 * i);
#pragma unroll
          for (int r = 0; r < ROWMLP_ROWS; ++r)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r] = fmaf(cur[r * dmax + f + i], w[i / 4][i % 4], acc[r]);
        }
      } else {
#pragma unroll 8
        for (int f = 0; f < dout; ++f) {
          const float w = wrow[f];
#pragma unroll
          for (int r = 0; r < ROWMLP_ROWS; ++r) acc[r] = fmaf(cur[r * dmax + f], w, acc[r]);
        }
      }
#pragma unroll
      for (int r = 0; r < ROWMLP_ROWS; ++r) {
        const int64_t row = row0 + r;
        float v = acc[r];
        if (row < a.n_rows) {
          if (l > 0) {
            if (!(a.act[l - 1][row * din + k] > 0.f)) v = 0.f;
            a.dz[l - 1][row * din + k] = v;
          } else {
            a.dx[row * din + k] = v;
          }
        } else {
          v = 0.f;
        }
        nxt[r * dmax + k] = v;
      }
    }
    __syncthreads();
    float *t = cur; cur = nxt; nxt = t;
  }
}

// The rows of one MLP, ROWMLP_ROWS per block, and behind them those of a second one (other == 0 rows: none):
// the two heads' backward passes do not depend on each other. Every block reads all the weights from L2,
// which bounds the launch: several rows per block as soon as that leaves a block per compute unit
// (1040 rows of the policy head, H = 128: 32 us with a block per row and 14 us for the value head
// after it, 23 us together with four rows per block). A row's sums do not depend on it.
template <int ROWMLP_ROWS>
__global__ __launch_bounds__(256) void rowmlp_bwd_kernel(const RowMlpBwdArgs a, const RowMlpBwdArgs other) {
  extern __shared__ float sm[];
  const int blocks = (int)((a.n_rows + ROWMLP_ROWS - 1) / ROWMLP_ROWS);
  if ((int)blockIdx.x < blocks) rowmlp_bwd_block<ROWMLP_ROWS>(a, blockIdx.x, sm);
  else rowmlp_bwd_block<ROWMLP_ROWS>(other, (int)blockIdx.x - blocks, sm);
}

// Weight gradients of a few affine layers over G or S rows each, one launch for all of them:
//   dW[k, f] += sum_rows x[row, k] dz[row, f],  db[f] += sum_rows dz[row, f]
// x = [x1 | x2] (x2 nullable); k = d_in is the bias row (x = 1). A block owns a 64 x 64 tile of one layer's
// [d_in + 1, d_out] and one chunk of its rows; rows go through LDS sixteen at a time (the next sixteen
// requested before the products of these), and a thread holds 4 x 4 sums: two 16-byte LDS reads for
// sixteen products, where one thread per entry waited for two loads per product (H = 128, 1040 rows,
// 16 states: 250 us for the eight layers of heads and readout, a launch and a reduction each; here 32 us
// in four launches; 4624 rows, H = 256: 760 -> 81 us). With one chunk the sums
// are added to dW / db directly; with several, chunk c writes partial[c][k][f], which
// small_wgrad_reduce_kernel adds up in a fixed order.
constexpr int kWgradJobs = 6, kWgradTile = 64, kWgradStage = 16;
struct SmallWgradJob {
  const float *x1, *x2, *dz;
  int w1, w2, d_in, d_out;       // w1 + w2 == d_in
  int64_t n_rows;
  int rows_per_chunk, n_chunks, tiles_k, tiles_f;
  int block0, entry0;            // the launch's first block / the reduction's first block of this layer
  float *dW, *db, *partial;      // partial: nullptr with one chunk
};
struct SmallWgradArgs {
  int n_jobs;
  SmallWgradJob job[kWgradJobs];
};
__global__ __launch_bounds__(256) void small_wgrad_kernel(const SmallWgradArgs a) {
  __shared__ __align__(16) float xs[kWgradStage][kWgradTile], zs[kWgradStage][kWgradTile];
  int ji = 0;
  while (ji + 1 < a.n_jobs && (int)blockIdx.x >= a.job[ji + 1].block0) ++ji;
  const SmallWgradJob &j = a.job[ji];
  int q = (int)blockIdx.x - j.block0;
  const int f0 = (q % j.tiles_f) * kWgradTile;
  q /= j.tiles_f;
  const int k0 = (q % j.tiles_k) * kWgradTile, chunk = q / j.tiles_k;
  const int64_t r0 = (int64_t)chunk * j.rows_per_chunk;
  const int64_t r1 = r0 + j.rows_per_chunk < j.n_rows ? r0 + j.rows_per_chunk : j.n_rows;
  const int t = threadIdx.x, tk = 4 * (t >> 4), tf = 4 * (t & 15);
  const int col = t & 63, row4 = t >> 6;                    // staging: column `col` of rows row4, row4 + 4, ..
  const int k = k0 + col, f = f0 + col;
  const bool in_x = k < j.d_in, in_f = f < j.d_out;
  const float *xp = k < j.w1 ? j.x1 + k : (in_x ? j.x2 + (k - j.w1) : j.x1);
  const int xstride = k < j.w1 ? j.w1 : j.w2;
  const float xelse = k == j.d_in ? 1.f : 0.f;
  float xv[kWgradStage / 4], zv[kWgradStage / 4];
  auto request = [&](int64_t r) {
#pragma unroll
    for (int i = 0; i < kWgradStage / 4; ++i) {
      const int64_t ri = r + row4 + 4 * i;
      const bool on = ri < r1;
      const int64_t rc = on ? ri : r1 - 1;
      const float x = in_x ? xp[rc * xstride] : xelse;
      const float z = in_f ? j.dz[rc * j.d_out + f] : 0.f;
      xv[i] = on ? x : 0.f;
      zv[i] = on ? z : 0.f;
    }
  };
  float acc[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) acc[m][n] = 0.f;
  request(r0);
  for (int64_t r = r0; r < r1; r += kWgradStage) {
#pragma unroll
    for (int i = 0; i < kWgradStage / 4; ++i) {
      xs[row4 + 4 * i][col] = xv[i];
      zs[row4 + 4 * i][col] = zv[i];
    }
    __syncthreads();
    if (r + kWgradStage < r1) request(r + kWgradStage);
#pragma unroll
    for (int i = 0; i < kWgradStage; ++i) {
      const f32x4 x = *(const f32x4 *)&xs[i][tk], z = *(const f32x4 *)&zs[i][tf];
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[m][n] = fmaf(x[m], z[n], acc[m][n]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int ko = k0 + tk + m, fo = f0 + tf + n;
      if (ko > j.d_in || fo >= j.d_out) continue;
      if (j.partial) j.partial[((size_t)chunk * (j.d_in + 1) + ko) * j.d_out + fo] = acc[m][n];
      else if (ko == j.d_in) j.db[fo] += acc[m][n];
      else j.dW[(size_t)ko * j.d_out + fo] += acc[m][n];
    }
}
// dW / db += the chunks' sums, every entry in chunk order (eight loads in flight); layers of one chunk have no blocks
__global__ __launch_bounds__(256) void small_wgrad_reduce_kernel(const SmallWgradArgs a) {
  int ji = 0;
  while (ji + 1 < a.n_jobs && (int)blockIdx.x >= a.job[ji + 1].entry0) ++ji;
  const SmallWgradJob &j = a.job[ji];
  const int64_t i = (int64_t)((int)blockIdx.x - j.entry0) * 256 + threadIdx.x, n = (int64_t)(j.d_in + 1) * j.d_out;
  if (i >= n) return;
  float sum = 0.f;
  int c = 0;
  for (; c + 8 <= j.n_chunks; c += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = j.partial[(size_t)(c + u) * n + i];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += v[u];
  }
  for (; c < j.n_chunks; ++c) sum += j.partial[(size_t)c * n + i];
  const int64_t nw = (int64_t)j.d_in * j.d_out;
  if (i < nw) j.dW[i] += sum;
  else j.db[i - nw] += sum;
}

// Clipped-surrogate objective of Section 3.3.4 and its derivatives w.r.t. the heads' outputs, one
// block for the whole minibatch (S is a few hundred at most; the means are block reductions in a
// fixed order). dlogp must be zero on entry: only the taken slots are written. A recorded action
// outside its state's slots, or on a masked slot, touches nothing of that state and turns all
// four entries of J into NaN.
__global__ __launch_bounds__(256) void ppo_objective_kernel(
    const float *logp, const float *value, const float *entropy, const int32_t *state_graph_ptr,
    const uint8_t *mask, const int32_t *action, const float *old_logp, const float *advantage, const float *v_target,
    int S, float eps, float c1, float c2, float *J, float *dlogp, float *dvalue, float *dentropy) {
  __shared__ float red[8];
  const int t = threadIdx.x;
  const float inv = 1.f / (float)(S > 0 ? S : 1);
  float clip = 0.f, vf = 0.f, ent = 0.f, bad = 0.f;
  for (int s = t; s < S; s += 256) {
    const int j0 = state_graph_ptr[s], n_slots = state_graph_ptr[s + 1] - j0, act = action[s];
    if (act < 0 || act >= n_slots || !mask[j0 + act]) {
      bad = 1.f;
      dvalue[s] = 0.f;
      dentropy[s] = 0.f;
      continue;
    }
    const int j = j0 + act;
    const float A = advantage[s];
    const float ratio = expf(logp[j] - old_logp[s]);
    const float s1 = ratio * A;
    const float s2 = fminf(fmaxf(ratio, 1.f - eps), 1.f + eps) * A;
    clip -= fminf(s1, s2);
    dlogp[j] = s1 <= s2 ? -s1 * inv : 0.f;
    const float dv = value[s] - v_target[s];
    vf += dv * dv;
    dvalue[s] = 2.f * c1 * dv * inv;
    ent -= entropy[s];
    dentropy[s] = -c2 * inv;
  }
  clip = block_sum(clip, red) * inv;
  vf = block_sum(vf, red) * inv;
  ent = block_sum(ent, red) * inv;
  bad = block_sum(bad, red);
  if (t == 0) {
    const float nan = __int_as_float(0x7fc00000);
    J[0] = bad > 0.f ? nan : clip + c1 * vf + c2 * ent;
    J[1] = bad > 0.f ? nan : clip;
    J[2] = bad > 0.f ? nan : vf;
    J[3] = bad > 0.f ? nan : ent;
  }
}
