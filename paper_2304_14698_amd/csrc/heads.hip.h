// Small fp32 kernels on per-graph and per-state data beside the row-MLPs (rowmm.hip.h): their weight gradients and the
// objective of Section 3.3.4. G and S rows only -- latency-bound, plain vector ALU code.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>
#include "segsum.hip.h"

// pool[g, :] /= max(n_g, 1)  (mean readout)
__global__ void mean_scale_kernel(float *pool, const int32_t *graph_node_ptr, int64_t G, int H,
                                  int inverse_only_grad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= G * H) return;
  const int64_t g = i / H;
  const int n = graph_node_ptr[g + 1] - graph_node_ptr[g];
  pool[i] = pool[i] / (float)(n > 1 ? n : 1);
}

// Block-wide sum over 256 threads in a fixed order: inside a wave by exchange, then the four waves' in order.
// red: 4 words of LDS (the result is read by all before it is written again).
__device__ __forceinline__ float block_sum(float v, float *red) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const float r = ((red[0] + red[1]) + red[2]) + red[3];
  __syncthreads();
  return r;
}

// Weight gradients of a few affine layers over G or S rows each, one launch for all of them:
//   dW[k, f] += sum_rows x[row, k] dz[row, f],  db[f] += sum_rows dz[row, f]
// x = [x1 | x2] (x2 nullable). A block owns a 64 x 64 tile of one layer's matrix and one chunk of its rows, a quarter of which
// each wave multiplies on v_mfma_f32_16x16x4_f32 (fp32 operands and sums): four rows of 64 columns of x and of dz are one 16-byte load a
// lane each, whose element j is the operand of columns 4 i + j, so sixteen instructions follow two loads and nothing goes through
// LDS before the waves' sums are added, in order. Bound by the round trips of a launch: 32 rows a wave are in flight together. The
// blocks of a layer's first 64 rows of dW add up dz for db. With one chunk the sums are added to dW / db
// directly; with several, chunk c writes partial[c][k][f] (row d_in: db), which small_wgrad_reduce_kernel adds up in a fixed order.
// us with their reductions, before (vector code, rows through LDS) / now: 104 rows of H = 64 14 / 9, 1040 of H = 128 15 / 13, 4624 of
// H = 256 36 / 30.
constexpr int kWgradJobs = 6, kWgradTile = 64, kWgradFly = 8;
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
// What a slot's gradient lacks of the mean embedding's, kMeanRows slots a block: demb[j] = mask[j] ? demb[j] + dmean[s] * inv_valid[s] : 0,
// s the slot's state. Nothing of the weight gradients depends on it, nor it on them.
constexpr int kMeanRows = 64;
struct MeanShareArgs {
  float *demb;                   // [G, H]
  const float *dmean, *inv_valid;
  const uint8_t *mask;
  const int32_t *state_graph_ptr;
  int G, S, H;
  int block0;                    // the launch's first block of these
};
__device__ __forceinline__ void add_mean_share(const MeanShareArgs &a, int j0, int *state, float *share) {
  const int t = threadIdx.x, n = a.G - j0 < kMeanRows ? a.G - j0 : kMeanRows;
  if (t < n) {
    int lo = 0, hi = a.S;                     // state_graph_ptr[lo] <= j0 + t < state_graph_ptr[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (a.state_graph_ptr[mid] <= j0 + t) lo = mid; else hi = mid;
    }
    state[t] = lo;
    share[t] = a.mask[j0 + t] ? a.inv_valid[lo] : -1.f;
  }
  __syncthreads();
  const int q = a.H / 4, step = 256 / q, c = (t % q) * 4;
  for (int r = t / q; r < n; r += 4 * step) {
    f32x4 m[4], d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {             // (past the last row the last again, not stored)
      const int k = r + i * step < n ? r + i * step : n - 1;
      m[i] = *(const f32x4 *)(a.dmean + (size_t)state[k] * a.H + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) d[i][e] = a.demb[(size_t)(j0 + k) * a.H + c + e];      // (a caller's array: of any alignment)
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = r + i * step;
      if (k >= n) break;
      const float w = share[k];
#pragma unroll
      for (int e = 0; e < 4; ++e) a.demb[(size_t)(j0 + k) * a.H + c + e] = w >= 0.f ? d[i][e] + m[i][e] * w : 0.f;
    }
  }
}
__global__ __launch_bounds__(256) void small_wgrad_kernel(const SmallWgradArgs a, const MeanShareArgs mean) {
  __shared__ __align__(16) float sums[4][kWgradTile][kWgradTile];
  __shared__ float dz_sum[4][kWgradTile];
  touch_args(a);
  touch_args(mean);
  if ((int)blockIdx.x >= mean.block0) {
    add_mean_share(mean, ((int)blockIdx.x - mean.block0) * kMeanRows, (int *)sums, dz_sum[0]);
    return;
  }
  int ji = 0;
#pragma unroll
  for (int i = 1; i < kWgradJobs; ++i) ji += i < a.n_jobs && (int)blockIdx.x >= a.job[i].block0 ? 1 : 0;
  const SmallWgradJob &j = a.job[ji];
  int q = (int)blockIdx.x - j.block0;
  const int f0 = (q % j.tiles_f) * kWgradTile;
  q /= j.tiles_f;
  const int k0 = (q % j.tiles_k) * kWgradTile, chunk = q / j.tiles_k;
  const int64_t r0 = (int64_t)chunk * j.rows_per_chunk;
  const int64_t r1 = r0 + j.rows_per_chunk < j.n_rows ? r0 + j.rows_per_chunk : j.n_rows;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), c16 = lane & 15, q4 = lane >> 4;
  const int quarter = (int)((r1 - r0 + 15) >> 4) << 2;      // rows of a wave, a multiple of four
  const int64_t w0 = r0 + wave * quarter, w1 = w0 + quarter < r1 ? w0 + quarter : r1;
  const int k = k0 + 4 * c16, f = f0 + 4 * c16;
  // (whole tiles of aligned rows 16 bytes a lane, others element by element; every load under no condition, its join would wait for it)
  const bool x_whole = k0 + kWgradTile <= j.w1 && (j.w1 & 3) == 0 && ((uintptr_t)j.x1 & 15) == 0;
  const bool z_whole = f0 + kWgradTile <= j.d_out && (j.d_out & 3) == 0;
  // what is there already, where the sums are added to it: requested with the rows
  const int col = t & 63, fo = f0 + col, rows = j.d_in - k0 < kWgradTile ? j.d_in - k0 : kWgradTile;
  const bool direct = !j.partial;
  float *dst = direct ? j.dW + (size_t)k0 * j.d_out + fo : j.partial + ((size_t)chunk * (j.d_in + 1) + k0) * j.d_out + fo;
  float *bias = direct ? j.db + fo : j.partial + ((size_t)chunk * (j.d_in + 1) + j.d_in) * j.d_out + fo;
  float old[kWgradTile / 4], old_bias = 0.f;
#pragma unroll
  for (int i = 0; i < kWgradTile / 4; ++i) {
    const int m = (t >> 6) + 4 * i;
    old[i] = 0.f;
    if (direct && fo < j.d_out && m < rows) old[i] = dst[(size_t)m * j.d_out];
  }
  if (direct && k0 == 0 && t < 64 && fo < j.d_out) old_bias = *bias;
  f32x4 acc[4][4], dzs = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  auto run = [&](auto xw, auto zw) {
    constexpr bool XW = decltype(xw)::value, ZW = decltype(zw)::value;
    for (int64_t r = w0; r < w1; r += 4 * kWgradFly) {
      f32x4 xv[kWgradFly], zv[kWgradFly];
#pragma unroll
      for (int i = 0; i < kWgradFly; ++i) {
        const int64_t ri = r + 4 * i + q4, rc = ri < w1 ? ri : w1 - 1;
        if constexpr (XW) {
          xv[i] = *(const f32x4 *)(j.x1 + rc * j.w1 + k);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int kc = k + e < j.d_in ? k + e : j.d_in - 1;
            xv[i][e] = *(kc < j.w1 ? j.x1 + rc * j.w1 + kc : j.x2 + rc * j.w2 + (kc - j.w1));
          }
        }
        if constexpr (ZW) {
          zv[i] = *(const f32x4 *)(j.dz + rc * j.d_out + f);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) zv[i][e] = j.dz[rc * j.d_out + (f + e < j.d_out ? f + e : j.d_out - 1)];
        }
      }
#pragma unroll
      for (int i = 0; i < kWgradFly; ++i) {
        const bool on = r + 4 * i + q4 < w1;                       // (columns past the last are not stored)
        xv[i] = on ? xv[i] : zero;
        zv[i] = on ? zv[i] : zero;
        dzs += zv[i];
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
          for (int n = 0; n < 4; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[i][m], zv[i][n], acc[m][n], 0, 0, 0);
      }
    }
  };
  typedef std::integral_constant<bool, true> yes;
  typedef std::integral_constant<bool, false> no;
  if (x_whole && z_whole) run(yes(), yes());
  else if (x_whole) run(yes(), no());
  else run(no(), no());
  // register i of tile (m, n): row 4 (4 q4 + i) + m, column 4 c16 + n
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *(f32x4 *)&sums[wave][16 * q4 + 4 * i + m][4 * c16] = f32x4{acc[m][0][i], acc[m][1][i], acc[m][2][i], acc[m][3][i]};
  if (k0 == 0) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      dzs[n] += __shfl_xor(dzs[n], 16);
      dzs[n] += __shfl_xor(dzs[n], 32);
    }
    if (q4 == 0) *(f32x4 *)&dz_sum[wave][4 * c16] = dzs;
  }
  __syncthreads();
  if (fo >= j.d_out) return;
#pragma unroll
  for (int i = 0; i < kWgradTile / 4; ++i) {
    const int m = (t >> 6) + 4 * i;
    if (m < rows) dst[(size_t)m * j.d_out] = old[i] + ((sums[0][m][col] + sums[1][m][col]) + (sums[2][m][col] + sums[3][m][col]));
  }
  if (k0 == 0 && t < 64) *bias = old_bias + ((dz_sum[0][col] + dz_sum[1][col]) + (dz_sum[2][col] + dz_sum[3][col]));
}
// dW / db += the chunks' sums, every entry in chunk order (eight loads in flight); layers of one chunk have no blocks
__global__ __launch_bounds__(256) void small_wgrad_reduce_kernel(const SmallWgradArgs a) {
  touch_args(a);
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
