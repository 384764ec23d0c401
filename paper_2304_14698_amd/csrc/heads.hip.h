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
  touch_args(a);
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
