// Row-MLPs on the fp32 matrix cores: sixteen rows of per-graph or per-state data per block through the readout MLP of the
// global-update layer (Section 3.4) or the policy and value heads (Section 3.3.2), and back; where a block has one row, by vector instructions (RowVector).
//
// What bounds them: every block reads all the weights from L2 (320 KB for a head at H = 256), and a row is too few products
// to hide that behind; so sixteen rows share a fragment (v_mfma_f32_16x16x4_f32, full fp32 operands and sums), the weights lie in
// fragment order (a fragment of 16 outputs by 16 contraction indices is one coalesced 1 KB load), and the eight waves of a
// block own different outputs, so that a layer costs one barrier. A wave requests half of the fragments of its next step -- across
// the barrier between two layers -- as soon as that half of this one's is used: at H = 256 a step's 32 instructions take longer than
// the L2's answer. Both halves of a layer's widths are padded to sixteen with zeros in the fragments; any width fits.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>
#include "mma.hip.h"
#include "segsum.hip.h"

constexpr int kRowTile = 16, kRowThreads = 512, kRowWaves = kRowThreads / 64, kRowFrags = 8;

// One affine map of a row-MLP: y = x M, M in fragment order ([output tile][contraction group][lane] of four floats:
// lane l has output 16 * tile + l % 16, contraction indices 16 * group + 4 * (l / 16) .. + 3).
struct RowMap {
  const f32x4 *w;
  int n_in, n_out;
};
// The widths of an MLP from its input on, where the kernel is made for them (kAnyWidth, kNarrow: known at run time only, at most 512 and 128).
// These launches are chains of a few round trips, and every width that has to be asked for first lengthens them.
constexpr int kAnyWidth = 0, kNarrow = -1;
template <int... W>
struct RowWidths {
  static constexpr int N = sizeof...(W) - 1;                       // maps
  static constexpr int w[N + 1] = {W...};
  // (any width: two waves per SIMD, whose registers hold twice the fragments in flight: at most 16 KB a wave, as a layer of 512 by 512 is 1 MB)
  static constexpr bool wide = N > 2 && ((W == kAnyWidth) || ...);
  static constexpr int waves = wide ? 2 : 4, frags = wide ? 2 * kRowFrags : kRowFrags;
  template <int M> static constexpr bool few = w[M + 1] == kNarrow || (w[M + 1] > 0 && w[M + 1] <= 16 * kRowWaves);   // at most a tile per wave
  template <int M> static __device__ __forceinline__ int in(const RowMap *map) { if constexpr (w[M] > 0) return w[M]; else return map[M].n_in; }
  template <int M> static __device__ __forceinline__ int out(const RowMap *map) { if constexpr (w[M + 1] > 0) return w[M + 1]; else return map[M].n_out; }
};
template <int M> using MapIndex = std::integral_constant<int, M>;

// floats of LDS between two rows of x: sixteen rows' 16-byte reads touch all banks
__host__ __device__ inline int row_pitch(int width) { return ((width + 15) >> 4) * 16 + 4; }

// x (LDS, sixteen rows `pitch` apart, padding columns zero) through the maps in turn; x2: room for as many. All 512 threads call it;
// stage() writes x, behind the first requests for weights (no barrier after it). Per output a lane holds four rows, 4 * (lane / 16) + i: their
// sums of map M's column f start from pre(M, f) and pass through post(M, f, sums), which leaves in them what goes to the next
// map's x (zeros in padding columns). Returns the x that holds the last results, after a barrier.
template <typename W>
struct RowMaps {
  static constexpr int FRAGS = W::frags, HALF = FRAGS / 2;
  const RowMap *map;
  int lane, wave, c16, q4, pitch;
  f32x4 frag[FRAGS];                             // of the wave's step; as soon as a half is used, that of the next step is requested in its place

  // A step is FRAGS fragments of one output tile (a unit) or, where there are more tiles than waves, of two; where there are
  // at most half as many tiles as waves, of one half of a tile's contraction (a unit too: the halves are added in LDS).
  template <int M> __device__ __forceinline__ int groups() const { return (W::template in<M>(map) + 15) >> 4; }
  template <int M> __device__ __forceinline__ int tiles() const { return (W::template out<M>(map) + 15) >> 4; }
  template <int M> __device__ __forceinline__ bool two() const { if constexpr (W::template few<M>) return false; else return tiles<M>() > kRowWaves; }
  template <int M> __device__ __forceinline__ int half() const {   // groups of the first half, or 0
    return tiles<M>() <= kRowWaves / 2 && groups<M>() > kRowFrags / 2 ? (groups<M>() + 1) >> 1 : 0;
  }
  template <int M> __device__ __forceinline__ int units() const { return two<M>() ? (tiles<M>() + 1) >> 1 : half<M>() ? 2 * tiles<M>() : tiles<M>(); }
  template <int M> __device__ __forceinline__ int steps() const {
    const int g = half<M>() ? half<M>() : groups<M>();
    return two<M>() ? (g + HALF - 1) / HALF : (g + FRAGS - 1) / FRAGS;
  }
  struct Step { const f32x4 *w0, *w1; int g0, last; bool two; };   // the tiles' fragments, its first group and the map's last
  template <int M> __device__ __forceinline__ Step step(int u, int s) const {
    const int G = groups<M>(), last = tiles<M>() - 1, t0 = two<M>() ? 2 * u : half<M>() ? u >> 1 : u, t1 = t0 < last ? t0 + 1 : last;
    return Step{map[M].w + (unsigned)(t0 * G) * 64u, map[M].w + (unsigned)(t1 * G) * 64u,
                s * (two<M>() ? HALF : FRAGS) + (u & 1 ? half<M>() : 0), G - 1, two<M>()};
  }
  // one half of a step's fragments (past the end the last one again: its products are left out)
  template <int PART> __device__ __forceinline__ void request(const Step &st) {
#pragma unroll
    for (int i = PART * HALF; i < PART * HALF + HALF; ++i) {
      int g = st.g0 + (st.two ? i >> 1 : i);
      g = g < st.last ? g : st.last;
      frag[i] = ((st.two && (i & 1) ? st.w1 : st.w0) + (unsigned)g * 64u)[lane];   // (the same for all lanes)
    }
  }
  template <int M> __device__ __forceinline__ void request_first() {
    if constexpr (M < W::N)
      if (wave < units<M>()) {
        const Step st = step<M>(wave, 0);
        request<0>(st);
        request<1>(st);
      }
  }
  template <int M, typename Pre, typename Post>
  __device__ __forceinline__ void run(float *x, float *x2, Pre &pre, Post &post) {
    const int T = tiles<M>(), n_units = units<M>(), n_steps = steps<M>(), n_out = W::template out<M>(map);
    const float *xr = x + c16 * pitch + 4 * q4;
    if (wave >= n_units) {
      request_first<M + 1>();
      if (half<M>()) __syncthreads();
    }
    for (int u = wave; u < n_units; u += kRowWaves) {
      const int t0 = two<M>() ? 2 * u : half<M>() ? u >> 1 : u, f0 = 16 * t0 + c16;
      const bool upper = half<M>() && (u & 1);
      const int gend = half<M>() && !upper ? half<M>() : groups<M>();
      // four sums per output, of every fourth contraction index: an instruction need not wait for the one before, and
      // rounding errors are those of chains a quarter as long
      f32x4 sum[2][4];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const float from = (two<M>() || k == 0) && !upper ? pre(MapIndex<M>(), f0 + 16 * k < n_out ? f0 + 16 * k : n_out - 1) : 0.f;
        sum[k][0] = f32x4{from, from, from, from};
#pragma unroll
        for (int j = 1; j < 4; ++j) sum[k][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      for (int s = 0; s < n_steps; ++s) {
        Step next;
        bool more = true;
        if (s + 1 < n_steps) next = step<M>(u, s + 1);
        else if (u + kRowWaves < n_units) next = step<M>(u + kRowWaves, 0);
        else if constexpr (M + 1 < W::N) {
          next = step<M + 1>(wave, 0);
          more = wave < units<M + 1>();
        } else more = false;
        const int g0 = s * (two<M>() ? HALF : FRAGS) + (upper ? half<M>() : 0);
        auto part = [&](auto which) {
          constexpr int PART = decltype(which)::value;
          const int gp = g0 + PART * (two<M>() ? HALF / 2 : HALF);
          f32x4 a[HALF];
          if (two<M>()) {
#pragma unroll
            for (int i = 0; i < HALF / 2; ++i) a[i] = *(const f32x4 *)(xr + 16 * (gp + i < gend ? gp + i : gend - 1));
#pragma unroll
            for (int i = 0; i < HALF / 2; ++i) {
              if (gp + i >= gend) break;
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                sum[0][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][j], frag[PART * HALF + 2 * i][j], sum[0][j], 0, 0, 0);
                sum[1][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][j], frag[PART * HALF + 2 * i + 1][j], sum[1][j], 0, 0, 0);
              }
            }
          } else {
#pragma unroll
            for (int i = 0; i < HALF; ++i) a[i] = *(const f32x4 *)(xr + 16 * (gp + i < gend ? gp + i : gend - 1));
#pragma unroll
            for (int i = 0; i < HALF; ++i) {
              if (gp + i >= gend) break;
#pragma unroll
              for (int j = 0; j < 4; ++j) sum[0][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][j], frag[PART * HALF + i][j], sum[0][j], 0, 0, 0);
            }
          }
          if (more) request<PART>(next);
        };
        part(MapIndex<0>());
        part(MapIndex<1>());
      }
      f32x4 acc[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) acc[k] = (sum[k][0] + sum[k][2]) + (sum[k][1] + sum[k][3]);
      if (half<M>()) {                               // (a wave has one unit at most: all pass this barrier once, see above)
        if (upper) {
#pragma unroll
          for (int i = 0; i < 4; ++i) x2[(4 * q4 + i) * pitch + f0] = acc[0][i];
        }
        __syncthreads();
        if (upper) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[0][i] += x2[(4 * q4 + i) * pitch + f0];
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if (k == 1 && (!two<M>() || t0 + 1 >= T)) break;
        const int f = f0 + 16 * k;
        if (f < n_out) post(MapIndex<M>(), f, acc[k]);
        else acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) x2[(4 * q4 + i) * pitch + f] = acc[k][i];
      }
    }
    __syncthreads();
    if constexpr (M + 1 < W::N) run<M + 1>(x2, x, pre, post);
  }
};
template <typename W, typename Stage, typename Pre, typename Post>
__device__ __forceinline__ float *row_maps(const RowMap *map, float *x, float *x2, int pitch, Stage stage, Pre pre, Post post) {
  RowMaps<W> m;
  m.map = map;
  m.lane = threadIdx.x & 63;
  m.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);       // (what steers the loops is the same for a wave's lanes)
  m.c16 = m.lane & 15;
  m.q4 = m.lane >> 4;
  m.pitch = pitch;
  m.template request_first<0>();
  stage();
  __syncthreads();
  m.template run<0>(x, x2, pre, post);
  return W::N % 2 ? x2 : x;
}

// ---- forward
struct RowFwdArgs {
  int relu_last;
  RowMap map[3];
  const float *b[3];
  const float *in1, *in2;  // in2 nullable
  int w1, w2;              // widths of in1 (a multiple of 4, rows 16-byte aligned) / in2; w1 + w2 == map[0].n_in
  int64_t n_rows;
  float *out;              // [n_rows, map[last].n_out]
  float *act[3];           // nullable each: every layer's output (after its ReLU)
  int pitch;               // of the widest layer
};
__host__ __device__ inline size_t row_lds_floats(int pitch) { return (size_t)(2 * kRowTile + 3) * pitch; }   // x, x2, the biases

// the layers' biases, `pitch` floats apart behind x and x2 (a sum that starts from one does not wait for memory); all widths are at
// most kRowThreads, and all loads in flight at once
template <typename W>
struct RowBiases {
  float v[W::N];
  template <int M = 0> __device__ __forceinline__ void request(const RowFwdArgs &a) {
    if constexpr (M < W::N) {
      const int n = W::template out<M>(a.map), t = threadIdx.x;
      v[M] = a.b[M][t < n ? t : n - 1];
      request<M + 1>(a);
    }
  }
  template <int M = 0> __device__ __forceinline__ void store(const RowFwdArgs &a, float *x, int pitch) const {
    if constexpr (M < W::N) {
      if ((int)threadIdx.x < W::template out<M>(a.map)) x[(2 * kRowTile + M) * pitch + threadIdx.x] = v[M];
      store<M + 1>(a, x, pitch);
    }
  }
};
// rows row0 .. row0 + 15 of [in1 | in2], zeros past the last row and column: two rows a wave, the first 256 columns of in1 and 64 of
// in2 in one round trip
struct RowInputs {
  f32x4 v[2];
  float g[2];
  __device__ __forceinline__ void request(const RowFwdArgs &a, int w1, int64_t row0) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int64_t row = row0 + 2 * (threadIdx.x >> 6) + i;
      row = row < a.n_rows ? row : a.n_rows - 1;
      v[i] = *(const f32x4 *)(a.in1 + row * w1 + (4 * lane < w1 ? 4 * lane : 0));
      g[i] = a.w2 ? a.in2[row * a.w2 + (lane < a.w2 ? lane : 0)] : 0.f;
    }
  }
  __device__ __forceinline__ void store(const RowFwdArgs &a, int w1, int width, int64_t row0, float *x, int pitch) const {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 2 * (threadIdx.x >> 6) + i;
      const bool on = row0 + r < a.n_rows;
      float *xr = x + r * pitch;
      if (4 * lane < w1) *(f32x4 *)(xr + 4 * lane) = on ? v[i] : f32x4{0.f, 0.f, 0.f, 0.f};
      if (w1 + lane < width) xr[w1 + lane] = on && lane < a.w2 ? g[i] : 0.f;
      for (int k = lane + 64; k < width - w1; k += 64) xr[w1 + k] = on && k < a.w2 ? a.in2[(row0 + r) * a.w2 + k] : 0.f;
    }
  }
};
// The layers of `a` on sixteen rows, row0 .. of which those below row_end are stored; stage() writes them and the biases to x. COHERENT_OUT
// stores a.out with device scope, for a consumer in another block of the same launch.
template <typename W, bool COHERENT_OUT, typename Stage>
__device__ __forceinline__ float *row_forward(const RowFwdArgs &a, int64_t row0, int64_t row_end, float *x, int pitch, Stage stage) {
  const int q4 = (threadIdx.x & 63) >> 4;
  const unsigned n_rows = row_end - row0 < kRowTile ? (unsigned)(row_end - row0) : kRowTile;
  const float *bias = x + 2 * kRowTile * pitch;
  const bool relu_last = a.relu_last;
  return row_maps<W>(a.map, x, x + kRowTile * pitch, pitch, stage,
    [&](auto m, int f) { return bias[decltype(m)::value * pitch + f]; },
    [&](auto m, int f, f32x4 &y) {
      constexpr int M = decltype(m)::value;
      constexpr bool last = M + 1 == W::N;
      const unsigned n_out = W::template out<M>(a.map);
      float *keep = a.act[M], *out = a.out + row0 * n_out;
      if (keep) keep += row0 * n_out;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (!last || relu_last) y[i] = fmaxf(y[i], 0.f);
        const unsigned r = 4 * q4 + i, at = r * n_out + f;
        if (keep && r < n_rows) keep[at] = y[i];
        if (last && r < n_rows) {
          if constexpr (COHERENT_OUT) __hip_atomic_store(out + at, y[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          else out[at] = y[i];
        }
      }
    });
}
template <typename W>
__global__ __launch_bounds__(kRowThreads, W::waves) void row_forward_kernel(const RowFwdArgs a) {
  extern __shared__ __align__(16) float sm[];
  touch_args(a);
  const int64_t row0 = (int64_t)blockIdx.x * kRowTile;
  const int pitch = a.pitch;
  (void)row_forward<W, false>(a, row0, a.n_rows, sm, pitch, [&]() {
    RowInputs in;
    RowBiases<W> b;
    in.request(a, a.w1, row0);
    b.request(a);
    in.store(a, a.w1, (W::template in<0>(a.map) + 15) & ~15, row0, sm, pitch);
    b.store(a, sm, pitch);
  });
}

// One row a block: the matrix instruction would spend its time on fifteen that are not there (H = 256: 3.6 us a layer of the readout, of one
// block on a compute unit). v_mfma_f32_16x16x4_f32 adds its four products to a sum one after
// the other, as four fmaf do (1M outputs each of ordinary, wide, subnormal and infinite operands: no bit differs); so a lane takes one of an
// output's four sums (RowMaps) through the same products in the same order, and a row's results are the same bits either way.
// Lane 4 * c + j of a wave has sum j of output 16 * tile + c: of a tile's fragments it reads every 64th float, the wave 256 bytes at a time, one
// stream per tile. x lies in LDS by quarters, contraction index k at (k % 4) * quarter + k / 4, so that a lane reads a group's four at once.
// floats a quarter of the widest row takes, its lanes' 16-byte reads in different banks; of two rows and the halves of a tile's contraction
constexpr int kRowQuarter = 512 / 4 + 8, kRowOneFloats = 2 * 4 * kRowQuarter + 16 * kRowWaves / 2;
template <typename W>
struct RowVector {
  static constexpr int most_tiles() {
    int n = 0;
    for (int k = 1; k <= W::N; ++k) {
      const int t = (W::w[k] > 0 ? W::w[k] + 15 : W::w[k] == kNarrow ? 16 * kRowWaves : 512) / 16;
      n = t > n ? t : n;
    }
    return n;
  }
  static constexpr int PER = (most_tiles() + kRowWaves - 1) / kRowWaves;       // tiles a wave, one in every kRowWaves
  static constexpr int RING = PER == 1 ? 12 : PER == 2 ? 6 : 4;                // groups in flight
  float w[RING][4][PER], from[PER];                   // fragments; what the sums start from
  const RowMap *map;
  int lane, wave;
  const float *p[PER];                                // of the map at hand: the tiles' streams
  int half, n, count;                                 // see RowMaps; this wave's groups (0: no tile) and tiles
  bool upper;
  template <int M> __device__ __forceinline__ int tiles() const { return (W::template out<M>(map) + 15) >> 4; }
  template <int M> __device__ __forceinline__ int tile(int i) const { return half ? wave >> 1 : wave + kRowWaves * i; }
  template <int M> __device__ __forceinline__ void begin(const float *bias) {
    const int G = (W::template in<M>(map) + 15) >> 4, T = tiles<M>(), n_out = W::template out<M>(map);
    half = T <= kRowWaves / 2 && G > kRowFrags / 2 ? (G + 1) >> 1 : 0;
    upper = half && (wave & 1);
    count = PER == 1 || half ? 1 : (T + kRowWaves - 1) / kRowWaves;
    const int g0 = upper ? half : 0;
    n = tile<M>(0) >= T ? 0 : half && !upper ? half : G - g0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int t = tile<M>(i) < T ? tile<M>(i) : T - 1, f = 16 * t + (lane >> 2);
      p[i] = (const float *)(map[M].w + (unsigned)(t * G + g0) * 64u) + lane;
      from[i] = (lane & 3) == 0 && !upper ? bias[f < n_out ? f : n_out - 1] : 0.f;
    }
  }
  // groups FROM .. TO - 1 of those in flight
  template <int FROM, int TO> __device__ __forceinline__ void request() {
#pragma unroll
    for (int r = FROM; r < TO; ++r)
      if (r < n) load(r, r);
  }
  __device__ __forceinline__ void load(int r, int g) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (i >= count) break;
#pragma unroll
      for (int q = 0; q < 4; ++q) w[r][q][i] = p[i][(unsigned)g * 256u + q * 64];
    }
  }
  // the map's results, passed through post(M, f, y) in the lane that has output f, to x2 (zeros in padding columns)
  template <int M, typename Post>
  __device__ __forceinline__ float *run(const RowFwdArgs &a, float *x, float *x2, float *extra, Post &post) {
    float s[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) s[i] = from[i];
    const float *xl = x + (lane & 3) * kRowQuarter + (upper ? 4 * half : 0);
    for (int g = 0; g < n; g += RING) {
#pragma unroll
      for (int r = 0; r < RING; ++r) {
        if (g + r >= n) break;
        const f32x4 v = *(const f32x4 *)(xl + 4 * (g + r));
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          if (i >= count) break;
#pragma unroll
          for (int q = 0; q < 4; ++q) s[i] = fmaf(v[q], w[r][q][i], s[i]);
        }
        if (g + r + RING < n) load(r, g + r + RING);
      }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      s[i] += __shfl_xor(s[i], 2);                    // (s0 + s2) + (s1 + s3)
      s[i] += __shfl_xor(s[i], 1);
    }
    const int T = tiles<M>(), n_out = W::template out<M>(map);
    const bool owns = n > 0 && !upper && (lane & 3) == 0;
    if (half) {
      const int f = 16 * tile<M>(0) + (lane >> 2);
      if (upper && n > 0 && (lane & 3) == 0) extra[f] = s[0];
      __syncthreads();
      if (owns) s[0] += extra[f];
    }
    if (owns) {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        if (i >= count || tile<M>(i) >= T) break;
        const int f = 16 * tile<M>(i) + (lane >> 2);
        if (f < n_out) post(MapIndex<M>(), f, s[i]);
        else s[i] = 0.f;
        x2[(f & 3) * kRowQuarter + (f >> 2)] = s[i];
      }
    }
    if constexpr (M + 1 < W::N) {
      begin<M + 1>(a.b[M + 1]);
      request<0, RING>();
    }
    __syncthreads();
    if constexpr (M + 1 < W::N) return run<M + 1>(a, x2, x, extra, post);
    else return x2;
  }
};
// The layers of `a` on one row, which stage() writes to x (kRowOneFloats of LDS; zeros in padding columns); as row_forward otherwise.
template <typename W, bool COHERENT_OUT, typename Stage>
__device__ __forceinline__ float *row_forward_one(const RowFwdArgs &a, int64_t row, float *x, Stage stage) {
  RowVector<W> m;
  constexpr int RING = RowVector<W>::RING;
  m.map = a.map;
  m.lane = threadIdx.x & 63;
  m.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool relu_last = a.relu_last;
  m.template begin<0>(a.b[0]);
  m.template request<0, RING / 2>();
  stage();
  m.template request<RING / 2, RING>();
  __syncthreads();
  auto post = [&](auto map, int f, float &y) {
    constexpr int M = decltype(map)::value;
    const int64_t at = row * W::template out<M>(a.map) + f;
    if (M + 1 < W::N || relu_last) y = fmaxf(y, 0.f);
    if (a.act[M]) a.act[M][at] = y;
    if constexpr (M + 1 == W::N) {
      if constexpr (COHERENT_OUT) __hip_atomic_store(a.out + at, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else a.out[at] = y;
    }
  };
  return m.template run<0>(a, x, x + 4 * kRowQuarter, x + 8 * kRowQuarter, post);
}

// ---- readout: the sum (or mean) of a graph's node states by a block, stored as pool[g, :] and left in row (LDS; nullable).
// (row: column k at (k % 4) * quarter + k / 4, see RowVector.) H / VEC lanes cover a node's row with 16-byte loads. The nodes are dealt over 512 / (H / VEC) groups, of which a thread of a block of
// THREADS threads holds V = 512 / THREADS (eight loads in flight in all), and the groups' sums are added in an order that does not
// depend on THREADS: a graph's sum is the same bits in every batch that comes here (of at most 4096 nodes a graph on average, see the readout's dispatch).
// MAPPED: row_of[n] is the row of h that holds node n's state (else row n); it is read a step ahead. part: THREADS * VEC floats of LDS.
template <typename T, int VEC, int H, bool MAPPED, int THREADS>
__device__ __forceinline__ void graph_pool(const T *h, const int32_t *graph_node_ptr, const int32_t *row_of, int g, int mean, float *pool,
                                           float *part, float *row, int quarter) {
  constexpr int tpr = H / VEC, Q = 256 / tpr, B = THREADS / tpr, NG = 2 * Q, V = 512 / THREADS, UF = 8 / V;
  const int t = threadIdx.x, c0 = (t % tpr) * VEC, q = t / tpr, n0 = graph_node_ptr[g], n1 = graph_node_ptr[g + 1];
  float acc[V][VEC];
#pragma unroll
  for (int v = 0; v < V; ++v)
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc[v][j] = 0.f;
  int at[V][UF];                                         // (past the end the graph's last row again, left out of the sum)
  auto places = [&](int n) {
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (int i = 0; i < UF; ++i) {
        const int k = n + v * B + i * NG;
        at[v][i] = k < n1 ? k : n1 - 1;
        if (MAPPED) at[v][i] = row_of[at[v][i]];
      }
  };
  if (n0 < n1) {
    places(n0 + q);
    for (int n = n0 + q; n - q < n1; n += UF * NG) {
      float x[V][UF][VEC];
#pragma unroll
      for (int v = 0; v < V; ++v)
#pragma unroll
        for (int i = 0; i < UF; ++i) RowVec<T, VEC>::load(h + (size_t)at[v][i] * H + c0, x[v][i]);
      places(n + UF * NG);
#pragma unroll
      for (int v = 0; v < V; ++v)
#pragma unroll
        for (int i = 0; i < UF; ++i)
#pragma unroll
          for (int j = 0; j < VEC; ++j) acc[v][j] += n + v * B + i * NG < n1 ? x[v][i][j] : 0.f;
    }
  }
  // the sum over q < Q of group q + group q + Q
  if constexpr (V == 2) {
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc[0][j] += acc[1][j];
  }
#pragma unroll
  for (int j = 0; j < VEC; j += 4) *(f32x4 *)(part + t * VEC + j) = f32x4{acc[0][j], acc[0][j + 1], acc[0][j + 2], acc[0][j + 3]};
  __syncthreads();
  if (t < H) {
    float a = 0.f;
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const float x = V == 2 ? part[k * H + t] : part[k * H + t] + part[(k + Q) * H + t];
      a = k ? a + x : x;
    }
    if (mean) a *= 1.f / (float)(n1 - n0 > 1 ? n1 - n0 : 1);
    pool[(size_t)g * H + t] = a;
    if (row) row[(t & 3) * quarter + (t >> 2)] = a;
  }
}
// Many graphs: a block sums one, the readout MLP follows in a launch of its own (row_forward_kernel), whose blocks
// share the weights among sixteen graphs. (1040 graphs of 338 nodes, by 512 threads a graph 13.8 us, by 256 11.4.)
constexpr int kPoolThreads = 256;
template <typename T, int VEC, int H, bool MAPPED>
__global__ __launch_bounds__(kPoolThreads) void graph_pool_kernel(const T *h, const int32_t *graph_node_ptr, const int32_t *row_of, int mean, float *pool) {
  __shared__ __align__(16) float part[kPoolThreads * VEC];
  graph_pool<T, VEC, H, MAPPED, kPoolThreads>(h, graph_node_ptr, row_of, blockIdx.x, mean, pool, part, nullptr, 0);
}
// Few graphs: both in one launch, a block per graph, the MLP's first weights requested ahead of the sum.
template <typename T, int VEC, int H, bool MAPPED>
__global__ __launch_bounds__(kRowThreads, 4) void graph_readout_kernel(const T *h, const int32_t *graph_node_ptr, const int32_t *row_of, int mean,
                                                                       float *pool, const RowFwdArgs a) {
  __shared__ __align__(16) float part[kRowThreads * VEC], x[kRowOneFloats];
  touch_args(a);
  const int g = blockIdx.x, n_in = H + a.w2;
  (void)row_forward_one<RowWidths<kAnyWidth, H, H>, false>(a, g, x, [&]() {
    for (int k = H + threadIdx.x; k < ((n_in + 15) & ~15); k += kRowThreads)
      x[(k & 3) * kRowQuarter + (k >> 2)] = k < n_in ? a.in2[(size_t)g * a.w2 + (k - H)] : 0.f;
    graph_pool<T, VEC, H, MAPPED, kRowThreads>(h, graph_node_ptr, row_of, g, mean, pool, part, x, kRowQuarter);
  });
}

// ---- reductions over a wave or the block, in a fixed order
struct BestSlot {
  float value;
  int index;             // lowest index that has it
};
__device__ __forceinline__ BestSlot better(const BestSlot &a, const BestSlot &b) {
  return b.value > a.value || (b.value == a.value && b.index < a.index) ? b : a;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ BestSlot wave_best(BestSlot b) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) b = better(b, BestSlot{__shfl_xor(b.value, o), __shfl_xor(b.index, o)});
  return b;
}
// the block's two sums; red: 2 * kRowWaves floats, which all have read when it returns
__device__ __forceinline__ float2 row_block_sum(float a, float b, float *red) {
  a = wave_sum(a);
  b = wave_sum(b);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[2 * w] = a; red[2 * w + 1] = b; }
  __syncthreads();
  float2 s = make_float2(red[0], red[1]);
#pragma unroll
  for (int k = 1; k < kRowWaves; ++k) { s.x += red[2 * k]; s.y += red[2 * k + 1]; }
  __syncthreads();
  return s;
}
__device__ __forceinline__ BestSlot row_block_best(BestSlot b, float *red) {
  b = wave_best(b);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[2 * w] = b.value; red[2 * w + 1] = __int_as_float(b.index); }
  __syncthreads();
  for (int k = 0; k < kRowWaves; ++k) b = better(b, BestSlot{red[2 * k], __float_as_int(red[2 * k + 1])});
  __syncthreads();
  return b;
}

// A state's masked log-softmax over its slots j0 .. j1 - 1: what its logits (ld: reads one) say of it, by a wave where
// the state has at most 64 slots (WIDE == 1) and by the block otherwise -- a state's results do not depend on what is beside it.
// A thread's first slot is read once and stays in registers.
template <int WIDE>
struct StateSoftmax {
  static constexpr int STEP = WIDE ? kRowThreads : 64;
  int j0, j1, first;       // this thread's slots: first, first + STEP, ..
  bool on;                 // of the first one
  float x;
  float lse, entropy, n_valid;
  int best;                // first slot that has the largest logit
  static __device__ __forceinline__ float2 sum(float a, float b, float *red) {
    if constexpr (WIDE) return row_block_sum(a, b, red);
    else return make_float2(wave_sum(a), wave_sum(b));
  }
  // go(j, its logit) for this thread's slots that are not masked
  template <typename Load, typename Go>
  __device__ __forceinline__ void each(Load ld, const uint8_t *mask, Go go) const {
    if (on) go(first, x);
    if constexpr (WIDE)
      for (int j = first + STEP; j < j1; j += STEP)
        if (mask[j]) go(j, ld(j));
  }
  template <typename Load>
  __device__ __forceinline__ StateSoftmax(Load ld, const uint8_t *mask, int begin, int end, float *red) {
    j0 = begin; j1 = end;
    first = j0 + (int)(threadIdx.x & (STEP - 1));
    x = first < j1 ? ld(first) : 0.f;                    // (beside the mask's load, not behind it)
    on = first < j1 && mask[first];
    BestSlot b{-INFINITY, 0x7fffffff};
    each(ld, mask, [&](int j, float v) { b = better(b, BestSlot{v, j}); });
    if constexpr (WIDE) b = row_block_best(b, red);
    else b = wave_best(b);
    best = b.index;
    float se = 0.f, cnt = 0.f;
    each(ld, mask, [&](int, float v) { se += expf(v - b.value); cnt += 1.f; });
    const float2 s = sum(se, cnt, red);
    lse = b.value + logf(s.x);
    n_valid = s.y;
    float ent = 0.f;
    each(ld, mask, [&](int, float v) { const float lp = v - lse; ent -= expf(lp) * lp; });
    entropy = sum(ent, 0.f, red).x;
  }
  // what the heads give
  template <typename Load>
  __device__ __forceinline__ void write(Load ld, const uint8_t *mask, float *logp, float *entropy_out, int32_t *action) const {
    if (first < j1) logp[first] = on ? x - lse : -INFINITY;
    if constexpr (WIDE)
      for (int j = first + STEP; j < j1; j += STEP) logp[j] = mask[j] ? ld(j) - lse : -INFINITY;
    if (first == j0) { *entropy_out = entropy; *action = best - j0; }
  }
};

// Both heads, forward, in one launch. The first blocks: the policy MLP of sixteen slots, of one or of several states;
// the block that finishes a state's last slot (a per-state counter, which it also resets; none where a block has all of
// them) does that state's masked log-softmax, entropy and first-max action. The last blocks: the mean
// embedding of the valid slots of value_rows states and the value head on it, independent of the policy blocks.
// Logits cross blocks through device-scope stores and loads (each completed before the block's
// counter increment is issued), so no cache write-back or invalidation is needed. logp null: the logits alone.
struct HeadsArgs {
  RowFwdArgs policy, value;          // of the same widths; value.in1 is not read
  const uint8_t *mask;
  const int32_t *state_graph_ptr;
  int G, S, value_rows;
  int32_t *counter;
  float *logp, *entropy;
  int32_t *action;
  float *zmean;
};
// ONE: a slot or state a block (value_rows 1), by vector instructions.
template <typename W, bool ONE>
__global__ __launch_bounds__(kRowThreads, W::waves) void heads_kernel(const HeadsArgs a) {
  constexpr int ROWS = ONE ? 1 : kRowTile;
  extern __shared__ __align__(16) float sm[];
  __shared__ float red[2 * kRowWaves];
  __shared__ int sh_state[ROWS], sh_done[ROWS], sh_n_done;
  __shared__ __align__(16) f32x4 part[kRowThreads];
  __shared__ int n_valid[kRowThreads];
  touch_args(a);
  constexpr int H = W::w[0];
  const int t = threadIdx.x, policy_blocks = (a.G + ROWS - 1) / ROWS, pitch = a.policy.pitch;
  const bool is_value = (int)blockIdx.x >= policy_blocks;
  const RowFwdArgs &mlp = is_value ? a.value : a.policy;            // (one copy of the layers' code for both)
  const int slot0 = blockIdx.x * ROWS;
  const int s0 = ((int)blockIdx.x - policy_blocks) * a.value_rows, s1 = s0 + a.value_rows < a.S ? s0 + a.value_rows : a.S;
  auto stage = [&]() {
    RowBiases<W> biases;
    if (!is_value) {
      // the block's slots; meanwhile find their states
      if constexpr (ONE) {
        if (t < H) sm[(t & 3) * kRowQuarter + (t >> 2)] = mlp.in1[(size_t)slot0 * H + t];
        if (a.logp && t < ROWS) sh_state[t] = -1;
        __syncthreads();
      } else {
        RowInputs in;
        in.request(mlp, H, slot0);
        biases.request(mlp);
        if (a.logp && t < ROWS) sh_state[t] = -1;
        __syncthreads();
        in.store(mlp, H, H, slot0, sm, pitch);
        biases.store(mlp, sm, pitch);
      }
      if (!a.logp) return;
      for (int s = t; s < a.S; s += kRowThreads) {
        const int p0 = a.state_graph_ptr[s], p1 = a.state_graph_ptr[s + 1];
        for (int r = p0 > slot0 ? p0 - slot0 : 0; r < ROWS && slot0 + r < p1; ++r) sh_state[r] = s;
      }
      return;
    }
    // the mean embedding of the valid slots: H / 4 threads cover a row with 16-byte loads, the 2048 / H thread groups
    // take every (2048 / H)-th slot, eight or (H = 256) twelve or sixteen loads in flight each; the groups' sums are added in order
    constexpr int U = H <= 128 ? 8 : W::w[1] == kNarrow ? 12 : 16;
    const float *emb = a.policy.in1;
    const int tpr = H / 4, ng = kRowThreads / tpr, c4 = (t % tpr) * 4, q = t / tpr; 
    if constexpr (!ONE) {
      for (int i = t; i < kRowTile * pitch; i += kRowThreads) sm[i] = 0.f;
      biases.request(mlp);
    }
    for (int s = s0; s < s1; ++s) {
      const int j0 = a.state_graph_ptr[s], j1 = a.state_graph_ptr[s + 1];
      f32x4 p = f32x4{0.f, 0.f, 0.f, 0.f};
      int cnt = 0;
      for (int j = j0 + q; j < j1; j += U * ng) {
        f32x4 v[U];
        bool on[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const int ji = j + i * ng < j1 ? j + i * ng : j;
          v[i] = *(const f32x4 *)(emb + (size_t)ji * H + c4);
          on[i] = j + i * ng < j1 && a.mask[ji];
        }
#pragma unroll
        for (int i = 0; i < U; ++i)
          if (on[i]) { p += v[i]; ++cnt; }
      }
      part[t] = p;
      n_valid[t] = cnt;
      __syncthreads();
      if (t < tpr) {
        f32x4 acc = part[t];
        int n = n_valid[0];
        for (int k = 1; k < ng; ++k) { acc += part[k * tpr + t]; n += n_valid[k * tpr]; }
        const float nv = (float)n;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] /= nv;
        *(f32x4 *)(a.zmean + (size_t)s * H + c4) = acc;
        if constexpr (ONE) {
#pragma unroll
          for (int i = 0; i < 4; ++i) sm[i * kRowQuarter + (c4 >> 2)] = acc[i];
        } else *(f32x4 *)(sm + (s - s0) * pitch + c4) = acc;
      }
      __syncthreads();
    }
    if constexpr (!ONE) biases.store(mlp, sm, pitch);
  };
  const float *y;
  if constexpr (ONE) y = row_forward_one<W, true>(mlp, is_value ? s0 : slot0, sm, stage);
  else y = row_forward<W, true>(mlp, is_value ? s0 : slot0, is_value ? s1 : a.G, sm, pitch, stage);
  if (is_value) return;
  if (!a.logp) return;
  __builtin_amdgcn_s_waitcnt(0x0F70);                              // vmcnt(0): this wave's logit stores have completed
  __syncthreads();
  if (t < ROWS) {
    // one thread per slot; that of a state's first slot here speaks for the state (the sixteen lanes are one wave's)
    const int s = sh_state[t];
    bool done = false;
    if (s >= 0 && (t == 0 || sh_state[t - 1] != s)) {
      int k = 1;
      while (t + k < ROWS && sh_state[t + k] == s) ++k;
      const int slots = a.state_graph_ptr[s + 1] - a.state_graph_ptr[s];
      done = k == slots;
      if (!done && atomicAdd(&a.counter[s], k) + k == slots) {
        a.counter[s] = 0;                                          // ready for the next launch
        done = true;
      }
    }
    const unsigned long long who = __ballot(done);
    if (done) sh_done[__popcll(who & ((1ull << t) - 1))] = s;
    if (t == 0) sh_n_done = __popcll(who);
  }
  __syncthreads();
  const float *logit = a.policy.out;
  auto with_logits = [&](int j0, int j1, auto go) {                // its own logits are still in LDS
    if (j0 >= slot0 && j1 <= slot0 + ROWS) go([&](int j) { return y[(j - slot0) * pitch]; });
    else go([&](int j) { return __hip_atomic_load(logit + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); });
  };
  const int n_done = sh_n_done;
  for (int i = 0; i < n_done; ++i) {
    const int s = sh_done[i], j0 = a.state_graph_ptr[s], j1 = a.state_graph_ptr[s + 1];
    if (j1 - j0 > 64) {
      with_logits(j0, j1, [&](auto ld) { StateSoftmax<1>(ld, a.mask, j0, j1, red).write(ld, a.mask, a.logp, a.entropy + s, a.action + s); });
    } else if (i % kRowWaves == t >> 6) {
      with_logits(j0, j1, [&](auto ld) { StateSoftmax<0>(ld, a.mask, j0, j1, red).write(ld, a.mask, a.logp, a.entropy + s, a.action + s); });
    }
  }
}

// The same per state where a batch has more states than counters: one block per state, logits from memory.
__global__ __launch_bounds__(kRowThreads) void state_policy_kernel(const float *logit, const uint8_t *mask, const int32_t *state_graph_ptr,
                                                                   float *logp, float *entropy, int32_t *action) {
  __shared__ float red[2 * kRowWaves];
  const int s = blockIdx.x, j0 = state_graph_ptr[s], j1 = state_graph_ptr[s + 1];
  auto ld = [&](int j) { return logit[j]; };
  if (j1 - j0 > 64) StateSoftmax<1>(ld, mask, j0, j1, red).write(ld, mask, logp, entropy + s, action + s);
  else if (threadIdx.x < 64 && j1 > j0) StateSoftmax<0>(ld, mask, j0, j1, red).write(ld, mask, logp, entropy + s, action + s);
}

// ---- backward: given dout [n_rows, width of the last layer] and every layer's saved output, the gradients dz[l] before
// the layers' ReLUs (stored, for the weight gradients) and dx [n_rows, d_in].
struct RowBwdArgs {
  int relu_last;
  RowMap map[3];           // map[0] is the last layer's: contraction over its outputs
  const float *act[3];     // saved outputs of each layer
  const float *dout;
  int64_t n_rows;
  float *dz[3];            // [n_rows, width of layer l]
  float *dx;               // [n_rows, d_in]
  int n_layers, pitch;
};
// LDS of a backward block: x, x2 and, of every layer but the last, the outputs whose ReLU the gradient passes
inline size_t row_bwd_lds_floats(const RowBwdArgs &a) {
  size_t n = 2 * a.pitch;
  for (int m = 0; m + 1 < a.n_layers; ++m) n += row_pitch(a.map[m].n_out);
  return kRowTile * n;
}

// Two rows a wave of a [*, w] array, row_of(r) for the block's row r < n (the last again past them): the first 256 columns
// requested together, before any is waited for (16 bytes a lane where every row is aligned to that -- a caller's array need not be -- else
// four loads)
struct RowPiece {
  f32x4 v[2];
  template <typename RowOf>
  __device__ __forceinline__ void request(const float *src, int w, int n, RowOf row_of, bool aligned = true) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 2 * (threadIdx.x >> 6) + i;
      const float *q = src + (int64_t)row_of(r < n ? r : n - 1) * w;
      if ((w & 3) == 0 && aligned) {
        v[i] = *(const f32x4 *)(q + (4 * lane < w ? 4 * lane : 0));
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[i][k] = q[4 * lane + k < w ? 4 * lane + k : w - 1];
      }
    }
  }
  // put(r, f, value) for the sixteen rows' w columns
  template <typename RowOf, typename Put>
  __device__ __forceinline__ void store(const float *src, int w, int n, RowOf row_of, Put put) const {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 2 * (threadIdx.x >> 6) + i;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (4 * lane + k < w) put(r, 4 * lane + k, v[i][k]);
      for (int f = 256 + lane; f < w; f += 64) put(r, f, src[(int64_t)row_of(r < n ? r : n - 1) * w + f]);
    }
  }
};
// The sixteen rows from row0, of which those below row_end exist (at least one).
template <typename W>
__device__ __forceinline__ void row_backward(const RowBwdArgs &a, int64_t row0, int64_t row_end, float *x, int pitch) {
  constexpr int L = W::N;
  static_assert(L == 2 || L == 3, "row-MLPs of two or three layers");
  const int lane = threadIdx.x & 63, q4 = lane >> 4;
  const int n = (int)(row_end - row0 < kRowTile ? row_end - row0 : kRowTile);
  // what post takes, of each map
  const int pitch0 = row_pitch(W::template out<0>(a.map)), pitch1 = row_pitch(W::template out<1>(a.map));
  float *const below0 = x + 2 * kRowTile * pitch, *const below1 = below0 + kRowTile * pitch0;
  (void)row_maps<W>(a.map, x, x + kRowTile * pitch, pitch,
    [&]() {
      auto own = [&](int r) { return row0 + r; };
      const int w = W::template in<0>(a.map), w0 = W::template out<0>(a.map), w1 = W::template out<1>(a.map);
      RowPiece p0, p1, pr, pd;
      p0.request(a.act[L - 2], w0, n, own);
      if (L > 2) p1.request(a.act[0], w1, n, own);
      if (a.relu_last) pr.request(a.act[L - 1], w, n, own);
      pd.request(a.dout, w, n, own, ((uintptr_t)a.dout & 15) == 0);
      p0.store(a.act[L - 2], w0, n, own, [&](int r, int f, float v) { below0[r * pitch0 + f] = v; });
      if (L > 2) p1.store(a.act[0], w1, n, own, [&](int r, int f, float v) { below1[r * pitch1 + f] = v; });
      if (a.relu_last) pr.store(a.act[L - 1], w, n, own, [&](int r, int f, float v) { x[r * pitch + f] = v; });
      float *dz = a.dz[L - 1] + row0 * w;
      pd.store(a.dout, w, n, own, [&](int r, int f, float v) {
        if (r >= n || (a.relu_last && !(x[r * pitch + f] > 0.f))) v = 0.f;
        x[r * pitch + f] = v;
        if (r < n) dz[r * w + f] = v;
      });
      const int wide = (w + 15) & ~15;
      for (int f = w + lane; f < wide; f += 64) {
        x[2 * (threadIdx.x >> 6) * pitch + f] = 0.f;
        x[(2 * (threadIdx.x >> 6) + 1) * pitch + f] = 0.f;
      }
    },
    [&](auto, int) { return 0.f; },
    [&](auto m, int f, f32x4 &y) {
      constexpr int M = decltype(m)::value;
      const unsigned w = W::template out<M>(a.map);
      float *to;
      if constexpr (M + 1 < L) to = a.dz[L - 2 - M] + row0 * w;
      else to = a.dx + row0 * w;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * q4 + i;
        if (M + 1 < L && !((M ? below1[r * pitch1 + f] : below0[r * pitch0 + f]) > 0.f)) y[i] = 0.f;
        if (r < n) to[r * w + f] = y[i];
        else y[i] = 0.f;
      }
    });
}
template <typename W>
__global__ __launch_bounds__(kRowThreads, W::waves) void row_backward_kernel(const RowBwdArgs a) {
  extern __shared__ __align__(16) float sm[];
  touch_args(a);
  row_backward<W>(a, (int64_t)blockIdx.x * kRowTile, a.n_rows, sm, a.pitch);
}

// Backward of the masked log-softmax, states_per_block states per block: from the logits and the outputs' gradients
//   dlogit_k = c_k - p_k * sum_valid c  -  dent * p_k * (logp_k + entropy),  c = dlogp      (0 when masked)
// and one over the number of the state's valid slots.
struct HeadsSoftmaxBwdArgs {
  const float *logit;
  const uint8_t *mask;
  const int32_t *state_graph_ptr;
  const float *dlogp, *dentropy;
  float *dlogit, *inv_valid;
  int S, states_per_block;
};
__global__ __launch_bounds__(kRowThreads) void heads_softmax_bwd_kernel(const HeadsSoftmaxBwdArgs a) {
  __shared__ float red[2 * kRowWaves];
  touch_args(a);
  const int t = threadIdx.x, s0 = blockIdx.x * a.states_per_block, s1 = s0 + a.states_per_block < a.S ? s0 + a.states_per_block : a.S;
  auto ld = [&](int j) { return a.logit[j]; };
  for (int s = s0; s < s1; ++s) {
    const int j0 = a.state_graph_ptr[s], j1 = a.state_graph_ptr[s + 1];
    auto slots = [&](auto wide) {
      using Softmax = StateSoftmax<decltype(wide)::value>;
      const int at = j0 + (int)(t & (Softmax::STEP - 1));
      const float first = at < j1 ? a.dlogp[at] : 0.f, de = a.dentropy[s];
      const Softmax m(ld, a.mask, j0, j1, red);
      auto c = [&](int j) { return j == m.first ? first : a.dlogp[j]; };
      float cs = 0.f;
      m.each(ld, a.mask, [&](int j, float) { cs += c(j); });
      cs = Softmax::sum(cs, 0.f, red).x;
      for (int j = m.first; j < j1; j += Softmax::STEP)
        if (j == m.first ? !m.on : !a.mask[j]) a.dlogit[j] = 0.f;
      m.each(ld, a.mask, [&](int j, float x) {
        const float lp = x - m.lse, p = expf(lp);
        a.dlogit[j] = c(j) - p * cs - de * p * (lp + m.entropy);
      });
      if (m.first == j0) a.inv_valid[s] = 1.f / m.n_valid;
    };
    if (j1 - j0 > 64) slots(MapIndex<1>());
    else if ((s - s0) % kRowWaves == t >> 6) slots(MapIndex<0>());    // (the same choice for all threads of a wave)
  }
}

// Both heads' MLPs back, in one launch: the value head's rows (value_rows states a block; its dx is the gradient of the mean
// embedding) in the first blocks, the policy head's in the others. A slot's dx still lacks its state's share of the mean embedding's
// gradient: the last blocks of small_wgrad_kernel's launch add it. Where few slots leave the chip empty, a launch is as long as one tile's way through
// the layers, so the two heads beside each other are what counts: us of a call with the value head in front of the policy head, in the softmax's
// launch / so, 15 slots, heads of 128 and 64, H = 64 36.8 / 28.4, H = 256 43.8 / 33.2, of 512 and 512 127 / 88 and 153 / 108; at 4624 slots of
// H = 256 and heads of 256 and 64 the launches 13.1 + 22.4 / 4.7 + 19.0.
struct HeadsBwdArgs {
  RowBwdArgs value, policy;          // of the same widths
  int value_rows, value_blocks;
};
template <typename W>
__global__ __launch_bounds__(kRowThreads, W::waves) void heads_backward_kernel(const HeadsBwdArgs a) {
  extern __shared__ __align__(16) float sm[];
  touch_args(a);
  const bool is_value = (int)blockIdx.x < a.value_blocks;
  const RowBwdArgs &mlp = is_value ? a.value : a.policy;            // (one copy of the layers' code for both)
  const int rows = is_value ? a.value_rows : kRowTile;
  const int64_t row0 = (int64_t)(is_value ? (int)blockIdx.x : (int)blockIdx.x - a.value_blocks) * rows;
  row_backward<W>(mlp, row0, row0 + rows < mlp.n_rows ? row0 + rows : mlp.n_rows, sm, a.policy.pitch);
}
