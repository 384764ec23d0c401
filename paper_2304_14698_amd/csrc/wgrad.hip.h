// Weight gradients of affine layers, dW = X^T dZ and db = 1^T dZ, over very tall X (rows = edges or
// nodes), deterministic. One launch takes the products of many layers (every MLP of a backward pass): the
// rows of each are cut into slices, a block accumulates TA columns of X times all H columns of dZ
// over one slice on the matrix cores in fp32 and writes its partial tile, and a second launch adds each
// entry's partials in slice order onto the caller's gradient vector.
//
// Bound by memory: H = 128, 468 k edges and 216 k nodes over five rounds, 876 MB of operands in 187 us (4.7 TB/s)
// and 19 us for the reduction; H = 256, 2.0 M edges and 1.45 M nodes, 8.8 GB in 2.23 ms (3.9 TB/s) and 90 us. With a
// launch and a reduction per product these were 531 us (40 launches) and 3.40 ms: every product
// had to fill the chip by itself, and so wrote and read again a partial tile per block (34 MB at H = 128, 67
// MB at H = 256) however few rows it had, and the edge attributes' nine columns passed over dZ once more.
//
// The contraction runs over rows, so an operand is "lane = column, elements = rows" while memory, and LDS with
// it, is row-major. bf16: an operand is two LDS transpose reads (ds_read_b64_tr_b16): in a group of 16
// lanes, lane L passes the address of 4 consecutive 16-bit elements -- lanes 4j .. 4j+3 together one
// 16-element piece of row j -- and receives element L of each of the four rows; so lane L points at
// tile[k0 + L / 4][c0 + 4 * (L % 4)] and gets tile[k0 .. k0+3][c0 + L]. fp32: four 4-byte reads, 32
// consecutive columns each, of rows 4 g .. 4 g + 3 of an eight-row step.
#pragma once
#include <algorithm>
#include <type_traits>
#include "mlp2r.hip.h"

// X: PLAIN = A [rows, Ka], EDGE = [h[sender] | h[receiver] (| attributes)], NODE = [h | received sum], ATTR =
// the edge attributes alone (when they are too wide for the EDGE product's extra columns)
enum { WG_PLAIN = 0, WG_EDGE = 1, WG_NODE = 2, WG_ATTR = 3 };
constexpr int kWgradExtra = 32;   // columns of X a block can take beside its TA: an EDGE product's attributes, the bias

struct WgradJob {
  const void *A;                       // PLAIN: [rows, Ka]; EDGE, NODE: [N, H]; operand type
  const void *agg;                     // NODE: [N, H] received sums
  const int32_t *src, *dst;            // EDGE: sender and receiver of each row; NODE: dst = row of agg per node, -1 = zeros
  const float *edge_feat;              // EDGE, ATTR: [rows, De]
  const void *dZ;                      // [rows, H] operand type
  int64_t n_rows;
  int kind, Ka, De;
  // plan (see plan_wgrads)
  int rows_per_slice, ny, kt;          // rows per slice, slices, column tiles
  int rot;                             // slice y runs on XCD (y + rot) % 8, see wgrad_place
  int extra;                           // tile 0 also takes the extra columns, rows kt TA .. of the partial
  int KaP;                             // rows of a slice's partial
  int k_rows, bias_row;                // partial rows [0, k_rows) go to dW, row bias_row to db (-1: no bias)
  float *partial;                      // [ny][KaP][H]
  float *dW, *db;
};
constexpr int kWgradMaxJobs = 24;      // (the argument block stays under 4 KB)
struct WgradLaunch {
  const void *zero_row;                // 1 KB of zeros, then 16 bytes that hold 1, 0, .. in the operand type
  int32_t tiles[kWgradMaxJobs];        // of each job: ny << 16 | rot << 8 | kt, 0 beyond the last
  int32_t entry0[kWgradMaxJobs];       // the reduction's first block of each job, INT_MAX beyond the last
  WgradJob job[kWgradMaxJobs];
};
// The job, slice and column tile of a block. Blocks are dealt round-robin to the 8 XCDs; XCD x takes, job after job,
// its share of the slices with all their column tiles, so that dZ enters its L2 once. Only the grid's
// last blocks may have nothing to do (job = kWgradMaxJobs): idle blocks in between, dealt to the compute units
// like any other, left some of them with two blocks one after the other and doubled the launch.
struct WgradPlace { int job, y, kq; };
__device__ __forceinline__ WgradPlace wgrad_place(const WgradLaunch &a, int block) {
  const int xcd = block & 7, i = block >> 3;
  WgradPlace p{0, 0, 0};
  int end = 0, first = 0;
#pragma unroll
  for (int k = 0; k < kWgradMaxJobs; ++k) {
    const int c = a.tiles[k], ny = c >> 16;
    end += (c & 255) * (ny / 8 + (((xcd - (c >> 8)) & 7) < (ny & 7) ? 1 : 0));
    if (i >= end) { p.job = k + 1; first = end; }
  }
  if (p.job < kWgradMaxJobs) {
    const int c = a.tiles[p.job], kt = c & 255;
    p.kq = (i - first) % kt;
    p.y = ((xcd - (c >> 8)) & 7) + 8 * ((i - first) / kt);
  }
  return p;
}

typedef short s16x4 __attribute__((ext_vector_type(4)));

// TA = X columns per block, 128 (four waves, two blocks per CU) or 256 (eight waves, one block per CU: dZ is
// read once per 256 instead of once per 128 columns). RS = rows per stage: what a block has in
// flight from memory while it multiplies the previous stage; one block per CU needs 64 in bf16.
// A slice may have tens of thousands of rows, and the error of a sum taken step after step grows with the root of the
// steps (of 2 rows in fp32, of 16 in bf16). So every FOLD rows the sums are added to second ones: in registers where there are
// as many again, in fp32 at H = 256 in the partial tile. Relative error of 2^20 rows' products of random sign
// against float64, one chain / folded: fp32 5.9e-7 / 2.3e-7 (H = 256 8.5e-7 / 2.4e-7), bf16, 2^22 rows, 5.0e-7 / 2.2e-7; of the
// encoder's fp32 gradients, 5 k to 110 k nodes, 1.0 to 3 times less. It costs nothing that can be measured at H <= 128 and
// 12 % of the launch in fp32 at H = 256 (93 k nodes 4.5 / 5.0 ms). bf16 at H = 256 keeps one chain (5.0e-7 at 2^21 rows; the
// gradients of 110 k nodes are 3.1e-2 from float64 for the operands' rounding, to three digits whatever the chain): 160 of 256
// registers hold sums, and the tile's way to memory and back every 2048 rows cost a quarter of the launch.
// A stage goes from memory into LDS directly (lds_direct_load16), as the rows lie there: 16-byte piece s of LDS
// row r holds piece s ^ swizzle(r), which moves the rows r .. r + 3 that a transpose read touches to
// different banks where their lengths, multiples of 256 bytes, would put them on the same.
template <typename T, int H, int TA, int RS>
struct WgradShape {
  static constexpr int NT = 2 * TA, V = Operand<T>::V, ST = 2 * V;   // threads, elements per 16 bytes, rows per step
  static constexpr int WA = TA / 64;                                 // waves along X; two along dZ
  static constexpr int NB = H / 64;                                  // 32-column blocks of dZ per wave
  static constexpr int NE = NB / WA > 0 ? NB / WA : 1;               // ... whose products with the extra columns it takes
  static constexpr int XP = TA / V, ZP = H / V, EP = kWgradExtra / V;    // pieces per row of X, dZ and the extra columns
  static constexpr int XB = RS * XP * 16, ZB = RS * ZP * 16, EB = RS * EP * 16;   // bytes of a stage
  static constexpr int XV = RS * XP / NT, ZV = RS * ZP / NT;         // pieces per thread and stage
  static constexpr size_t LDS = 2 * (size_t)(XB + ZB + EB);
  static constexpr bool SECOND = H <= 128;                           // second sums in registers ...
  static constexpr int FOLD = SECOND ? (sizeof(T) == 4 ? 128 : 1024) : sizeof(T) == 4 ? 192 : 0;   // ... or in the partial tile (0: none)
  static_assert(ZV >= 1 && XV >= 1 && RS % ST == 0 && RS * EP == NT / 2 && (NT / XP) % 4 == 0 && (NT / ZP) % 4 == 0 && FOLD % RS == 0, "");
};
// swizzle(r) in 64-byte blocks, for rows of P pieces
template <typename T, int P>
__device__ __forceinline__ int wgrad_swizzle(int row) {
  if constexpr (sizeof(T) == 4 || P <= 4) return 0;        // (fp32 operands are whole 128-byte lines of one row)
  else return P >= 16 ? row & 3 : (row >> 1) & 1;
}
// This lane's address, inside a stage of rows of P pieces, of 32-column block b for a step's first rows
template <typename T, int P>
__device__ __forceinline__ int wgrad_lane_offset(int lane, int b) {
  if constexpr (sizeof(T) == 2) {
    const int L = lane & 15, row = 8 * (lane >> 5) + L / 4;
    return row * P * 16 + (b ^ wgrad_swizzle<T, P>(row)) * 64 + 32 * ((lane >> 4) & 1) + 8 * (L % 4);
  } else {
    return 4 * (lane >> 5) * P * 16 + b * 128 + (lane & 31) * 4;
  }
}
// Rows of one column as an MFMA operand; p = this lane's address (above) in the step
template <typename T, int P>
__device__ __forceinline__ typename Operand<T>::vec lds_column_operand(const char *p) {
  if constexpr (sizeof(T) == 2) {
    typedef s16x4 __attribute__((address_space(3))) * lp;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + 4 * P * 16));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  } else {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = *(const float *)(p + e * P * 16);
    return v;
  }
}

// The stage loop of one block. Rows past the slice and columns past Ka come from the row of zeros, the all-ones
// column from the piece behind it: a select on the address, so that no load is under a condition. The row
// indices of gathered X columns are fetched two stages ahead. EXTRA: also 32 columns beside the tile, an
// EDGE product's [attributes | 1 | 0 ..], else the all-ones column alone.
template <typename T, int H, int TA, int RS>
struct WgradSums {
  using S = WgradShape<T, H, TA, RS>;
  f32x16 main[2][S::NB], extra[S::NE];   // of 32-column blocks of X (the extra columns) and of dZ
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < S::NB; ++i) main[m][i][r] = 0.f;
#pragma unroll
      for (int i = 0; i < S::NE; ++i) extra[i][r] = 0.f;
    }
  }
  __device__ __forceinline__ void add(const WgradSums &o, bool with_extra) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < S::NB; ++i) main[m][i] += o.main[m][i];
    if (with_extra)
#pragma unroll
      for (int i = 0; i < S::NE; ++i) extra[i] += o.extra[i];
  }
};
// A 32-column block's sums to the partial tile (rows H apart; out: this lane's column), or added to what is there
template <int H>
__device__ __forceinline__ void wgrad_put(float *out, int g, bool add, f32x16 &s) {
  unsigned at = (unsigned)(4 * g * H);
  asm volatile("" : "+v"(at));           // (formed here: kept over the stage loop, the addresses of all blocks spill)
  if (add) {
    float t[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) t[r] = out[at + (unsigned)(acc_row(r, 0) * H)];
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] += t[r];
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) out[at + (unsigned)(acc_row(r, 0) * H)] = s[r];
}
template <typename T, int H, int TA, int RS, int KIND, bool EXTRA, typename Fold>
__device__ __forceinline__ void wgrad_run(const WgradJob &j, const char *zero_row, int ka0, int64_t r_begin, int64_t r_end, char *smem,
                                          WgradSums<T, H, TA, RS> &sums, Fold fold) {
  using S = WgradShape<T, H, TA, RS>;
  using Opd = Operand<T>;
  using vec = typename Opd::vec;
  constexpr int V = S::V, ST = S::ST, XV = S::XV, ZV = S::ZV, NB = S::NB, NE = S::NE, NT = S::NT, XP = S::XP, ZP = S::ZP, EP = S::EP;
  auto &acc = sums.main;
  auto &acce = sums.extra;
  constexpr bool GATHER = KIND == WG_EDGE || KIND == WG_NODE, ATTRS = EXTRA && KIND == WG_EDGE;
  char *const Xs = smem, *const Zs = smem + 2 * S::XB, *const Es = Zs + 2 * S::ZB;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wa = wave % S::WA, wb = wave / S::WA;
  const int n_stage = (int)((r_end - r_begin + RS - 1) / RS);

  // ---- this thread's pieces of a stage: X rows xr, xr + NT / XP, .., columns xc .. xc + V - 1; the same of dZ
  // (the swizzle is the same for all of them)
  const int xr = tid / XP, zr = tid / ZP;
  const int xc = ka0 + V * ((tid % XP) ^ (4 * wgrad_swizzle<T, XP>(xr)));
  const int zc = V * ((tid % ZP) ^ (4 * wgrad_swizzle<T, ZP>(zr)));
  const bool second = xc >= H;                             // EDGE: receiver's state; NODE: received sum
  [[maybe_unused]] const int32_t *idx_arr = KIND == WG_NODE || second ? j.dst : j.src;
  [[maybe_unused]] const T *gbase = (second && KIND == WG_NODE ? (const T *)j.agg : (const T *)j.A) + (GATHER && second ? xc - H : xc);
  // PLAIN: what columns past Ka read
  [[maybe_unused]] const char *past = zero_row + (xc == j.Ka ? 1024 : 0);
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem) + wave * 1024);

  auto row_at = [&](int st, int r) {
    const int64_t row = r_begin + (int64_t)st * RS + r;
    return row < r_end ? row : r_end - 1;
  };
  auto live = [&](int st, int r) { return r_begin + (int64_t)st * RS + r < r_end; };
  auto load_idx = [&](int st, int (&ix)[XV]) {
#pragma unroll
    for (int c = 0; c < XV; ++c) ix[c] = GATHER ? idx_arr[row_at(st, xr + NT / XP * c)] : 0;
  };
  // V columns k .. of [attributes | 1 | 0 ..] of a row, as requested and as used
  struct Attr { f32x4 q[V / 4]; };
  auto load_attr = [&](int64_t row, int k) {
    Attr r;
#pragma unroll
    for (int i = 0; i < V / 4; ++i)
      r.q[i] = *(const f32x4 *)(k + 4 * i + 4 <= j.De ? j.edge_feat + (size_t)row * j.De + k + 4 * i : (const float *)zero_row);
    return r;
  };
  auto attr_operand = [&](const Attr &r, int k, bool on) {
    vec x;
#pragma unroll
    for (int i = 0; i < V; ++i)                            // (De is a multiple of 4)
      x[i] = Opd::from_float(i % 4 == 0 && k + i == j.De ? 1.f : r.q[i / 4][i % 4]);
    return on ? x : Opd::zero();
  };
  auto fetch = [&](int st, const int (&ix)[XV]) {
    const int buf = st & 1;
    if constexpr (KIND != WG_ATTR) {
#pragma unroll
      for (int c = 0; c < XV; ++c) {
        const int r = xr + NT / XP * c;
        const int64_t row = row_at(st, r);
        const int64_t srow = KIND == WG_EDGE || (KIND == WG_NODE && second) ? (int64_t)ix[c] : row;
        const char *p = KIND == WG_PLAIN ? (xc + V <= j.Ka ? (const char *)((const T *)j.A + (size_t)row * j.Ka + xc) : past)
                                         : (KIND == WG_NODE && srow < 0 ? zero_row : (const char *)(gbase + (size_t)srow * H));
        lds_direct_load16(live(st, r) ? p : zero_row, lds0 + buf * S::XB + c * NT * 16);
      }
    }
#pragma unroll
    for (int c = 0; c < ZV; ++c) {
      const int r = zr + NT / ZP * c;
      const char *p = (const char *)((const T *)j.dZ + (size_t)row_at(st, r) * H + zc);
      lds_direct_load16(live(st, r) ? p : zero_row, lds0 + 2 * S::XB + buf * S::ZB + c * NT * 16);
    }
  };
  // pieces that are converted on their way: the extra columns (the upper half of the threads repeats the lower
  // half's), and the tiles of an ATTR product
  [[maybe_unused]] const int er = (tid % (NT / 2)) / EP, ec = (tid % EP) * V;
  [[maybe_unused]] Attr en, xn[KIND == WG_ATTR ? XV : 1];
  auto request = [&](int st) {
    if constexpr (ATTRS) en = load_attr(row_at(st, er), ec);
    if constexpr (KIND == WG_ATTR)
#pragma unroll
      for (int c = 0; c < XV; ++c) xn[c] = load_attr(row_at(st, xr + NT / XP * c), xc);
  };
  auto commit = [&](int st) {
    if constexpr (ATTRS) *(vec *)(Es + (st & 1) * S::EB + er * EP * 16 + ec * (int)sizeof(T)) = attr_operand(en, ec, live(st, er));
    if constexpr (KIND == WG_ATTR)
#pragma unroll
      for (int c = 0; c < XV; ++c)
        *(vec *)(Xs + (st & 1) * S::XB + (tid + NT * c) * 16) = attr_operand(xn[c], xc, live(st, xr + NT / XP * c));
  };
  auto arrived = [&]() {                                   // this wave's direct loads are in LDS
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
  };
  int ix1[XV];
  {
    int ix0[XV];
    load_idx(0, ix0);
    load_idx(1, ix1);
    request(0);
    fetch(0, ix0);
    commit(0);
    arrived();
  }
  __syncthreads();
  int xo[2], zo[NB];
#pragma unroll
  for (int m = 0; m < 2; ++m) xo[m] = wgrad_lane_offset<T, XP>(lane, 2 * wa + m);
#pragma unroll
  for (int i = 0; i < NB; ++i) zo[i] = wgrad_lane_offset<T, ZP>(lane, wb * NB + i);
  [[maybe_unused]] const int eo = wgrad_lane_offset<T, EP>(lane, 0);
  [[maybe_unused]] int ez[NE];
#pragma unroll
  for (int i = 0; i < NE; ++i) ez[i] = wgrad_lane_offset<T, ZP>(lane, wb * NB + wa * NE + i);
  [[maybe_unused]] vec first_column = Opd::zero();         // EXTRA without attributes: column 0 all ones
  if constexpr (EXTRA && !ATTRS)
#pragma unroll
    for (int i = 0; i < V; ++i) first_column[i] = Opd::from_float((lane & 31) == 0 ? 1.f : 0.f);
  for (int st = 0; st < n_stage; ++st) {
    const int sn = st + 1;
    int ix2[XV];
    load_idx(st + 2 < n_stage ? st + 2 : st, ix2);
    if (sn < n_stage) {
      request(sn);
      fetch(sn, ix1);
    }
    const char *xs = Xs + (st & 1) * S::XB, *zs = Zs + (st & 1) * S::ZB;
#pragma unroll
    for (int k = 0; k < RS / ST; ++k) {
      vec xa[2], xb[NB];
#pragma unroll
      for (int m = 0; m < 2; ++m) xa[m] = lds_column_operand<T, XP>(xs + xo[m] + ST * k * XP * 16);
#pragma unroll
      for (int i = 0; i < NB; ++i) xb[i] = lds_column_operand<T, ZP>(zs + zo[i] + ST * k * ZP * 16);
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < NB; ++i) Opd::mma(xa[m], xb[i], acc[m][i]);
      if constexpr (EXTRA) {
        if (wa * NE < NB) {                                // (uniform; fewer blocks than waves at H = 64, and at H = 128 with eight waves)
          vec xe = first_column;
          if constexpr (ATTRS) xe = lds_column_operand<T, EP>(Es + (st & 1) * S::EB + eo + ST * k * EP * 16);
#pragma unroll
          for (int i = 0; i < NE; ++i) Opd::mma(xe, lds_column_operand<T, ZP>(zs + ez[i] + ST * k * ZP * 16), acce[i]);
        }
      }
    }
    if (sn < n_stage) commit(sn);
    arrived();
    __syncthreads();
    if constexpr (S::FOLD > 0) {
      if (sn % (S::FOLD / RS) == 0 && sn < n_stage) fold();
    }
#pragma unroll
    for (int c = 0; c < XV; ++c) ix1[c] = ix2[c];
  }
}

template <typename T, int H, int TA, int RS>
__global__ __launch_bounds__(2 * TA, 2) void wgrad_kernel(const WgradLaunch a) {
  using S = WgradShape<T, H, TA, RS>;
  constexpr int NB = S::NB, NE = S::NE;
  extern __shared__ __align__(16) char smem[];
  const WgradPlace place = wgrad_place(a, blockIdx.x);
  if (place.job == kWgradMaxJobs) return;
  const WgradJob &j = a.job[place.job];
  touch_args(j);
  const int kq = place.kq, y = place.y;
  const int ka0 = kq * TA;
  const int64_t r_begin = (int64_t)y * j.rows_per_slice;
  const int64_t r_end = r_begin + j.rows_per_slice < j.n_rows ? r_begin + j.rows_per_slice : j.n_rows;
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave % S::WA, wb = wave / S::WA;
  const bool extra = j.extra && kq == 0;

  WgradSums<T, H, TA, RS> sums;
  sums.clear();
  float *const out0 = j.partial + (size_t)y * j.KaP * H;
  bool put_before = false;
  auto put = [&]() __attribute__((always_inline)) {
    float *out = out0 + (size_t)(ka0 + 64 * wa) * H + 32 * wb * NB + l32;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < NB; ++i) wgrad_put<H>(out + (size_t)32 * m * H + 32 * i, g, put_before, sums.main[m][i]);
    if (extra && wa * NE < NB) {
      float *oe = out0 + (size_t)j.kt * TA * H + 32 * (wb * NB + wa * NE) + l32;
#pragma unroll
      for (int i = 0; i < NE; ++i) wgrad_put<H>(oe + 32 * i, g, put_before, sums.extra[i]);
    }
    put_before = true;
  };
  // with: the extra columns too
  auto run = [&](auto kind, auto with) {
    constexpr int KIND = decltype(kind)::value;
    constexpr bool WITH = decltype(with)::value;
    const char *zeros = (const char *)a.zero_row;
    if constexpr (S::SECOND) {
      WgradSums<T, H, TA, RS> second;
      second.clear();
      auto fold = [&]() __attribute__((always_inline)) { second.add(sums, WITH); sums.clear(); };
      wgrad_run<T, H, TA, RS, KIND, WITH>(j, zeros, ka0, r_begin, r_end, smem, sums, fold);
      sums.add(second, WITH);
    } else {
      auto fold = [&]() __attribute__((always_inline)) { put(); sums.clear(); };
      wgrad_run<T, H, TA, RS, KIND, WITH>(j, zeros, ka0, r_begin, r_end, smem, sums, fold);
    }
  };
  using std::integral_constant;
  typedef integral_constant<bool, true> yes;
  typedef integral_constant<bool, false> no;
  if (j.kind == WG_EDGE) {
    if (extra) run(integral_constant<int, WG_EDGE>(), yes());
    else run(integral_constant<int, WG_EDGE>(), no());
  } else if (j.kind == WG_NODE) {
    if (extra) run(integral_constant<int, WG_NODE>(), yes());
    else run(integral_constant<int, WG_NODE>(), no());
  } else if (j.kind == WG_PLAIN) {
    if (extra) run(integral_constant<int, WG_PLAIN>(), yes());
    else run(integral_constant<int, WG_PLAIN>(), no());
  } else {
    run(integral_constant<int, WG_ATTR>(), no());
  }
  put();
}

// dW[k, f] += sum over slices of partial[slice, k, f] for k < k_rows; db[f] += row bias_row. A block handles
// 32 consecutive entries of one job; its 8 thread groups take every eighth slice (eight loads in flight
// each) and their sums are added in group order, so the result has one fixed summation order.
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const WgradLaunch a, int H) {
  __shared__ float part[8][32];
  int ji = 0;                                                // (every job's first block in one batch of scalar loads, no search)
#pragma unroll
  for (int k = 1; k < kWgradMaxJobs; ++k) ji += (int)blockIdx.x >= a.entry0[k] ? 1 : 0;
  const WgradJob &j = a.job[ji];
  const int e = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int i = ((int)blockIdx.x - a.entry0[ji]) * 32 + e;   // (H is a multiple of 32: a block's entries are in one row)
  const int k = i / H, f = i - k * H;
  const bool bias = k >= j.k_rows;
  const float *p = j.partial + (size_t)(bias ? j.bias_row : k) * H + f;
  const size_t cs = (size_t)j.KaP * H;
  float s = 0.f;
  int c = g;
  for (; c + 56 < j.ny; c += 64) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(size_t)(c + 8 * u) * cs];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; c < j.ny; c += 8) s += p[(size_t)c * cs];
  part[g][e] = s;
  __syncthreads();
  if (g == 0) {
    float t = part[0][e];
#pragma unroll
    for (int u = 1; u < 8; ++u) t += part[u][e];
    if (!bias) j.dW[(size_t)k * H + f] += t;
    else j.db[f] += t;
  }
}

// ---- host: the plan of one launch
struct WgradPlan {
  int blocks = 0, entries = 0;         // of the products' launch and of the reduction's
  size_t partial_floats = 0;
};
// Cuts the rows of the jobs (n_rows, kind, Ka, De, db set; a reduction alone: kt = 0 with ny, KaP, k_rows and
// partial set) into slices of one length: the shortest multiple of `rs` whose blocks are resident at once,
// `resident` of them, evenly over the XCDs -- a second pass of a few blocks would take as long as the first.
inline WgradPlan plan_wgrads(WgradLaunch &a, int n, int H, int ta, int rs, int resident) {
  int64_t work = 0;
  for (int i = 0; i < n; ++i) {
    WgradJob &j = a.job[i];
    if (j.ny) continue;
    const bool edge = j.kind == WG_EDGE, node = j.kind == WG_NODE;
    const int main_cols = edge || node ? 2 * H : j.Ka;
    // an all-ones column of its own only where no tile has room for it
    j.extra = edge ? j.De < kWgradExtra : j.db && (node || (j.kind == WG_PLAIN && j.Ka % ta == 0));
    j.kt = (main_cols + (!edge && !node && j.db && !j.extra ? 1 : 0) + ta - 1) / ta;
    j.KaP = j.kt * ta + (j.extra ? kWgradExtra : 0);
    const int past = j.extra ? j.kt * ta : main_cols;          // first row behind the H-wide parts' (EDGE: kt ta = 2 H)
    if (!j.k_rows) j.k_rows = edge && j.extra ? 2 * H + j.De : main_cols;   // (given: the columns behind it are padding)
    j.bias_row = !j.db || (edge && !j.extra) ? -1 : edge ? past + j.De : past;
    work += (int64_t)j.kt * j.n_rows;
  }
  int most = 0;                        // blocks of the XCD that has most
  int64_t rps = std::max<int64_t>(64, (work + resident - 1) / resident);
  for (;; rps += std::max<int64_t>(rs, rps / 32)) {
    rps = (rps + rs - 1) / rs * rs;
    int load[8] = {};
    bool least = true;                 // every job has a single slice
    for (int kt = 8; kt >= 1; --kt)    // (wide jobs first: the others even out what they leave)
      for (int i = 0; i < n; ++i) {
        WgradJob &j = a.job[i];
        if (j.kt != kt && !(kt == 8 && j.kt > 8)) continue;
        j.rows_per_slice = (int)std::min<int64_t>(rps, INT32_MAX / 2);
        j.ny = (int)((j.n_rows + j.rows_per_slice - 1) / j.rows_per_slice);
        least &= j.ny == 1;
        int best_max = INT32_MAX;
        for (int rot = 0; rot < 8; ++rot) {
          int m = 0;
          for (int x = 0; x < j.ny % 8; ++x) m = std::max(m, load[(x + rot) % 8]);
          if (m < best_max) { best_max = m; j.rot = rot; }
        }
        for (int x = 0; x < 8; ++x) load[(x + j.rot) % 8] += j.kt * (j.ny / 8 + (x < j.ny % 8 ? 1 : 0));
      }
    most = *std::max_element(load, load + 8);
    if (8 * most <= resident || least) break;
  }
  WgradPlan p;
  p.blocks = 8 * most;
  for (int i = 0; i < kWgradMaxJobs; ++i) { a.tiles[i] = 0; a.entry0[i] = INT32_MAX; }
  for (int i = 0; i < n; ++i) {
    WgradJob &j = a.job[i];
    if (j.kt) a.tiles[i] = j.ny << 16 | j.rot << 8 | j.kt;
    a.entry0[i] = p.entries;
    p.entries += (j.k_rows + (j.bias_row >= 0 ? 1 : 0)) * (H / 32);
    if (j.kt) p.partial_floats += (size_t)j.ny * j.KaP * H;
  }
  return p;
}
// an upper bound of partial_floats for any jobs of one launch
inline size_t wgrad_partial_bound(int H, int ta, int resident, int De) {
  const int tiles = 2 * H / ta + 1 + (De + 1 + ta - 1) / ta;   // column tiles of a job at most
  return (size_t)std::max(resident, kWgradMaxJobs * tiles) * (ta + kWgradExtra) * H;
}
