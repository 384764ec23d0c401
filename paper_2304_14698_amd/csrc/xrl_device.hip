// Device side of the library: context, weight upload, workspace, kernel sequencing.
#include <hip/hip_runtime.h>

#include <pthread.h>
#include <sys/mman.h>

#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

#include "heads.hip.h"
#include "rowmm.hip.h"
#include "mlp2.hip.h"
#include "mlp2_bwd.hip.h"
#include "mlp2_bwdz.hip.h"
#include "mlp2p.hip.h"
#include "resident.hip.h"
#include "mlp2r.hip.h"
#include "gat.hip.h"
#include "wgrad.hip.h"
#include "segsum.hip.h"
#include "distinct.hip.h"
#include "room.h"
#include "xrl_internal.h"

using namespace xrl;

#define HIP_TRY(expr)                                                                       \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess)                                                                   \
      return fail(XRL_ERR_HIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, \
                  __LINE__);                                                                \
  } while (0)

namespace {

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

struct EncMlp {           // device pointers of one encoder MLP
  const void *W1s = nullptr, *W2s = nullptr;
  const void *W1p = nullptr, *W2p = nullptr;     // forward in parts (xrl_ctx::parts): edge and node MLPs
  const float *W1 = nullptr, *W2 = nullptr;      // as they are given
  const void *W2bt = nullptr, *W1bt = nullptr;   // backward: contraction over the weight's columns
  const float *b1 = nullptr, *b2 = nullptr;
  int nslab1 = 0;
  // embed MLP, in place of W1s: W1's rows for [edge-attr sum | dense attrs] in fragment order (fp32), and
  // its rows for the one-hot op type as a plain [Tn, H] table
  const void *W1x = nullptr;
  const float *table = nullptr;
  int nslabx = 0;
};

}  // namespace

// ---- fragment-ordered weight copies ----------------------------------------------------------
// SWZ_FRAGMENT (layer-1 weights): [slab][column block][lane][j]: lane l, element j of slab s holds
//   W[s*2V + (l/32)*V + j][32*cb + l%32], zero beyond K.
// SWZ_CHAIN, for a weight whose contraction index is fed from an accumulator tile:
//   [chunk][column block][lane][j], element j of chunk c in lane group g is contraction index
//   2V*c + 8*(j/4) + 4*g + j%4 (the accumulator layout), lane l addresses column 32*cb + l%32; used
//   for the forward's layer 2 and for the backward's W2^T and W1^T products.
// SWZ_FRAGMENT3, SWZ_CHAIN3: those orders for V = 8, each fragment as the three bf16 parts of its fp32 elements, the
//   lanes' first parts, then their second, then their third.
// SWZ_ROWS: [output tile][contraction group][lane][j]: lane l, element j of the row-MLPs' fragments (RowMap) holds
//   W[16 * group + 4 * (l / 16) + j][16 * tile + l % 16] (cb: contraction groups, n: outputs), zero beyond K and n.
// W[k][f] = weights[src + k' * sk + f * sf], k' = k, or k + k_gap from k_gap_at on.
enum { SWZ_FRAGMENT = 0, SWZ_CHAIN, SWZ_FRAGMENT3, SWZ_CHAIN3, SWZ_ROWS };
struct SwzJob {
  int64_t dst;       // byte offset of the copy
  int64_t src, n;    // flat offset; SWZ_ROWS: outputs
  int64_t groups;    // lane fragments of V elements
  int32_t kind, V, bf16, K, cb, sk, sf, k_gap_at, k_gap, pad;
};

namespace {
// One row of blocks (y) per copy, a lane fragment (16 bytes in bf16 and fp32 operands) per thread and
// step; the last rows copy the flat vector itself, four 16-byte pieces per thread. Bound by the latency of two round trips. (One
// row of blocks for the flat vector, 4 bytes a step, took 36 steps and most of the launch, and loads under conditions came one by one: H = 128, fp32 25 us, so 10; H = 256 47, so 17.)
constexpr int kFlatPieces = 4;
__global__ __launch_bounds__(256) void arrange_weights_kernel(const SwzJob *jobs, int n_jobs, const float *w, int64_t n_w,
                                                              char *dst, float *d_w) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if ((int)blockIdx.y >= n_jobs) {
    const int64_t n4 = n_w / 4, all = stride * (gridDim.y - n_jobs);
    i += stride * ((int)blockIdx.y - n_jobs);
    if (i < n_w - 4 * n4) d_w[4 * n4 + i] = w[4 * n4 + i];
    for (; i < n4; i += all * kFlatPieces) {
      f32x4 v[kFlatPieces];
#pragma unroll
      for (int k = 0; k < kFlatPieces; ++k) v[k] = ((const f32x4 *)w)[i + k * all < n4 ? i + k * all : i];
#pragma unroll
      for (int k = 0; k < kFlatPieces; ++k)
        if (i + k * all < n4) ((f32x4 *)d_w)[i + k * all] = v[k];
    }
    return;
  }
  const SwzJob j = jobs[blockIdx.y];
  for (; i < j.groups; i += stride) {
    const int l = (int)(i & 63), g = l >> 5;
    const int64_t t = i >> 6;
    const int cb = (int)(t % j.cb), s = (int)(t / j.cb);
    if (j.kind == SWZ_ROWS) {
      const int f = 16 * s + (l & 15), k0 = 16 * cb + 4 * (l >> 4), fc = f < (int)j.n ? f : (int)j.n - 1;
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = w[j.src + (int64_t)(k0 + e < j.K ? k0 + e : j.K - 1) * j.sk + (int64_t)fc * j.sf];
#pragma unroll
      for (int e = 0; e < 4; ++e) if (k0 + e >= j.K || f >= (int)j.n) o[e] = 0.f;
      ((f32x4 *)(dst + j.dst))[i] = o;
      continue;
    }
    const float *p = w + j.src + (int64_t)(32 * cb + (l & 31)) * j.sf;
    const bool frag = j.kind == SWZ_FRAGMENT || j.kind == SWZ_FRAGMENT3;
    float v[8];
    auto gather = [&](auto width) {      // (every load under no condition: all in flight at once)
      constexpr int V = decltype(width)::value;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const int k0 = frag ? s * 2 * V + g * V + e : 2 * V * s + 8 * (e >> 2) + 4 * g + (e & 3);
        int k = k0 < j.K ? k0 : j.K - 1;
        if (frag && k >= j.k_gap_at) k += j.k_gap;
        v[e] = p[(int64_t)k * j.sk];
      }
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const int k0 = frag ? s * 2 * V + g * V + e : 2 * V * s + 8 * (e >> 2) + 4 * g + (e & 3);
        if (k0 >= j.K) v[e] = 0.f;
      }
    };
    if (j.V == 8) gather(std::integral_constant<int, 8>());
    else gather(std::integral_constant<int, 4>());
    if (j.kind == SWZ_FRAGMENT3 || j.kind == SWZ_CHAIN3) {
      const Split3 parts = split3(v);
      for (int k = 0; k < 3; ++k) *(bf16x8 *)(dst + j.dst + ((t * 3 + k) * 64 + l) * 16) = parts.p[k];
    } else if (j.bf16) {
      *(bf16x8 *)(dst + j.dst + i * 16) = pack_bf16x8(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]);
    } else {
      float *o = (float *)(dst + j.dst) + i * j.V;
      for (int e = 0; e < j.V; ++e) o[e] = v[e];
    }
  }
}
}  // namespace

// kernels whose launches can be timed with HIP events (xrl_set_timing / xrl_read_timing; WGRAD_EDGE, _NODE and _EMBED, whose products
// share launches, are names that may still be read: no launch is only theirs)
enum { TK_EMBED = 0, TK_EDGE, TK_EDGE_FIXUP, TK_NODE, TK_POOL, TK_READOUT, TK_HEADS, TK_GAT_LINEAR,
       TK_GAT_AGGREGATE, TK_BWD_EDGE, TK_BWD_NODE, TK_BWD_EMBED, TK_WGRAD, TK_GRAD_GATHER, TK_GAT_BWD, TK_RESIDENT,
       TK_WGRAD_EDGE, TK_WGRAD_NODE, TK_WGRAD_EMBED, TK_ROUND, TK_LEVELS, TK_COUNT };
static const char *const kTimedNames[TK_COUNT] = {"embed", "edge", "edge_fixup", "node", "pool", "readout",
                                                  "heads", "gat_linear", "gat_aggregate", "bwd_edge", "bwd_node",
                                                  "bwd_embed", "wgrad", "grad_gather", "gat_bwd", "resident",
                                                  "wgrad_edge", "wgrad_node", "wgrad_embed", "round", "levels"};

constexpr int64_t kMaxFusedStates = 4096;  // most states that the heads' launch counts slots of
constexpr int kCounts = 3 * kMaxLevels;
constexpr int64_t kPersistentMinRows = 8192;   // rows from which the persistent kernels replace the split one
constexpr size_t kZeroRow = 1024 + 256;        // 1 KB of zeros and behind it one element that is 1 (see WgradLaunch)
constexpr size_t kGradRoom = (size_t)2 << 30;   // gradients kept for a launch of weight gradients (see encode_backward_impl)
constexpr size_t kSliceBytes = (size_t)4 << 20;   // table rows are gathered from by column slices: an XCD's L2
constexpr int kAvecChunks = 1024;              // most chunks of rows of an attention vector's gradient
constexpr int64_t kClusterMaxGraphs = 256; // largest G of the one-launch encoder with several blocks per graph

// Scratch of xrl_policy_value_static, the entry point that allocates nothing: per-state counters,
// the logits when the caller does not ask for them, and the per-state mean embeddings. One copy
// per GPU, held until the process ends; host code never passes the array's name to a kernel, only
// the address hipGetSymbolAddress reports for the current device (static_scratch below).
constexpr int64_t kStaticMaxSlots = kMaxFusedStates;         // G
constexpr int64_t kStaticMaxStateFloats = 65536;             // S * hidden
constexpr size_t kStaticCounterOff = 0;
constexpr size_t kStaticLogitOff = kStaticCounterOff + sizeof(int32_t) * kStaticMaxSlots;
constexpr size_t kStaticZmeanOff = kStaticLogitOff + sizeof(float) * kStaticMaxSlots;
constexpr size_t kStaticBytes = kStaticZmeanOff + sizeof(float) * kStaticMaxStateFloats;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

struct xrl_ctx {
  xrl_model_desc m;
  Layout L;
  hipStream_t stream = nullptr;
  int elem = 4;                 // bytes per stored activation / operand
  int n_cu = 256;               // compute units of the device
  int max_lds = 65536;          // LDS bytes one block may use
  int64_t p_min_rows = 8192;    // smallest row count for the persistent kernels (XRL_PERSISTENT_MIN_ROWS) when saving
  int64_t p_min_rows_forward = 8192;   // for the backward pass, and when not
  int64_t wide_min_rows = 1 << 18;   // rows of a launch's products from which 256-column weight-gradient tiles are used (XRL_WGRAD_WIDE_MIN_ROWS)
  int64_t pool_window_nodes = 4096;  // nodes per compute unit from which the pool's gradient of H = 256 goes by windows of graphs (XRL_POOL_WINDOW_NODES)
  int sum_steps = 0;                 // steps of a group of class_sum_kernel, 0: by the rows (XRL_SUM_STEPS)
  size_t grad_room = kGradRoom;      // XRL_GRAD_ROOM
  int64_t round_blocks = 0;          // blocks per compute unit up to which a round is one launch, see mlp2_round_kernel (XRL_ROUND_BLOCKS)
  bool round_any = false;            // ... whatever their in-edges (if it is set)
  int64_t resident_max_graphs = 0;   // largest batch (graphs) for the one-launch encoder (XRL_RESIDENT_MAX_GRAPHS)
  int64_t resident_max_tiles = 0;    // ... and the most 32-row tiles (nodes, or edges) of one graph (XRL_RESIDENT_MAX_TILES)
  float *d_w = nullptr;         // flat fp32 weights
  int32_t *d_counter = nullptr; // kMaxFusedStates per-state counters of heads_kernel, zero between launches
  unsigned *d_arrived = nullptr; // kClusterMaxGraphs per-graph counters of encode_cluster_kernel, zero between launches
  unsigned *h_fault = nullptr;   // pinned host word a kernel sets when one of its bounded waits gives up ...
  unsigned *d_fault = nullptr;   // ... and the address kernels write it through
  // mlp_layers = 1 (the layers of Section 3.4 exactly as printed: one learned matrix each) runs on the
  // two-layer kernels: the context's own model and layout (m, L) have a second layer whose matrix
  // is the identity and whose bias is zero -- relu(relu(z) I + 0) = relu(z) exactly, in both
  // precisions -- and the caller's one-layer vector is spread into that layout on upload. The
  // backward passes run on an internal gradient vector whose real tensors are then added to the
  // caller's (the identity layers' gradients are dropped).
  bool single_layer = false;
  Layout Lu;                      // the caller's layout (single_layer)
  float *d_dw_int = nullptr;      // [L.total] internal gradient vector (single_layer)
  int32_t *d_wmap = nullptr;      // [Lu.total] index in the internal vector of each of the caller's weights
  int64_t cluster_max_graphs = 0; // largest batch (graphs) for the one-launch encoder with several blocks per graph
  int64_t resident_max_forward = 0, cluster_max_forward = 0;   // the same two limits of encodes that do not save
  unsigned cluster_spin_limit = kClusterSpinLimit;   // polls after which one of its waits gives up (XRL_CLUSTER_SPIN_LIMIT)
  int device = 0;               // the device that was current at xrl_create
  char *static_ws = nullptr;    // this device's copy of `scratch` (its device address)
  void *zero_row = nullptr;     // 1 KB of zeros behind the weights
  bool agg_skip = false;        // last encode: the received-sum rows of nodes without in-edges were not written
                                // (their readers go by the batch's agg_src)
  char *d_swz = nullptr;        // fragment-ordered encoder weights, then the list they are made by
  size_t swz_bytes = 0;
  const SwzJob *swz_jobs = nullptr;   // device
  int n_swz_jobs = 0;
  int64_t swz_max_groups = 0;
  float *d_wstage = nullptr, *h_wstage = nullptr;   // new weights on their way (device; pinned host), internal layout
  hipEvent_t wstage_free = nullptr;   // recorded behind the last transfer out of h_wstage
  EncMlp embed;
  std::vector<EncMlp> edge, node;
  std::vector<const void *> gatW;   // XRL_ROUND_GAT: fragment-ordered W of each round
  std::vector<const void *> gatWt;  //   and of W^T (backward: dh = dz W^T)
  std::vector<float *> gat_ss, gat_sd;   // saved per-node scores of each round (inside ws)
  std::unordered_map<int64_t, RowMap> row_fwd, row_bwd;   // readout and head matrices in fragment order, and transposed
  // workspaces (grow-only): encoder activations, and a separate small one for the heads
  char *ws = nullptr;
  size_t ws_bytes = 0;
  char *hws = nullptr;
  size_t hws_bytes = 0;
  char *bws = nullptr;          // backward scratch
  size_t bws_bytes = 0;
  bool room_refused = false;    // (see fit_room)
  size_t levels_refused = SIZE_MAX;   // least size of ws with levels in it that there was no memory for
  // buffers of the last encode (inside ws)
  uint64_t id = 0;              // unique per context
  int32_t *d_counts = nullptr;  // class and tile counts of the levels of a batch, and their copy in pinned memory
  int32_t *h_counts = nullptr;
  int64_t distinct_min_us = 300;   // smallest estimated encode that is reduced to distinct nodes (XRL_DISTINCT_MIN_US;
                                   // 0 = every batch that can be, -1 = none)
  int64_t min_rows_now = 0;     // the one in force, or 1 for the levels of a reduced batch that is saved
  std::vector<void *> hx;       // last encode of a reduced batch: h of the level below, per class
  std::shared_ptr<DevicePool> blocks;
  hipStream_t copy_stream = nullptr;   // uploads of kCopyStreamBytes and more
  bool captured = false;        // calls on it have been captured: graphs hold addresses in the workspaces
  uint64_t enc_batch = 0;
  bool enc_saved = false;
  float *pool = nullptr, *carry = nullptr, *ro_act[2] = {nullptr, nullptr};
  std::vector<void *> h, agg;   // h[0..R], agg[1..R] (index 0 unused)
  // what the forward kernels of large bf16 batches keep for the backward pass (inside ws): relu(z1)
  // of the embed MLP and of every round's edge and node MLP, and the mask bits of every round's
  // per-edge output (which is summed per receiver and never stored itself)
  bool fwd_kept = false, embed_kept = false;   // (attention rounds: of the embed MLP alone)
  void *z1_embed = nullptr;
  std::vector<void *> z1_edge, z1_node;
  std::vector<uint16_t *> ym_edge, ym_node, zm_edge, zm_node;   // mask bits of y and of z1, per round
  uint16_t *ym_embed = nullptr, *zm_embed = nullptr;
  bool parts() const { return elem == 4 && m.hidden == 128; }   // the forward's edge and node MLPs run on mlp2_split3_kernel
  // optional per-kernel timing
  bool timing = false;
  struct Span { int kind; hipEvent_t a, b; };
  std::vector<Span> spans;
  std::vector<hipEvent_t> free_events;
};

namespace {
// Brackets the launches made during its lifetime with two events on the ctx stream.
struct Timed {
  xrl_ctx *c;
  int idx = -1;
  Timed(xrl_ctx *ctx, int kind) : c(ctx) {
    if (!c->timing) return;
    hipEvent_t ev[2];
    for (int i = 0; i < 2; ++i) {
      if (!c->free_events.empty()) { ev[i] = c->free_events.back(); c->free_events.pop_back(); }
      else if (hipEventCreate(&ev[i]) != hipSuccess) return;
    }
    c->spans.push_back({kind, ev[0], ev[1]});
    idx = (int)c->spans.size() - 1;
    (void)hipEventRecord(ev[0], c->stream);
  }
  ~Timed() { if (idx >= 0) (void)hipEventRecord(c->spans[idx].b, c->stream); }
};
}  // namespace

namespace {
// Device address of `scratch` on the current device, looked up once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char *g_scratch_ptr[kMaxDevices] = {};
int static_scratch(int dev, char **out) {
  if (dev < 0 || dev >= kMaxDevices) return fail(XRL_ERR_UNSUPPORTED, "device ordinal %d", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(XRL_ERR_HIP, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[dev] = (char *)p;
  }
  *out = g_scratch_ptr[dev];
  return XRL_OK;
}
}  // namespace

// ---- memory of packed batches ----------------------------------------------------------------
// Pinned host blocks and device blocks are kept when a batch is freed: pinning and unpinning, hipMalloc
// and hipFree (which waits for the whole device) and the page faults of fresh memory took most of
// packing and uploading a state of a few hundred thousand nodes. Both pools are bounded and are given
// back with the last context (host) or their context (device).
namespace {
constexpr size_t kMaxPinnedBlock = (size_t)128 << 20;    // larger batches stay in ordinary memory
constexpr size_t kMaxPinnedTotal = (size_t)1 << 30;      // pinned by all batches together
constexpr size_t kMaxIdlePinned = (size_t)256 << 20, kMaxIdleDevice = (size_t)1 << 30;
constexpr size_t kMaxIdleBlocks = 4;
constexpr size_t kCopyStreamBytes = (size_t)8 << 20;     // uploads from this size on leave on the copy stream

// capacity classes: four per power of two, so that batches of about one size share blocks
size_t block_capacity(size_t bytes) {
  size_t step = 16384;
  while (step * 8 < bytes) step *= 2;
  return (bytes + step - 1) / step * step;
}

struct HostPool {
  std::mutex mu;
  std::vector<HostBlock> idle;      // oldest first
  size_t idle_bytes = 0, pinned_bytes = 0;
  int contexts = 0;
  int device = 0;                   // that of the last context made, where blocks are pinned
  bool child = false;               // this process was forked off one that had a context: no HIP call from here
  struct Live { char *p; size_t cap; void *copy; };
  std::vector<Live> live;           // pinned blocks in the hands of batches (copy: while forking)
};
HostPool &host_pool() {
  static HostPool *p = new HostPool;   // (never destroyed: a batch may be freed by a static destructor)
  return *p;
}
// Pinned memory is not there in a forked process. It gets ordinary memory with the same contents at the same
// addresses for the batches it inherits, and none of the pool: it packs, views and frees batches like a
// process that never had a GPU.
void fork_prepare() {
  HostPool &hp = host_pool();
  hp.mu.lock();
  for (HostPool::Live &x : hp.live) {
    x.copy = mmap(nullptr, x.cap, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (x.copy != MAP_FAILED) memcpy(x.copy, x.p, x.cap);
  }
}
void fork_parent() {
  HostPool &hp = host_pool();
  for (HostPool::Live &x : hp.live)
    if (x.copy != MAP_FAILED) (void)munmap(x.copy, x.cap);
  hp.mu.unlock();
}
void fork_child() {
  HostPool &hp = host_pool();
  for (HostPool::Live &x : hp.live)
    if (x.copy != MAP_FAILED) (void)mremap(x.copy, x.cap, x.cap, MREMAP_MAYMOVE | MREMAP_FIXED, x.p);
  hp.live.clear();
  hp.idle.clear();
  hp.idle_bytes = hp.pinned_bytes = 0;
  hp.contexts = 0;
  hp.child = true;
  hp.mu.unlock();
}
// Blocks change hands in calls that touch no stream: they must not disturb a capture that this or another
// thread has under way.
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};
// Whether a call made while memory changes hands went well. A failure is dealt with on the spot and must not be
// found by the next check of a launch.
bool went_well(hipError_t e) {
  if (e != hipSuccess) (void)hipGetLastError();
  return e == hipSuccess;
}
// The calling thread's current device, for as long as this lives.
struct OnDevice {
  int before = 0;
  bool changed = false;
  explicit OnDevice(int device) {
    changed = went_well(hipGetDevice(&before)) && before != device && went_well(hipSetDevice(device));
  }
  ~OnDevice() { if (changed) (void)went_well(hipSetDevice(before)); }
};
void host_block_release(HostBlock &b) {
  if (!b.pinned) {
    free(b.p);
    b = HostBlock();
    return;
  }
  if (host_pool().child) {               // (see fork_child)
    (void)munmap(b.p, b.cap);
    b = HostBlock();
    return;
  }
  RelaxedCapture relaxed;
  if (b.copied) {
    (void)went_well(hipEventSynchronize((hipEvent_t)b.copied));
    (void)went_well(hipEventDestroy((hipEvent_t)b.copied));
  }
  (void)went_well(hipHostFree(b.p));
  b = HostBlock();
}
void host_pool_context(int change, int device = 0) {
  HostPool &hp = host_pool();
  static std::once_flag once;
  std::call_once(once, [] { (void)pthread_atfork(fork_prepare, fork_parent, fork_child); });
  std::vector<HostBlock> drop;
  {
    std::lock_guard<std::mutex> lk(hp.mu);
    if (hp.child) return;
    hp.contexts += change;
    if (change > 0) hp.device = device;
    if (hp.contexts == 0) {
      drop.swap(hp.idle);
      hp.pinned_bytes -= hp.idle_bytes;
      hp.idle_bytes = 0;
    }
  }
  for (HostBlock &b : drop) host_block_release(b);
}
}  // namespace

HostBlock host_block_take(size_t bytes) {
  HostPool &hp = host_pool();
  HostBlock b;
  const size_t cap = block_capacity(bytes);
  bool pin = false;
  int device = 0;
  std::unique_lock<std::mutex> lk(hp.mu);
  device = hp.device;
  if (hp.contexts > 0 && cap <= kMaxPinnedBlock) {
    RelaxedCapture relaxed;
    // the oldest idle block of a fitting class whose last transfer is over; one still being read by a
    // transfer only if no other block may be added
    int pick = -1, busy = -1;
    for (size_t i = 0; i < hp.idle.size() && pick < 0; ++i) {
      const HostBlock &x = hp.idle[i];
      if (x.cap < bytes || x.cap > 2 * cap) continue;
      if (!x.copied || went_well(hipEventQuery((hipEvent_t)x.copied))) pick = (int)i;
      else if (busy < 0) busy = (int)i;
    }
    if (pick < 0 && hp.idle.size() >= kMaxIdleBlocks) pick = busy;
    if (pick >= 0) {
      b = hp.idle[pick];
      hp.idle.erase(hp.idle.begin() + pick);
      hp.idle_bytes -= b.cap;
      hp.live.push_back({b.p, b.cap, nullptr});
    } else if (hp.pinned_bytes + cap <= kMaxPinnedTotal) {
      pin = true;
      hp.pinned_bytes += cap;
    }
  }
  lk.unlock();
  if (b.p) {
    RelaxedCapture relaxed;
    if (b.copied) (void)went_well(hipEventSynchronize((hipEvent_t)b.copied));
    return b;
  }
  b.cap = cap;
  if (pin) {
    RelaxedCapture relaxed;
    OnDevice on(device);                 // (the packing thread may never have chosen one)
    const hipError_t e = hipHostMalloc((void **)&b.p, cap, hipHostMallocPortable);
    lk.lock();
    if (e == hipSuccess) {
      b.pinned = true;
      hp.live.push_back({b.p, cap, nullptr});
      return b;
    }
    hp.pinned_bytes -= cap;
    lk.unlock();
    (void)hipGetLastError();
    b.p = nullptr;
  }
  b.p = (char *)aligned_alloc(4096, (cap + 4095) / 4096 * 4096);
  return b;
}

void host_block_give(HostBlock &b) {
  if (!b.p) return;
  if (b.pinned) {
    HostPool &hp = host_pool();
    std::lock_guard<std::mutex> lk(hp.mu);
    for (size_t i = 0; i < hp.live.size(); ++i)
      if (hp.live[i].p == b.p) { hp.live.erase(hp.live.begin() + i); break; }
    if (hp.contexts > 0 && hp.idle.size() < kMaxIdleBlocks && hp.idle_bytes + b.cap <= kMaxIdlePinned) {
      hp.idle.push_back(b);
      hp.idle_bytes += b.cap;
      b = HostBlock();
      return;
    }
    if (!hp.child) hp.pinned_bytes -= b.cap;
  }
  host_block_release(b);
}

// Idle device blocks of one context, reused by its later uploads. A block comes with an event behind its
// last use on the context's stream, for users on another stream (the copy stream).
struct DeviceBlock {
  void *p = nullptr;
  size_t cap = 0;
  hipEvent_t used = nullptr;         // nullptr: never used
};
struct DevicePool {
  std::mutex mu;
  std::vector<DeviceBlock> idle;     // oldest first
  size_t idle_bytes = 0;
  hipStream_t stream = nullptr;      // the context's
  int device = 0;                    // the stream's
  bool closed = false;
  // on_stream: the block will be used on the context's own stream, where its last use is over by then; else
  // a block whose last use is over already is preferred, and a new one to waiting
  hipError_t take(size_t bytes, bool on_stream, DeviceBlock *out) {
    const size_t cap = block_capacity(bytes);
    {
      std::lock_guard<std::mutex> lk(mu);
      int pick = -1, busy = -1;
      for (size_t i = 0; i < idle.size() && pick < 0; ++i) {
        if (idle[i].cap < bytes || idle[i].cap > 2 * cap) continue;
        if (on_stream || went_well(hipEventQuery(idle[i].used))) pick = (int)i;
        else if (busy < 0) busy = (int)i;
      }
      if (pick < 0 && idle.size() >= kMaxIdleBlocks) pick = busy;
      if (pick >= 0) {
        *out = idle[pick];
        idle_bytes -= out->cap;
        idle.erase(idle.begin() + pick);
        return hipSuccess;
      }
    }
    *out = DeviceBlock();
    out->cap = cap;
    return allocate(&out->p, cap);
  }
  // hipMalloc; where the device has no room, once more without the idle blocks
  hipError_t allocate(void **p, size_t bytes) {
    const hipError_t e = hipMalloc(p, bytes);
    if (went_well(e)) return e;
    std::vector<DeviceBlock> drop;
    {
      std::lock_guard<std::mutex> lk(mu);
      drop.swap(idle);
      idle_bytes = 0;
    }
    if (drop.empty()) return e;
    for (DeviceBlock &x : drop) release(x);
    const hipError_t again = hipMalloc(p, bytes);
    (void)went_well(again);
    return again;
  }
  void give(DeviceBlock &b) {
    if (!b.p) return;
    {
      std::lock_guard<std::mutex> lk(mu);
      OnDevice on(device);               // (the event and the stream have to be of one device)
      hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
      if (!closed && idle.size() < kMaxIdleBlocks && idle_bytes + b.cap <= kMaxIdleDevice &&
          went_well(hipStreamIsCapturing(stream, &cs)) && cs == hipStreamCaptureStatusNone &&
          (b.used || went_well(hipEventCreateWithFlags(&b.used, hipEventDisableTiming))) &&
          went_well(hipEventRecord(b.used, stream))) {
        idle.push_back(b);
        idle_bytes += b.cap;
        b = DeviceBlock();
        return;
      }
    }
    release(b);
  }
  static void release(DeviceBlock &b) {
    RelaxedCapture relaxed;
    if (b.p) (void)went_well(hipFree(b.p));     // (waits for the device)
    if (b.used) (void)went_well(hipEventDestroy(b.used));
    b = DeviceBlock();
  }
  void close() {
    std::lock_guard<std::mutex> lk(mu);
    closed = true;
    for (DeviceBlock &x : idle) release(x);
    idle.clear();
    idle_bytes = 0;
  }
};

// A graph in receiver order as the message kernels take it: the batch's own, or that of the
// representatives of one level (see distinct.hip.h).
struct LevelGraph {
  int64_t N = 0, E = 0, n_tiles = 0, receivers = 0;   // (receivers: nodes with in-edges, of a level)
  const int32_t *in_ptr = nullptr, *in_src = nullptr, *in_dst = nullptr, *out_ptr = nullptr, *out_pos = nullptr;
  const int32_t *tile_ptr = nullptr, *agg_src = nullptr, *node_op = nullptr;
  const float *edge_feat = nullptr, *node_dense = nullptr;
  // level l > 0: each class's class one level below, and the rows [edges | classes | received] grouped by
  // the class one level below that their gradients go to (see GroupArgs)
  int32_t *self = nullptr, *down_ptr = nullptr, *down = nullptr, *down_seg = nullptr;
  const int32_t *below_src = nullptr, *below_dst = nullptr;   // fp32: the classes one level below of each edge's sender and receiver
};
struct Distinct {
  int levels = 0;                          // rounds + 1
  LevelGraph lv[kMaxLevels];
  int32_t *cls[kMaxLevels] = {};           // [N] class of each node at each level
  int32_t *mem_ptr = nullptr, *mem_graph = nullptr, *mem_seg = nullptr;   // the batch's nodes by class at the last level
  bool grouped = false;                    // the groupings the backward pass needs have been made ...
  bool grouped_fold = false;               // ... for gradients that arrive summed per receiver
  DeviceBlock block[2];
};

extern "C" void xrl_batch_release_device(xrl_batch *b) {
  if (b && b->dev.block) {
    auto give = [&](DeviceBlock &x) {
      if (host_pool().child) x = DeviceBlock();        // (the device's memory is the parent's)
      else if (b->pool && !b->shared) b->pool->give(x);
      else DevicePool::release(x);
    };
    if (b->distinct)
      for (DeviceBlock &x : b->distinct->block) give(x);
    b->distinct.reset();
    DeviceBlock x;
    x.p = b->dev.block; x.cap = b->dev.bytes; x.used = (hipEvent_t)b->dev.used;
    give(x);
    b->pool.reset();
    b->dev = xrl_batch_device();
    b->uploaded = false;
  }
}

namespace {

// Internal index of the first element of the caller's tensor `t` (single-layer contexts): the tensor of
// the same name in the internal layout.
int64_t internal_offset(const xrl_ctx *c, const WeightTensor &t) {
  for (const WeightTensor &u : c->L.tensors)
    if (u.name == t.name) return u.offset;
  return -1;
}

// Where the fragment-ordered copies of the weights lie, and which rows and columns of the flat vector
// they are made of: fixed by the model, made once per context (plan_weights).
int plan_weights(xrl_ctx *c) {
  const xrl_model_desc &m = c->m;
  const int V = c->elem == 2 ? 8 : 4, H = m.hidden, De = m.d_edge, Tn = m.n_op_types, Dd = m.n_node_dense;
  size_t off = 0;
  std::vector<SwzJob> jobs;
  auto put = [&](SwzJob j) {
    j.dst = (int64_t)(off = align_up(off));
    off += (size_t)j.groups * (j.kind == SWZ_FRAGMENT3 || j.kind == SWZ_CHAIN3 ? 48 : j.V * (j.bf16 ? 2 : 4));
    jobs.push_back(j);
    return (size_t)j.dst;
  };
  // layer-1 order of a matrix given by its strides (sk between contraction rows, sf between columns)
  auto frag = [&](int64_t w, int K, int M, int v, bool bf16, int sk, int sf, int k_gap_at = 1 << 30, int k_gap = 0) {
    SwzJob j = {};
    j.kind = SWZ_FRAGMENT; j.V = v; j.bf16 = bf16 ? 1 : 0; j.K = K; j.cb = M / 32; j.src = w; j.sk = sk; j.sf = sf;
    j.k_gap_at = k_gap_at; j.k_gap = k_gap;
    j.groups = (int64_t)((K + 2 * v - 1) / (2 * v)) * j.cb * 64;
    return put(j);
  };
  auto chain = [&](int64_t w, int Kc, int M, int sk, int sf) {
    SwzJob j = {};
    j.kind = SWZ_CHAIN; j.V = V; j.bf16 = V == 8 ? 1 : 0; j.K = Kc; j.cb = M / 32; j.src = w; j.sk = sk; j.sf = sf;
    j.groups = (int64_t)(Kc / (2 * V)) * j.cb * 64;
    return put(j);
  };
  struct Ref { size_t w1 = 0, w2, w2bt, w1bt = 0, w1x = 0, w1p = 0, w2p = 0; int ns = 0, nsx = 0; };
  std::vector<Ref> refs;
  const bool b16 = c->elem == 2;
  auto add = [&](const MlpRef &r, bool embed) {
    Ref ref;
    if (embed) {                                        // (see EncMlp::W1x: fp32 operands in both modes, the one-hot rows left out)
      ref.w1x = frag(r.w[0], De + Dd, H, 4, false, H, 1, De, Tn);
      ref.nsx = (De + Dd + 7) / 8;
    } else {
      ref.w1 = frag(r.w[0], r.d_in[0], H, V, b16, H, 1);
      ref.ns = (r.d_in[0] + 2 * V - 1) / (2 * V);
    }
    ref.w2 = chain(r.w[1], H, H, H, 1);
    ref.w2bt = chain(r.w[1], H, H, 1, H);               // W2^T
    if (!embed) ref.w1bt = chain(r.w[0], H, 2 * H, 1, H);   // (W1^T)[:, :2H]: edge and node MLPs
    if (!embed && c->parts()) {                         // forward of fp32 edge and node MLPs: in parts
      auto parts = [&](int64_t w, int K, int kind) {
        SwzJob j = {};
        j.kind = kind; j.V = 8; j.K = K; j.cb = H / 32; j.src = w; j.sk = H; j.sf = 1;
        j.k_gap_at = 1 << 30;
        j.groups = (int64_t)((K + 15) / 16) * j.cb * 64;
        return put(j);
      };
      ref.w1p = parts(r.w[0], r.d_in[0], SWZ_FRAGMENT3);
      ref.w2p = parts(r.w[1], H, SWZ_CHAIN3);
    }
    refs.push_back(ref);
  };
  add(c->L.embed, true);
  const bool gat = m.round_kind == XRL_ROUND_GAT;
  std::vector<size_t> gat_off, gat_off_t;
  for (int r = 0; r < m.rounds; ++r) {
    if (gat) {                                          // W and W^T of each round
      gat_off.push_back(frag(c->L.gat[r].W, H, H, V, b16, H, 1));
      gat_off_t.push_back(frag(c->L.gat[r].W, H, H, V, b16, 1, H));
    } else {
      add(c->L.edge[r], false);
      add(c->L.node[r], false);
    }
  }
  // the row-MLPs' matrices, keyed by flat offset: fragments of y = x W and of its transpose
  struct RowRef { int64_t w; int n_in, n_out; size_t fwd, bwd; };
  std::vector<RowRef> row_maps;
  auto rows = [&](int64_t w, int K, int64_t n, int sk, int sf) {
    SwzJob j = {};
    j.kind = SWZ_ROWS; j.V = 4; j.K = K; j.n = n; j.cb = (K + 15) / 16; j.src = w; j.sk = sk; j.sf = sf;
    j.groups = (n + 15) / 16 * j.cb * 64;
    return put(j);
  };
  for (const MlpRef *r : {&c->L.readout, &c->L.policy, &c->L.value})
    for (int l = 0; l < r->n_layers; ++l) {
      const int in = r->d_in[l], out = r->d_out[l];
      row_maps.push_back({r->w[l], in, out, rows(r->w[l], in, out, out, 1), rows(r->w[l], out, in, 1, out)});
    }
  const size_t o_jobs = align_up(off);
  c->swz_bytes = o_jobs + jobs.size() * sizeof(SwzJob);
  HIP_TRY(hipMalloc((void **)&c->d_swz, c->swz_bytes));
  HIP_TRY(hipMemcpy(c->d_swz + o_jobs, jobs.data(), jobs.size() * sizeof(SwzJob), hipMemcpyHostToDevice));
  c->swz_jobs = (const SwzJob *)(c->d_swz + o_jobs);
  c->n_swz_jobs = (int)jobs.size();
  c->swz_max_groups = 0;
  for (const SwzJob &j : jobs) c->swz_max_groups = std::max(c->swz_max_groups, j.groups);
  HIP_TRY(hipMalloc((void **)&c->d_wstage, sizeof(float) * (size_t)c->L.total));
  HIP_TRY(hipHostMalloc((void **)&c->h_wstage, sizeof(float) * (size_t)c->L.total, hipHostMallocDefault));
  HIP_TRY(hipEventCreateWithFlags(&c->wstage_free, hipEventDisableTiming));
  if (c->single_layer) {
    // the inserted second layers: identity matrices and zero biases, written once
    memset(c->h_wstage, 0, sizeof(float) * (size_t)c->L.total);
    auto identity = [&](const MlpRef &r) {
      for (int k = 0; k < H; ++k) c->h_wstage[(size_t)r.w[1] + (size_t)k * H + k] = 1.f;
    };
    identity(c->L.embed);
    identity(c->L.readout);
    for (const MlpRef &r : c->L.edge) identity(r);
    for (const MlpRef &r : c->L.node) identity(r);
  }
  auto bind = [&](EncMlp &e, const Ref &ref, const MlpRef &r) {
    e.W1s = c->d_swz + ref.w1;
    e.W2s = c->d_swz + ref.w2;
    e.W1p = c->d_swz + ref.w1p;
    e.W2p = c->d_swz + ref.w2p;
    e.W1 = c->d_w + r.w[0];
    e.W2 = c->d_w + r.w[1];
    e.W2bt = c->d_swz + ref.w2bt;
    e.W1bt = c->d_swz + ref.w1bt;
    e.b1 = c->d_w + r.b[0];
    e.b2 = c->d_w + r.b[1];
    e.nslab1 = ref.ns;
    e.W1x = c->d_swz + ref.w1x;
    e.nslabx = ref.nsx;
    e.table = c->d_w + r.w[0] + (size_t)m.d_edge * H;    // meaningful for the embed MLP only
  };
  for (const RowRef &r : row_maps) {
    c->row_fwd[r.w] = RowMap{(const f32x4 *)(c->d_swz + r.fwd), r.n_in, r.n_out};
    c->row_bwd[r.w] = RowMap{(const f32x4 *)(c->d_swz + r.bwd), r.n_out, r.n_in};
  }
  size_t i = 0;
  bind(c->embed, refs[i++], c->L.embed);
  if (gat) {
    for (int r = 0; r < m.rounds; ++r) {
      c->gatW.push_back(c->d_swz + gat_off[r]);
      c->gatWt.push_back(c->d_swz + gat_off_t[r]);
    }
    return XRL_OK;
  }
  c->edge.resize(m.rounds);
  c->node.resize(m.rounds);
  for (int r = 0; r < m.rounds; ++r) {
    bind(c->edge[r], refs[i++], c->L.edge[r]);
    bind(c->node[r], refs[i++], c->L.node[r]);
  }
  return XRL_OK;
}

// dst[0 .. n) = src[0 .. n); false when an element is not finite
bool copy_finite(float *dst, const float *src, int64_t n) {
  memcpy(dst, src, sizeof(float) * (size_t)n);
  const uint32_t *u = (const uint32_t *)dst;
  uint32_t bad = 0;
  for (int64_t i = 0; i < n; ++i) bad |= (uint32_t)((u[i] & 0x7f800000u) == 0x7f800000u);
  return bad == 0;
}

// Calls that send host memory which may change or go away after they return: a replay would read it again.
int refuse_capture(const xrl_ctx *c, const char *who) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(c->stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone) return XRL_OK;
  (void)hipGetLastError();
  return fail(XRL_ERR_HIP, "%s: the stream is being captured", who);
}

// New weights: copied (and checked) piece by piece into pinned memory, each piece on its way to the GPU
// while the next is copied, then one kernel writes the flat vector and every fragment-ordered
// copy. Queued on the context's stream; the caller's vector is free on return. A value that is not
// finite leaves the old weights in place. From the call until the GPU is done, five rounds: 0.15 ms at
// H = 128 (2.6 MB), 0.35 ms at H = 256 (9.4 MB), of which the caller's thread is held 0.08 and 0.26 ms by
// the copy and its check; one thread arranging the copies on the host took 2.3 and 10.5 ms.
int upload_weights(xrl_ctx *c, const float *w_user) {
  if (int rc = refuse_capture(c, "xrl_set_weights")) return rc;
  HIP_TRY(hipEventSynchronize(c->wstage_free));            // the pinned copy of the call before has left
  constexpr int64_t kPiece = 1 << 16;                       // floats: stays in the core's cache between copy and check
  constexpr int64_t kSend = 1 << 19;                        // floats per transfer
  int64_t sent = 0;
  auto send = [&](int64_t end, bool all) -> int {
    if (end - sent < kSend && !all) return XRL_OK;
    if (end > sent)
      HIP_TRY(hipMemcpyAsync(c->d_wstage + sent, c->h_wstage + sent, sizeof(float) * (size_t)(end - sent),
                             hipMemcpyHostToDevice, c->stream));
    sent = end;
    return XRL_OK;
  };
  auto take = [&](int64_t to, int64_t from, int64_t n) -> int {
    for (int64_t i = 0; i < n; i += kPiece) {
      const int64_t k = std::min(kPiece, n - i);
      if (!copy_finite(c->h_wstage + to + i, w_user + from + i, k)) {
        int64_t at = from + i;
        while (std::isfinite(w_user[at])) ++at;
        return fail(XRL_ERR_VALUE, "weights[%lld] is not finite", (long long)at);
      }
      const int rc = send(to + i + k, false);
      if (rc) return rc;
    }
    return XRL_OK;
  };
  int rc = XRL_OK;
  if (c->single_layer) {                                    // (tensors in the order of the internal vector too)
    for (const WeightTensor &t : c->Lu.tensors) {
      const int64_t n = t.cols > 0 ? t.rows * t.cols : t.rows;
      if ((rc = take(internal_offset(c, t), t.offset, n))) break;
    }
  } else {
    rc = take(0, 0, c->L.total);
  }
  if (!rc) rc = send(c->L.total, true);
  (void)hipEventRecord(c->wstage_free, c->stream);
  if (rc) return rc;
  const unsigned gx = (unsigned)std::min<int64_t>((c->swz_max_groups + 255) / 256, 256);
  const unsigned flat = (unsigned)((c->L.total / 4 + (int64_t)gx * 256 * kFlatPieces - 1) / ((int64_t)gx * 256 * kFlatPieces));
  arrange_weights_kernel<<<dim3(gx, (unsigned)c->n_swz_jobs + std::max(flat, 1u)), dim3(256), 0, c->stream>>>(
      c->swz_jobs, c->n_swz_jobs, c->d_wstage, c->L.total, c->d_swz, c->d_w);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

int ensure_ws(xrl_ctx *c, size_t bytes) {
  if (bytes <= c->ws_bytes) return XRL_OK;
  HIP_TRY(hipStreamSynchronize(c->stream));
  if (c->ws) HIP_TRY(hipFree(c->ws));
  c->ws = nullptr;
  c->ws_bytes = 0;
  c->enc_batch = 0;
  c->enc_saved = false;
  hipError_t e = c->blocks->allocate((void **)&c->ws, bytes);
  if (e != hipSuccess) {
    c->ws = nullptr;
    return fail(XRL_ERR_OOM, "workspace of %zu bytes: %s", bytes, hipGetErrorString(e));
  }
  c->ws_bytes = bytes;
  return XRL_OK;
}

int ensure_buf(xrl_ctx *c, char **buf, size_t *have, size_t bytes, const char *what) {
  if (bytes <= *have) return XRL_OK;
  HIP_TRY(hipStreamSynchronize(c->stream));
  if (*buf) HIP_TRY(hipFree(*buf));
  *buf = nullptr;
  *have = 0;
  hipError_t e = c->blocks->allocate((void **)buf, bytes);
  if (e != hipSuccess) {
    *buf = nullptr;
    return fail(XRL_ERR_OOM, "%s of %zu bytes: %s", what, bytes, hipGetErrorString(e));
  }
  *have = bytes;
  return XRL_OK;
}
int ensure_hws(xrl_ctx *c, size_t bytes) { return ensure_buf(c, &c->hws, &c->hws_bytes, bytes, "head workspace"); }
int ensure_bws(xrl_ctx *c, size_t bytes) { return ensure_buf(c, &c->bws, &c->bws_bytes, bytes, "backward workspace"); }

__global__ void fill_zero_kernel(float *p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

struct Bump {
  char *base;
  size_t off = 0;
  template <typename T> T *take(size_t n) {
    T *p = (T *)(base + off);
    off += align_up(n * sizeof(T));
    return p;
  }
};

bool is_capturing(const xrl_ctx *c) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  return went_well(hipStreamIsCapturing(c->stream, &cap)) && cap != hipStreamCaptureStatusNone;
}

int check_batch(xrl_ctx *c, const xrl_batch *b, const char *who) {
  if (!c || !b) return fail(XRL_ERR_NULL, "%s: ctx or batch is NULL", who);
  if (!b->uploaded) return fail(XRL_ERR_STATE, "%s: batch was not uploaded (xrl_batch_upload)", who);
  const xrl_model_desc &x = c->m, &y = b->model;
  if (x.n_op_types != y.n_op_types || x.n_node_dense != y.n_node_dense || x.d_edge != y.d_edge ||
      x.d_global != y.d_global)
    return fail(XRL_ERR_SHAPE, "%s: batch was packed for different feature widths", who);
  if (b->owner != c->id) {               // uploaded by another context, perhaps on another stream
    const_cast<xrl_batch *>(b)->shared = true;
    RelaxedCapture relaxed;              // (this stream or another may be under capture: the wait is no part of it)
    if (b->mem.copied) HIP_TRY(hipEventSynchronize((hipEvent_t)b->mem.copied));
  }
  if (!(c->captured && b->shared) && is_capturing(c)) {
    c->captured = true;
    const_cast<xrl_batch *>(b)->shared = true;   // (replays may run on any stream)
  }
  return XRL_OK;
}

// ---------------------------------------------------------------- launch helpers
template <typename TIn, typename TOut, int VEC, int RT>
int launch_segsum_rt(xrl_ctx *c, const void *vals, const int32_t *perm, const int32_t *ptr,
                     const int32_t *row_seg, int64_t n_rows, int64_t n_seg, int D, void *out,
                     float *carry) {
  if (n_seg == 0) return XRL_OK;
  if (n_rows == 0) {
    static_assert(sizeof(TOut) == 4, "zero fill below writes fp32 words");
    const int64_t n = n_seg * D;
    fill_zero_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream>>>((float *)out, n);
    HIP_TRY(hipGetLastError());
    return XRL_OK;
  }
  SegsumArgs a;
  a.vals = vals; a.perm = perm; a.ptr = ptr; a.n_rows = n_rows; a.n_seg = n_seg;
  a.zero_row = c->zero_row;
  a.row_seg = perm ? nullptr : row_seg;
  a.D = D; a.RT = RT; a.out = out; a.carry = carry;
  const int64_t nsub = (n_rows + RT - 1) / RT;
  const int64_t threads = nsub * (D / VEC);
  const int64_t blocks = (threads + 255) / 256;
  segsum_kernel<TIn, TOut, VEC, RT><<<dim3((unsigned)blocks), dim3(256), 0, c->stream>>>(a);
  const int64_t fthreads = nsub * (D / 4);
  segsum_fixup<TOut><<<dim3((unsigned)((fthreads + 255) / 256)), dim3(256), 0, c->stream>>>(
      ptr, row_seg, n_rows, n_seg, D, RT, carry, (TOut *)out);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

// Rows per sub-tile: 16 keeps sixteen 16-byte loads in flight per lane; tiny inputs (under 1 MB)
// use 4 so that they still produce a few waves per compute unit.
inline int segsum_rt(int64_t n_rows, int D, size_t elem) { return (size_t)n_rows * D * elem < ((size_t)1 << 20) ? 4 : 16; }

template <typename TIn, typename TOut, int VEC>
int launch_segsum(xrl_ctx *c, const void *vals, const int32_t *perm, const int32_t *ptr,
                  const int32_t *row_seg, int64_t n_rows, int64_t n_seg, int D, void *out,
                  float *carry) {
  if (segsum_rt(n_rows, D, sizeof(TIn)) == 4)
    return launch_segsum_rt<TIn, TOut, VEC, 4>(c, vals, perm, ptr, row_seg, n_rows, n_seg, D, out, carry);
  return launch_segsum_rt<TIn, TOut, VEC, 16>(c, vals, perm, ptr, row_seg, n_rows, n_seg, D, out, carry);
}

size_t segsum_carry_floats(int64_t n_rows, int D) { return (size_t)((n_rows + 3) / 4) * 2 * D; }

template <typename T1, typename T, int H, int KIND>
int launch_mlp2_split(xrl_ctx *c, const Mlp2Args &a) {
  using S = SplitTile<T, H>;
  auto kern = mlp2_split_kernel<T1, T, H, KIND>;
  static bool attr_set = false;          // one attribute per kernel instantiation
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, S::BYTES));
    attr_set = true;
  }
  kern<<<dim3((unsigned)((a.n_blocks + 7) / 8 * 8)), dim3(2 * H), S::BYTES, c->stream>>>(a);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

// Whole rounds (see mlp2_round_kernel): forward only, where the two kernels of a round would be split ones, up to
// round_blocks blocks per compute unit whose fullest has kRoundEdges in-edges, which are 32 at a time one pass after the other
// where a launch of their own takes them side by side.
template <typename T, int H>
int launch_round_h(xrl_ctx *c, const RoundArgs &a) {
  if constexpr (RoundTile<T, H>::FITS) {
    auto kern = mlp2_round_kernel<T, H>;
    static bool attr_set = false;
    if (!attr_set) {
      HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, RoundTile<T, H>::BYTES));
      attr_set = true;
    }
    kern<<<dim3((unsigned)((a.node.n_blocks + 7) / 8 * 8)), dim3(2 * H), RoundTile<T, H>::BYTES, c->stream>>>(a);
    HIP_TRY(hipGetLastError());
    return XRL_OK;
  }
  return fail(XRL_ERR_UNSUPPORTED, "launch_round_h: hidden = %d", H);
}
int64_t round_nodes(const xrl_ctx *c, int64_t N) {        // of a block
  return std::max<int64_t>(kRoundNodesMin, std::min<int64_t>(kRoundNodesMax, (N + c->n_cu - 1) / c->n_cu));
}
// in_ptr: the graph's, on the host; nullptr for a level of a reduced batch, where only the mean is known, and half as much
// again left for the fullest block.
template <typename T>
bool round_applies(const xrl_ctx *c, const LevelGraph &g, const int32_t *in_ptr) {
  const int H = c->m.hidden;
  const bool fits = H == 64 ? RoundTile<T, 64>::FITS : H == 128 ? RoundTile<T, 128>::FITS : RoundTile<T, 256>::FITS;
  if (std::max(g.N, g.E) >= c->min_rows_now) return false;      // (the persistent kernels')
  if (!fits || g.N <= 0 || g.N > kRoundNodesMax * c->round_blocks * c->n_cu) return false;
  if (c->round_any) return true;
  const int64_t nodes = round_nodes(c, g.N);
  if (!in_ptr) return g.E * nodes * 3 <= kRoundEdges * 2 * g.N;
  for (int64_t n = 0; n < g.N; n += nodes)                      // (at most round_blocks n_cu blocks, or N / 16)
    if (in_ptr[std::min(n + nodes, g.N)] - in_ptr[n] > kRoundEdges) return false;
  return true;
}
template <typename T>
int launch_round(xrl_ctx *c, RoundArgs &a) {
  a.nodes = (int)round_nodes(c, a.node.n_rows);
  a.node.n_blocks = (a.node.n_rows + a.nodes - 1) / a.nodes;
  switch (c->m.hidden) {
    case 64: return launch_round_h<T, 64>(c, a);
    case 128: return launch_round_h<T, 128>(c, a);
    case 256: return launch_round_h<T, 256>(c, a);
  }
  return fail(XRL_ERR_UNSUPPORTED, "hidden = %d", c->m.hidden);
}

template <int H, int KIND>
int launch_mlp2_split3(xrl_ctx *c, const Mlp2Args &a) {
  using S = Split3Tile<H>;
  auto kern = mlp2_split3_kernel<H, KIND>;
  static bool attr_set = false;          // one attribute per kernel instantiation
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, S::BYTES));
    attr_set = true;
  }
  kern<<<dim3((unsigned)((a.n_blocks + 7) / 8 * 8)), dim3(2 * H), S::BYTES, c->stream>>>(a);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

template <typename T, int H>
int launch_mlp2_h(xrl_ctx *c, int kind, const Mlp2Args &a) {
  if (a.n_rows <= 0) return XRL_OK;
  if constexpr (sizeof(T) == 4 && H == 128) {              // (xrl_ctx::parts)
    if (kind == KIND_EDGE) return launch_mlp2_split3<H, KIND_EDGE>(c, a);
    if (kind == KIND_NODE) return launch_mlp2_split3<H, KIND_NODE>(c, a);
    return launch_mlp2_split<float, T, H, KIND_EMBED>(c, a);
  } else {
  if (kind == KIND_EMBED) return launch_mlp2_split<float, T, H, KIND_EMBED>(c, a);
  if (kind == KIND_EDGE) return launch_mlp2_split<T, T, H, KIND_EDGE>(c, a);
  return launch_mlp2_split<T, T, H, KIND_NODE>(c, a);
  }
}

// Persistent LDS-resident-weights variant (bf16, H <= 128, edge and node kinds).
constexpr int kPersistWaves = 8;
inline size_t mlp2p_lds_bytes(int H, int nslab1) {
  const int MB = H / 32, HS = H / 16;
  return ((size_t)nslab1 * MB + (size_t)HS * MB) * 1024 + (size_t)MB * 256 +
         (size_t)kPersistWaves * RowStage<bf16_t, 128>::BYTES;   // staging sized for the widest H served
}

template <int H, int KIND, bool SAVE>
int launch_mlp2p_ks(xrl_ctx *c, Mlp2Args &a, size_t lds) {
  constexpr int NW = kPersistWaves;
  auto kern = mlp2p_kernel<bf16_t, H, KIND, NW, SAVE>;
  static bool attr_set = false;          // one attribute per kernel instantiation
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr_set = true;
  }
  const int64_t n_wt = KIND == KIND_EDGE ? a.n_tiles : (a.n_rows + 31) / 32;
  a.n_blocks = n_wt;
  int64_t grid = ((n_wt + NW - 1) / NW + 7) / 8 * 8;
  const int64_t cap = (int64_t)c->n_cu / 8 * 8;
  if (grid > cap) grid = cap;
  kern<<<dim3((unsigned)grid), dim3(64 * NW), lds, c->stream>>>(a);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

template <int H, int KIND>
int launch_mlp2p_k(xrl_ctx *c, Mlp2Args &a, size_t lds) {
  return a.z1 ? launch_mlp2p_ks<H, KIND, true>(c, a, lds) : launch_mlp2p_ks<H, KIND, false>(c, a, lds);
}

template <int H>
int launch_mlp2p(xrl_ctx *c, int kind, Mlp2Args &a) {
  const size_t lds = mlp2p_lds_bytes(H, a.nslab1);
  if (kind == KIND_EDGE) return launch_mlp2p_k<H, KIND_EDGE>(c, a, lds);
  return launch_mlp2p_k<H, KIND_NODE>(c, a, lds);
}

constexpr int embedp_waves(int H) { return H > 128 ? 4 : kPersistWaves; }
inline size_t embedp_lds_bytes(int H, int nslabx, int Tn) {
  const int MB = H / 32, HS = H / 16;
  const size_t w = ((size_t)nslabx * MB + (size_t)HS * MB) * 1024 + (size_t)MB * 256;
  if (H > 128) return w + (size_t)embedp_waves(H) * BlockStage<bf16_t>::BYTES;     // table stays in global memory
  return w + (size_t)Tn * H * 4 + (size_t)kPersistWaves * RowStage<bf16_t, 128>::BYTES;
}

template <int H, bool SAVE, bool LEVEL = false>
int launch_embedp_s(xrl_ctx *c, Mlp2Args &a) {
  constexpr int NW = embedp_waves(H);
  const size_t lds = embedp_lds_bytes(H, a.nslabx, a.Tn);
  auto kern = embedp_kernel<bf16_t, H, NW, SAVE, LEVEL>;
  static size_t attr_lds = 0;
  if (lds > attr_lds) {
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr_lds = lds;
  }
  const int64_t n_wt = (a.n_rows + 31) / 32;
  a.n_blocks = n_wt;
  int64_t grid = ((n_wt + NW - 1) / NW + 7) / 8 * 8;
  const int per_cu = 2 * lds <= (size_t)c->max_lds ? 2 : 1;   // blocks that fit a CU's LDS
  const int64_t cap = (int64_t)c->n_cu / 8 * 8 * per_cu;
  if (grid > cap) grid = cap;
  kern<<<dim3((unsigned)grid), dim3(64 * NW), lds, c->stream>>>(a);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

template <int H>
int launch_embedp(xrl_ctx *c, Mlp2Args &a) {
  return a.z1 ? launch_embedp_s<H, true>(c, a) : launch_embedp_s<H, false>(c, a);
}

inline bool mlp2p_applies(const xrl_ctx *c, int kind, const Mlp2Args &a) {
  const int H = c->m.hidden;
  if (c->elem != 2 || a.n_rows <= 0) return false;
  if (a.n_rows < c->min_rows_now) return false;
  if (kind == KIND_EMBED) {
    const int pieces = 4 * 64 * embedp_waves(H);             // see embedp_kernel
    return a.nslabx <= 2 && a.nslabx * (H / 32) * 64 <= pieces && (H > 128 || a.Tn * (H / 4) <= pieces) &&
           embedp_lds_bytes(H, a.nslabx, a.Tn) <= (size_t)c->max_lds;
  }
  if (H > 128) return false;
  if (kind == KIND_EDGE && a.nslab1 != 2 * (H / 16) + 1) return false;   // edge attrs must fit one slab
  return mlp2p_lds_bytes(H, a.nslab1) <= (size_t)c->max_lds;
}

// Register-stationary variant (bf16, edge and node kinds).
template <int H, int KIND, bool SAVE, bool LEVEL = false>
int launch_mlp2r_ks(xrl_ctx *c, Mlp2Args &a) {
  using R = RTile<H, KIND>;
  auto kern = mlp2r_kernel<H, KIND, SAVE, LEVEL>;
  static bool attr_set = false;
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, R::BYTES));
    attr_set = true;
  }
  const int64_t n_wt = KIND == KIND_EDGE ? a.n_tiles : (a.n_rows + 31) / 32;
  a.n_blocks = n_wt;
  const int by_lds = c->max_lds / R::BYTES, by_waves = 4 * R::WAVES_PER_SIMD / R::MB;
  const int per_cu = by_lds < by_waves ? by_lds : by_waves;      // blocks that can be resident on a CU
  int64_t grid = (n_wt + 7) / 8 * 8;
  const int64_t cap = (int64_t)c->n_cu / 8 * 8 * per_cu;
  if (grid > cap) grid = cap;
  kern<<<dim3((unsigned)grid), dim3(R::NT), R::BYTES, c->stream>>>(a);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

template <int H, int KIND>
int launch_mlp2r_k(xrl_ctx *c, Mlp2Args &a) {
  return a.z1 ? launch_mlp2r_ks<H, KIND, true>(c, a) : launch_mlp2r_ks<H, KIND, false>(c, a);
}

template <int H>
int launch_mlp2r(xrl_ctx *c, int kind, Mlp2Args &a) {
  return kind == KIND_EDGE ? launch_mlp2r_k<H, KIND_EDGE>(c, a) : launch_mlp2r_k<H, KIND_NODE>(c, a);
}

inline bool mlp2r_applies(const xrl_ctx *c, int kind, const Mlp2Args &a) {
  // H = 256 only: at H <= 128 the weights fit LDS, a wave then runs its tile without block
  // barriers, and that kernel (mlp2p) measured faster (the template itself covers 64 and 128)
  const int H = c->m.hidden;
  if (c->elem != 2 || H != 256 || kind == KIND_EMBED || a.n_rows <= 0) return false;
  if (a.n_rows < c->min_rows_now) return false;
  if (kind == KIND_EDGE && (a.De > 8 || a.nslab1 != 2 * (H / 16) + 1)) return false;   // edge attrs: half a slab
  return RTile<256, KIND_EDGE>::BYTES <= c->max_lds;
}

template <typename T>
int launch_mlp2(xrl_ctx *c, int kind, Mlp2Args &a) {
  if (mlp2r_applies(c, kind, a))
    return launch_mlp2r<256>(c, kind, a);
  if (mlp2p_applies(c, kind, a)) {
    if (kind == KIND_EMBED)
      return c->m.hidden == 64 ? launch_embedp<64>(c, a) : c->m.hidden == 128 ? launch_embedp<128>(c, a) : launch_embedp<256>(c, a);
    return c->m.hidden == 64 ? launch_mlp2p<64>(c, kind, a) : launch_mlp2p<128>(c, kind, a);
  }
  a.n_blocks = kind == KIND_EDGE ? a.n_tiles : (a.n_rows + 31) / 32;
  switch (c->m.hidden) {
    case 64: return launch_mlp2_h<T, 64>(c, kind, a);
    case 128: return launch_mlp2_h<T, 128>(c, kind, a);
    case 256: return launch_mlp2_h<T, 256>(c, kind, a);
  }
  return fail(XRL_ERR_UNSUPPORTED, "hidden = %d", c->m.hidden);
}

// z = h W of the attention rounds (and the backward's dh = dz W^T): W in LDS where it fits.
template <typename T, int H>
int launch_gat_linear_h(xrl_ctx *c, GatArgs &a) {
  using S = GatLds<T, H>;
  if constexpr (S::FITS) {
    auto kern = gat_linear_lds_kernel<T, H>;
    static bool attr_set = false;
    if (!attr_set) {
      HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, S::BYTES));
      attr_set = true;
    }
    const int64_t n_wt = (a.n_rows + 31) / 32, want = ((n_wt + S::NW - 1) / S::NW + 7) / 8 * 8;
    const int64_t cap = (int64_t)c->n_cu / 8 * 8 * S::PER_CU;
    kern<<<dim3((unsigned)std::min(want, cap)), dim3(64 * S::NW), S::BYTES, c->stream>>>(a);
  } else {
    a.n_blocks = (a.n_rows + 127) / 128;
    gat_linear_kernel<T, H><<<dim3((unsigned)((a.n_blocks + 7) / 8 * 8)), dim3(256), 0, c->stream>>>(a);
  }
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}
template <typename T>
int launch_gat_linear(xrl_ctx *c, GatArgs &a) {
  switch (c->m.hidden) {
    case 64: return launch_gat_linear_h<T, 64>(c, a);
    case 128: return launch_gat_linear_h<T, 128>(c, a);
    case 256: return launch_gat_linear_h<T, 256>(c, a);
  }
  return fail(XRL_ERR_UNSUPPORTED, "hidden = %d", c->m.hidden);
}

// An attention round's aggregation with the product of the next round, where W fits LDS twice per compute unit and there
// are few tiles per block: with more the barriers cost what the launches and the way of h through memory did
// (the figures at gat_round_kernel).
constexpr int64_t kGatRoundRows = 65536;
template <typename T>
bool gat_round_applies(const xrl_ctx *c, int64_t n) {
  const int H = c->m.hidden;
  return n <= kGatRoundRows && ((H == 64 && GatRound<T, 64>::FITS) || (H == 128 && GatRound<T, 128>::FITS));
}
template <typename T, int H>
int launch_gat_round_h(xrl_ctx *c, const GatArgs &a, const GatNext &next) {
  using S = GatRound<T, H>;
  if constexpr (S::FITS) {
    auto kern = gat_round_kernel<T, H>;
    static bool attr_set = false;
    if (!attr_set) {
      HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, S::BYTES));
      attr_set = true;
    }
    const int64_t want = ((a.n_rows + 31) / 32 + 7) / 8 * 8, cap = (int64_t)c->n_cu / 8 * 8 * S::PER_CU;
    kern<<<dim3((unsigned)std::min(want, cap)), dim3(S::NT), S::BYTES, c->stream>>>(a, next);
    HIP_TRY(hipGetLastError());
  }
  return XRL_OK;
}
template <typename T>
int launch_gat_round(xrl_ctx *c, const GatArgs &a, const GatNext &next) {
  return c->m.hidden == 64 ? launch_gat_round_h<T, 64>(c, a, next) : launch_gat_round_h<T, 128>(c, a, next);
}

// Beyond 64 KB, with what a kernel holds besides, a launch has to be allowed its LDS: 71 KB for the backward pass of heads of 256 and 64 at
// H = 256, more for wider ones and for hundreds of global attributes. The permission is the process's, one per kernel, while the size is a
// context's; so it is given once, for the most that any model needs: rows of 512 forward, heads of 512 and 512 back.
constexpr int kRowWidest = 512;
const size_t kRowForwardMost = row_lds_floats(row_pitch(kRowWidest)) * sizeof(float);
const size_t kRowBackwardMost = sizeof(float) * kRowTile * 4 * row_pitch(kRowWidest);
template <auto KERN>
int allow_row_lds(size_t most) {
  static std::atomic<bool> allowed{false};
  if (!allowed.load(std::memory_order_relaxed)) {
    HIP_TRY(hipFuncSetAttribute((const void *)KERN, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most));
    allowed.store(true, std::memory_order_relaxed);
  }
  return XRL_OK;
}
template <auto KERN, typename... Args>
int launch_rows(size_t most, int64_t blocks, size_t lds_floats, hipStream_t stream, const Args &...args) {
  const size_t lds = lds_floats * sizeof(float);
  if (int rc = allow_row_lds<KERN>(most)) return rc;
  KERN<<<dim3((unsigned)blocks), dim3(kRowThreads), lds, stream>>>(args...);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}
inline int64_t row_blocks(int64_t n) { return (n + kRowTile - 1) / kRowTile; }

// go(forward widths, backward widths) of the heads and of the readout MLP: the paper's head widths are known to the kernels, any
// others asked for; the readout's backward pass stops at the pool (the global attributes are inputs). Others of up to 128 have a kernel
// that never takes two tiles a wave, of half the registers, two blocks on a compute unit: us forward / forward and backward at H = 128, by vector
// code / with one kernel for all widths / so: heads of 17 and 3, 20 k slots 46 / 59 / 33 and 137 / 106 / 71, of 128 and 64 72 / 75 / 43 and 227 / 140 / 97,
// 15 slots 14.2 / 13.5 / 13.0 and 34 / 30 / 28. Wider: of 512 and 512, 4624 slots 189 / 87 / 75 and 553 / 230 / 209, 257 slots 43 / 45 / 39 and
// 141 / 109 / 98 (with few slots they go by launch_heads' rule).
template <typename Go>
int with_head_widths(const xrl_ctx *c, Go go) {
  const bool paper = c->m.head_hidden[0] == 256 && c->m.head_hidden[1] == 64, narrow = std::max(c->m.head_hidden[0], c->m.head_hidden[1]) <= 16 * kRowWaves;
  auto of = [&](auto h) -> int {
    constexpr int H = decltype(h)::value;
    return paper ? go(RowWidths<H, 256, 64, 1>(), RowWidths<1, 64, 256, H>()) :
           narrow ? go(RowWidths<H, kNarrow, kNarrow, 1>(), RowWidths<1, kNarrow, kNarrow, H>()) :
                    go(RowWidths<H, kAnyWidth, kAnyWidth, 1>(), RowWidths<1, kAnyWidth, kAnyWidth, H>());
  };
  return c->m.hidden == 64 ? of(std::integral_constant<int, 64>()) : c->m.hidden == 128 ? of(std::integral_constant<int, 128>()) :
                                                                                         of(std::integral_constant<int, 256>());
}
template <typename Go>
int with_readout_widths(const xrl_ctx *c, Go go) {
  return c->m.hidden == 64 ? go(RowWidths<kAnyWidth, 64, 64>(), RowWidths<64, 64, 64>()) :
         c->m.hidden == 128 ? go(RowWidths<kAnyWidth, 128, 128>(), RowWidths<128, 128, 128>()) : go(RowWidths<kAnyWidth, 256, 256>(), RowWidths<256, 256, 256>());
}

RowFwdArgs row_fwd_args(const xrl_ctx *c, const MlpRef &r, bool relu_last, const float *in1, int w1, const float *in2, int w2,
                        int64_t n_rows, float *out, float *const *act) {
  RowFwdArgs a;
  memset(&a, 0, sizeof(a));
  a.relu_last = relu_last ? 1 : 0;
  int widest = r.d_in[0];
  for (int l = 0; l < r.n_layers; ++l) {
    a.map[l] = c->row_fwd.at(r.w[l]);
    a.b[l] = c->d_w + r.b[l];
    a.act[l] = act ? act[l] : nullptr;
    widest = std::max(widest, r.d_out[l]);
  }
  a.in1 = in1; a.in2 = in2; a.w1 = w1; a.w2 = w2; a.n_rows = n_rows; a.out = out;
  a.pitch = row_pitch(widest);
  return a;
}
int launch_readout(xrl_ctx *c, const RowFwdArgs &a) {
  if (a.n_rows <= 0) return XRL_OK;
  return with_readout_widths(c, [&](auto fwd, auto) {
    return launch_rows<row_forward_kernel<decltype(fwd)>>(kRowForwardMost, row_blocks(a.n_rows), row_lds_floats(a.pitch), c->stream, a);
  });
}

// States per block of what the heads do a state at a time: one while each gets a block of its own on the chip, then as many as
// share the value head's fragments
inline int value_rows(const xrl_ctx *c, int64_t S) {
  return (int)std::min<int64_t>(kRowTile, (S + c->n_cu - 1) / c->n_cu);
}
// Policy MLP, per-state softmax statistics and value head (Section 3.3.2) in one launch; a batch of more states than there
// are counters runs the softmax in a second one. pact / vact (nullable) receive every layer's output for the backward
// pass, which has no use for what the softmax gives: logp null leaves it out.
int launch_heads(xrl_ctx *c, const xrl_batch *b, const float *d_emb, float *logit, float *logp, float *entropy,
                 int32_t *action, float *zmean, float *value, float *const *pact, float *const *vact, int32_t *counter) {
  const int H = c->m.hidden;
  const xrl_batch_device &d = b->dev;
  HeadsArgs a;
  a.policy = row_fwd_args(c, c->L.policy, false, d_emb, H, nullptr, 0, b->G, logit, pact);
  a.value = row_fwd_args(c, c->L.value, false, nullptr, H, nullptr, 0, b->S, value, vact);
  const bool counted = b->S <= kMaxFusedStates;
  a.mask = d.mask; a.state_graph_ptr = d.state_graph_ptr; a.G = (int)b->G; a.S = (int)b->S;
  a.value_rows = value_rows(c, b->S);
  a.counter = counter; a.logp = counted ? logp : nullptr; a.entropy = entropy; a.action = action; a.zmean = zmean;
  const int64_t blocks = row_blocks(b->G) + (b->S + a.value_rows - 1) / a.value_rows;
  const int rc = with_head_widths(c, [&](auto fwd, auto) {
    using W = decltype(fwd);
    // (heads wider than 128: a slot or state a block, by vector instructions, where each block has a compute unit to itself, of H <= 128 half of one.
    // us by vector code of another order / sixteen slots a block / so: heads of 512 and 512, H = 256, 15 slots 34 / 42 / 22, 254 47 / 44 / 27, 258 47 / 44 / 44;
    // H = 128 31 / 37 / 20, 42 / 39 / 25, 42 / 39 / 31, 701 47 / 41 / 52; of 300 and 100, H = 128, 15 slots 16 / 18 / 13, 258 19 / 20 / 16, 511 25 / 20 / 20.)
    if constexpr (W::wide)
      if (b->G + b->S <= (H == 256 ? 1 : 2) * c->n_cu) return launch_rows<heads_kernel<W, true>>(kRowForwardMost, b->G + b->S, kRowOneFloats, c->stream, a);
    return launch_rows<heads_kernel<W, false>>(kRowForwardMost, blocks, row_lds_floats(a.policy.pitch), c->stream, a);
  });
  if (rc) {
    // (a launch that the runtime rejected has not run; one that failed later may have left
    // counters of unfinished states above zero: they go back to zero before the next use)
    if (counter == c->d_counter) (void)hipMemsetAsync(counter, 0, sizeof(int32_t) * kMaxFusedStates, c->stream);
    return rc;
  }
  if (logp && !counted) {
    state_policy_kernel<<<dim3((unsigned)b->S), dim3(kRowThreads), 0, c->stream>>>(logit, d.mask, d.state_graph_ptr, logp, entropy, action);
    HIP_TRY(hipGetLastError());
  }
  return XRL_OK;
}

// row_src (or nullptr): the row of src to export for each row, -1 = a row of zeros; cls (or nullptr): the
// row instead, where row_src does not say zeros
template <typename T>
__global__ void export_rows_kernel(const T *src, int64_t n_rows, int D, const int32_t *row_src, const int32_t *cls, float *dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_rows * D) return;
  if (row_src || cls) {
    const int64_t r = i / D;
    const int64_t s = row_src && row_src[r] < 0 ? -1 : (cls ? cls[r] : row_src[r]);
    dst[i] = s < 0 ? 0.f : (float)src[s * D + (i - r * D)];
    return;
  }
  dst[i] = (float)src[i];
}


template <typename T, int H, int KIND>
int launch_mlp2_bwd_k(xrl_ctx *c, const Mlp2BwdArgs &a) {
  constexpr int lds = BwdTile<T, H>::BYTES;
  auto kern = mlp2_bwd_kernel<T, H, KIND>;
  static bool attr_set = false;          // one attribute per kernel instantiation
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    attr_set = true;
  }
  kern<<<dim3((unsigned)((a.n_blocks + 7) / 8 * 8)), dim3(2 * H), lds, c->stream>>>(a);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

// Edge and node MLPs in bf16 from many rows on: a wave per tile, four of them sharing the weights' way from L2. It takes as long
// for a part of a pass of the chip (H = 64: 131 k rows, 128: 66 k, 256: 33 k) as for a whole one, so it is taken by the share of its passes
// that is filled. us, split / wide, by that share: H = 64, edge 0.39 14.6 / 15.1, 0.57 19.1 / 18.6, 0.62 32.3 / 29.0, 0.81 98.2 / 83.2, node 0.54 18.7 / 21.3,
// 0.62 20.5 / 21.6, 0.67 37.9 / 37.4, 0.72 23.6 / 22.4; H = 128, edge 0.63 26.3 / 26.8, 0.65 44.1 / 41.8, 0.72 81.3 / 68.1, 0.98 34.4 / 28.8, node 0.62 41.2 /
// 42.9, 0.69 94.4 / 84.7; H = 256, edge 0.76 124.8 / 131.8 and 174.8 / 185.8, 0.79 81.2 / 88.2, 0.87 238 / 234, 0.995 271 / 242, node 0.75 75.3 / 78.8, 0.83
// 214 / 210, 0.93 101 / 88.9.
template <int H, int KIND>
int launch_mlp2_bwd_wide(xrl_ctx *c, const Mlp2BwdArgs &args, bool *launched) {
  auto kern = mlp2_bwd_wide_kernel<H, KIND>;
  static std::atomic<int> per_cu{0};     // blocks resident on a compute unit
  int fit = per_cu;
  if (!fit) {
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, BwdWide<H>::BYTES));
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit, (const void *)kern, 256, BwdWide<H>::BYTES));
    per_cu = fit = std::max(fit, 1);
  }
  constexpr int64_t kFilled = H == 64 ? (KIND == KIND_EDGE ? 50 : 66) : H == 128 ? 65 : 82;    // percent
  Mlp2BwdArgs a = args;
  a.n_blocks = (a.n_rows + 127) / 128;
  const int64_t pass = (int64_t)fit * c->n_cu, passes = (a.n_blocks + pass - 1) / pass;
  *launched = 100 * a.n_blocks >= kFilled * passes * pass;
  if (!*launched) return XRL_OK;
  kern<<<dim3((unsigned)((a.n_blocks + 7) / 8 * 8)), dim3(256), BwdWide<H>::BYTES, c->stream>>>(a);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

template <typename T, int H>
int launch_mlp2_bwd_h(xrl_ctx *c, int kind, const Mlp2BwdArgs &a) {
  if (a.n_rows <= 0) return XRL_OK;
  if (kind == KIND_EMBED) return launch_mlp2_bwd_k<T, H, KIND_EMBED>(c, a);
  if constexpr (sizeof(T) == 2) {
    bool launched = false;
    const int rc = kind == KIND_EDGE ? launch_mlp2_bwd_wide<H, KIND_EDGE>(c, a, &launched) : launch_mlp2_bwd_wide<H, KIND_NODE>(c, a, &launched);
    if (rc || launched) return rc;
  }
  if (kind == KIND_EDGE) return launch_mlp2_bwd_k<T, H, KIND_EDGE>(c, a);
  return launch_mlp2_bwd_k<T, H, KIND_NODE>(c, a);
}

template <typename T>
int launch_mlp2_bwd(xrl_ctx *c, int kind, Mlp2BwdArgs &a) {
  a.n_blocks = (a.n_rows + 31) / 32;
  switch (c->m.hidden) {
    case 64: return launch_mlp2_bwd_h<T, 64>(c, kind, a);
    case 128: return launch_mlp2_bwd_h<T, 128>(c, kind, a);
    case 256: return launch_mlp2_bwd_h<T, 256>(c, kind, a);
  }
  return fail(XRL_ERR_UNSUPPORTED, "hidden = %d", c->m.hidden);
}

template <int H, int KIND, bool FOLD, bool GIVEN = false>
int launch_mlp2_bwdz_k(xrl_ctx *c, Mlp2BwdzArgs &a) {
  using S = BwdzShape<H>;
  auto kern = mlp2_bwdz_kernel<H, KIND, FOLD, GIVEN>;
  static bool attr_set = false;          // one attribute per kernel instantiation
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS));
    attr_set = true;
  }
  const int64_t wave_tiles = KIND == KIND_EDGE ? a.n_tiles : (a.n_rows + 31) / 32;   // EDGE: the packer's edge tiles
  a.n_blocks = (wave_tiles + S::NW - 1) / S::NW;               // groups of NW tiles
  const unsigned grid = (unsigned)((a.n_blocks + 7) / 8 * 8);
  kern<<<dim3(grid), dim3(64 * S::NW), S::LDS, c->stream>>>(a);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

template <int H>
int launch_mlp2_bwdz_h(xrl_ctx *c, int kind, Mlp2BwdzArgs &a, bool fold, bool given) {
  if (a.n_rows <= 0) return XRL_OK;
  if (kind == KIND_EMBED)
    return given ? launch_mlp2_bwdz_k<H, KIND_EMBED, false, true>(c, a) : launch_mlp2_bwdz_k<H, KIND_EMBED, false>(c, a);
  if (kind == KIND_EDGE) return fold ? launch_mlp2_bwdz_k<H, KIND_EDGE, true>(c, a) : launch_mlp2_bwdz_k<H, KIND_EDGE, false>(c, a);
  return given ? launch_mlp2_bwdz_k<H, KIND_NODE, false, true>(c, a) : launch_mlp2_bwdz_k<H, KIND_NODE, false>(c, a);
}

// fold (EDGE): dx_b receives the gradients w.r.t. h_receiver summed per receiver, [N, H].
// given (NODE, EMBED): a.dy is dz2 already (the gradient gather applied the layer's output mask)
int launch_mlp2_bwdz(xrl_ctx *c, int kind, Mlp2BwdzArgs &a, bool fold, bool given) {
  switch (c->m.hidden) {
    case 64: return launch_mlp2_bwdz_h<64>(c, kind, a, fold, given);
    case 128: return launch_mlp2_bwdz_h<128>(c, kind, a, fold, given);
    case 256: return launch_mlp2_bwdz_h<256>(c, kind, a, fold, given);
  }
  return fail(XRL_ERR_UNSUPPORTED, "hidden = %d", c->m.hidden);
}

// Weight-gradient products waiting for one launch (see wgrad.hip.h), and the memory their partials go to.
struct WgradQueue {
  WgradLaunch a;
  int n = 0;
  float *partial = nullptr;
  size_t partial_floats = 0;
};
constexpr int wgrad_rows(size_t elem, int ta) { return elem == 2 ? ta / 4 : 16; }   // rows per stage: 32 and 64 in bf16
// Memory for the partials of a launch's jobs: those on 256-column and those on 128-column tiles.
inline size_t wgrad_partial_floats(const xrl_ctx *c) {
  const int H = c->m.hidden, De = c->m.d_edge;
  return wgrad_partial_bound(H, 128, 2 * c->n_cu, De) + (c->elem == 2 && H == 256 ? wgrad_partial_bound(H, 256, c->n_cu, De) : 0);
}

template <typename T, int H, int TA>
int launch_wgrads(xrl_ctx *c, WgradLaunch &a, int n, float *partial, size_t floats, size_t *used) {
  constexpr int RS = wgrad_rows(sizeof(T), TA);
  using S = WgradShape<T, H, TA, RS>;
  const WgradPlan p = plan_wgrads(a, n, H, TA, RS, c->n_cu * 256 / TA);
  if (p.partial_floats > floats) return fail(XRL_ERR_STATE, "weight gradients: %zu floats of partial sums, %zu planned", p.partial_floats, floats);
  for (int i = 0; i < n; ++i)
    if (a.job[i].kt) {
      a.job[i].partial = partial;
      partial += (size_t)a.job[i].ny * a.job[i].KaP * H;
    }
  *used = p.partial_floats;
  a.zero_row = c->zero_row;
  auto kern = wgrad_kernel<T, H, TA, RS>;
  static bool attr_set = false;          // one attribute per kernel instantiation
  if (!attr_set) {
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS));
    attr_set = true;
  }
  if (p.blocks > 0) kern<<<dim3((unsigned)p.blocks), dim3(S::NT), S::LDS, c->stream>>>(a);
  if (p.entries > 0) wgrad_reduce_kernel<<<dim3((unsigned)p.entries), dim3(256), 0, c->stream>>>(a, H);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

// Launches what waits. At H = 256, 256-column tiles where the H-wide parts fill them and enough rows wait that the
// chip's blocks, one per CU, are long against their start: products of 68 k rows in all 87 / 98 us (128-column /
// 256-column tiles), 250 k 147 / 147, 437 k 202 / 198, 671 k 268 / 258, 1.2 M 405 / 379, 3 M 1188 / 960. At H = 128 the
// second layers' products do not fill them and the others gain too little: 1.4 M rows, all on
// 128-column tiles 187 us, two launches 110 + 85.
template <typename T>
int flush_wgrads(xrl_ctx *c, WgradQueue &q) {
  if (q.n == 0) return XRL_OK;
  Timed t(c, TK_WGRAD);
  const int n = q.n;
  q.n = 0;
  float *partial = q.partial;
  size_t left = q.partial_floats, used = 0;
  auto run = [&](auto h) -> int {
    constexpr int H = decltype(h)::value;
    int n_narrow = n;
    if constexpr (sizeof(T) == 2 && H == 256) {
      int64_t rows = 0;
      for (int i = 0; i < n; ++i) rows += q.a.job[i].n_rows;
      if (rows >= c->wide_min_rows) {
        WgradLaunch wide;
        int n_wide = 0;
        n_narrow = 0;
        for (int i = 0; i < n; ++i) {
          const WgradJob j = q.a.job[i];
          const bool fits = j.kind == WG_EDGE || j.kind == WG_NODE || (j.kind == WG_PLAIN && j.Ka % 256 == 0 && j.ny == 0);
          if (fits) wide.job[n_wide++] = j;
          else q.a.job[n_narrow++] = j;
        }
        const int rc = n_wide ? launch_wgrads<T, H, 256>(c, wide, n_wide, partial, left, &used) : XRL_OK;
        if (rc) return rc;
        partial += used;
        left -= used;
      }
    }
    return n_narrow ? launch_wgrads<T, H, 128>(c, q.a, n_narrow, partial, left, &used) : XRL_OK;
  };
  switch (c->m.hidden) {
    case 64: return run(std::integral_constant<int, 64>());
    case 128: return run(std::integral_constant<int, 128>());
    case 256: return run(std::integral_constant<int, 256>());
  }
  return fail(XRL_ERR_UNSUPPORTED, "hidden = %d", c->m.hidden);
}

// Puts a product in the queue (launching what waits when the queue is full). EDGE: the attributes become a product of
// their own when they are too wide for the extra columns.
template <typename T>
int queue_wgrad(xrl_ctx *c, WgradQueue &q, const WgradJob &job) {
  if (job.n_rows <= 0) return XRL_OK;
  if (q.n + 2 > kWgradMaxJobs)
    if (int rc = flush_wgrads<T>(c, q)) return rc;
  q.a.job[q.n++] = job;
  if (job.kind == WG_EDGE && job.De >= kWgradExtra) {
    q.a.job[q.n - 1].db = nullptr;
    WgradJob attr = job;
    attr.kind = WG_ATTR;
    attr.Ka = job.De;
    attr.dW = job.dW + (size_t)2 * c->m.hidden * c->m.hidden;
    q.a.job[q.n++] = attr;
  }
  return XRL_OK;
}

RowBwdArgs row_bwd_args(const xrl_ctx *c, const MlpRef &r, bool relu_last, float *const *act, const float *dout,
                        int64_t n_rows, float *const *dz, float *dx) {
  RowBwdArgs a;
  memset(&a, 0, sizeof(a));
  a.relu_last = relu_last ? 1 : 0;
  int widest = r.d_in[0];
  for (int l = 0; l < r.n_layers; ++l) {
    a.map[r.n_layers - 1 - l] = c->row_bwd.at(r.w[l]);
    a.act[l] = act[l];
    a.dz[l] = dz[l];
    widest = std::max(widest, r.d_out[l]);
  }
  a.dout = dout; a.n_rows = n_rows; a.dx = dx;
  a.n_layers = r.n_layers;
  a.pitch = row_pitch(widest);
  return a;
}
int launch_readout_backward(xrl_ctx *c, const RowBwdArgs &a) {
  if (a.n_rows <= 0) return XRL_OK;
  return with_readout_widths(c, [&](auto, auto bwd) {
    return launch_rows<row_backward_kernel<decltype(bwd)>>(kRowBackwardMost, row_blocks(a.n_rows), row_bwd_lds_floats(a), c->stream, a);
  });
}

// dW, db of every layer of one or two small row-MLPs in one launch (and one reduction): x of layer 0 is
// [x1 | x2], of layer l > 0 act[l-1]. mean: what else the launch does (see MeanShareArgs). Rows are cut into chunks of kSmallWgradRows, fewer and larger ones
// where `partial` (partial_floats long) has no room for as many.
constexpr int kSmallWgradRows = 128;
struct SmallWgradMlp {
  const MlpRef *r;
  const float *x1, *x2;
  int w1, w2;
  float *const *act, *const *dz;
  int64_t n_rows;
};
inline int64_t small_wgrad_chunks(int64_t n_rows) {
  return std::min<int64_t>((n_rows + kSmallWgradRows - 1) / kSmallWgradRows, 64);
}
inline size_t small_wgrad_partial_floats(const MlpRef &r, int64_t n_rows) {
  size_t n = 0;
  for (int l = 0; l < r.n_layers; ++l) n += (size_t)(r.d_in[l] + 1) * r.d_out[l];
  const int64_t nc = small_wgrad_chunks(n_rows);
  return nc > 1 ? n * (size_t)nc : 0;
}
int launch_small_wgrads(xrl_ctx *c, const SmallWgradMlp *mlps, int n_mlps, float *dweights, float *partial, size_t partial_floats,
                        const MeanShareArgs *mean = nullptr) {
  SmallWgradArgs a;
  memset(&a, 0, sizeof(a));
  int blocks = 0, entries = 0;
  size_t used = 0;
  auto tiles = [](int n) { return (n + kWgradTile - 1) / kWgradTile; };
  // (as many chunks as give each compute unit the two blocks it has room for: 4624 rows, H = 256, in chunks of 128 31 us,
  // so 27 and a reduction of 5 in place of 7)
  int many = 0;
  for (int i = 0; i < n_mlps; ++i)
    for (int l = 0; l < mlps[i].r->n_layers && mlps[i].n_rows > kSmallWgradRows; ++l) many += tiles(mlps[i].r->d_in[l]) * tiles(mlps[i].r->d_out[l]);
  const int64_t most_chunks = std::max(1, 2 * c->n_cu / std::max(1, many));
  for (int i = 0; i < n_mlps; ++i) {
    const SmallWgradMlp &m = mlps[i];
    if (m.n_rows <= 0) continue;
    for (int l = 0; l < m.r->n_layers; ++l) {
      SmallWgradJob &j = a.job[a.n_jobs++];
      j.d_in = m.r->d_in[l]; j.d_out = m.r->d_out[l];
      j.x1 = l == 0 ? m.x1 : m.act[l - 1];
      j.w1 = l == 0 ? m.w1 : j.d_in;
      j.x2 = l == 0 ? m.x2 : nullptr;
      j.w2 = l == 0 ? m.w2 : 0;
      j.dz = m.dz[l];
      j.n_rows = m.n_rows;
      const size_t n = (size_t)(j.d_in + 1) * j.d_out;
      int64_t nc = std::min(small_wgrad_chunks(m.n_rows), most_chunks);
      if (partial && used + (size_t)nc * n > partial_floats) nc = (int64_t)((partial_floats - used) / n);
      if (!partial || nc < 2) nc = 1;
      j.rows_per_chunk = (int)((m.n_rows + nc - 1) / nc);
      j.n_chunks = (int)((m.n_rows + j.rows_per_chunk - 1) / j.rows_per_chunk);
      j.tiles_k = tiles(j.d_in);
      j.tiles_f = tiles(j.d_out);
      j.block0 = blocks;
      j.entry0 = entries;
      j.dW = dweights + m.r->w[l];
      j.db = dweights + m.r->b[l];
      blocks += j.tiles_k * j.tiles_f * j.n_chunks;
      if (j.n_chunks > 1) {
        j.partial = partial + used;
        used += (size_t)j.n_chunks * n;
        entries += (int)((n + 255) / 256);
      }
    }
  }
  if (blocks == 0) return XRL_OK;
  MeanShareArgs m = {};
  if (mean) m = *mean;
  m.block0 = blocks;
  blocks += (m.G + kMeanRows - 1) / kMeanRows;
  small_wgrad_kernel<<<dim3((unsigned)blocks), dim3(256), 0, c->stream>>>(a, m);
  if (entries > 0) small_wgrad_reduce_kernel<<<dim3((unsigned)entries), dim3(256), 0, c->stream>>>(a);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

// dh[n, :] = dx[graph(n), :H] (divided by the graph's node count for the mean readout), stored in
// the operand type like every later dh; one thread per four columns. node_graph null: one row per
// graph (n = the graph)
template <typename T>
__global__ void broadcast_dpool_kernel(const float *dx, int ldx, const int32_t *node_graph,
                                       const int32_t *graph_node_ptr, int mean, int64_t N, int H, T *dh) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int q = H / 4;
  if (i >= N * q) return;
  const int64_t n = i / q;
  const int f = (int)(i - n * q) * 4, gph = node_graph ? node_graph[n] : (int)n;
  float v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = dx[(size_t)gph * ldx + f + j];
  if (mean) {
    const int cnt = graph_node_ptr[gph + 1] - graph_node_ptr[gph];
    const float d = (float)(cnt > 1 ? cnt : 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] /= d;
  }
  store4<T>(dh + (size_t)n * H + f, v);
}

// The node-update layer's input rows written out for its weight gradient:
// X[n, :] = [sum over node n's in-edges (receiver order: the node-update kernel's order) of their
// attribute rows | one-hot operator type | dense attributes | zeros up to Kp columns]; one thread per
// node and eight columns.
template <typename T>
__global__ void embed_input_rows_kernel(const float *edge_feat, const int32_t *in_ptr, const int32_t *node_op,
                                        const float *node_dense, int64_t N, int De, int Tn, int Dd, int Kp, T *X) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int q = Kp / 8;
  if (i >= N * q) return;
  const int64_t n = i / q;
  const int k0 = (int)(i - n * q) * 8;
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = 0.f;
  if (k0 < De) {
    // (De is a multiple of 4 and k0 of 8: columns k0 .. k0+3 are attributes, k0+4 .. k0+7 all or none)
    const bool two = k0 + 8 <= De;
    const int e1 = in_ptr[n + 1];
    for (int e = in_ptr[n]; e < e1; ++e) {
      const float *p = edge_feat + (size_t)e * De + k0;
      const f32x4 lo = *(const f32x4 *)p;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] += lo[j];
      if (two) {
        const f32x4 hi = *(const f32x4 *)(p + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[4 + j] += hi[j];
      }
    }
  }
  const int op = node_op[n];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int k = k0 + j;
    if (k >= De && k < De + Tn) v[j] = k - De == op ? 1.f : 0.f;
    else if (k >= De + Tn && k < De + Tn + Dd) v[j] = node_dense[(size_t)n * Dd + (k - De - Tn)];
  }
  store4<T>(X + (size_t)n * Kp + k0, v);
  store4<T>(X + (size_t)n * Kp + k0 + 4, v + 4);
}

// ---- batches reduced to distinct nodes (distinct.hip.h)
LevelGraph batch_graph(const xrl_batch *b) {
  const xrl_batch_device &d = b->dev;
  LevelGraph g;
  g.N = b->N; g.E = b->E; g.n_tiles = b->n_tiles;
  g.in_ptr = d.in_ptr; g.in_src = d.in_src; g.in_dst = d.in_dst; g.out_ptr = d.out_ptr; g.out_pos = d.out_pos;
  g.tile_ptr = d.tile_ptr; g.agg_src = d.agg_src; g.node_op = d.node_op; g.edge_feat = d.edge_feat; g.node_dense = d.node_dense;
  return g;
}
Distinct *distinct_of(const xrl_ctx *c, const xrl_batch *b) {
  return b->owner == c->id ? b->distinct.get() : nullptr;   // (the owner's alone: it is made and used on its stream)
}

// Rows of a level's list [edges | classes | received]. fold: received rows are summed per class.
int64_t level_rows(const LevelGraph &g, bool fold) { return g.E + g.N + (fold ? g.N : g.E); }
// The groupings of a reduced batch that the backward pass goes by.
GroupArgs groupings(const xrl_batch *b, Distinct *q, bool fold) {
  GroupArgs a;
  memset(&a, 0, sizeof(a));
  int64_t item = 0, key = 0;
  auto add = [&](int64_t items, int64_t keys, const int32_t *k, const int32_t *val, int32_t *ptr, int32_t *seg, int32_t *out) {
    a.item0[a.n] = item; a.key0[a.n] = (uint32_t)key;
    a.key[a.n] = k; a.val[a.n] = val;
    a.ptr[a.n] = ptr; a.seg[a.n] = seg; a.out[a.n] = out;
    item += items; key += keys;
    ++a.n;
    a.item0[a.n] = item; a.key0[a.n] = (uint32_t)key;
  };
  const int R = q->levels - 1;
  for (int l = 1; l <= R; ++l) {
    LevelGraph &g = q->lv[l];
    a.n_edges[a.n] = g.E; a.n_cls[a.n] = g.N; a.src[a.n] = g.in_src; a.dst[a.n] = fold ? nullptr : g.in_dst; a.agg_src[a.n] = g.agg_src;
    add(level_rows(g, fold), q->lv[l - 1].N, g.self, nullptr, g.down_ptr, g.down_seg, g.down);
  }
  a.n_cls[a.n] = b->N;
  add(b->N, q->lv[R].N, q->cls[R], b->dev.node_graph, q->mem_ptr, q->mem_seg, q->mem_graph);
  return a;
}
// A stable sort of n (key, value) items, keys below n_keys: the memory it takes, and the sort, whose items `fill` puts into
// that memory. Returns where they lie then.
size_t sort_bytes_of(int64_t n) {
  const int64_t nb = (n + kSortItems - 1) / kSortItems;
  return 2 * align_up((size_t)n * 8) + align_up((size_t)nb * 256 * 4) + 1024;
}
template <typename Fill>
uint2 *sort_items(xrl_ctx *c, char *mem, int64_t n, uint32_t n_keys, Fill fill) {
  const int nb = (int)((n + kSortItems - 1) / kSortItems);
  Bump bump{mem};
  uint2 *x = bump.take<uint2>((size_t)n), *y = bump.take<uint2>((size_t)n);
  int32_t *hist = bump.take<int32_t>((size_t)nb * 256), *total = bump.take<int32_t>(256);
  fill(x);
  for (int shift = 0; shift < 32 && (n_keys - 1) >> shift; shift += 8) {
    sort_count_kernel<<<dim3((unsigned)nb), dim3(256), 0, c->stream>>>(x, n, shift, hist, nb);
    sort_scan_kernel<<<dim3(256), dim3(256), 0, c->stream>>>(hist, nb, total);
    sort_scatter_kernel<<<dim3((unsigned)nb), dim3(256), 0, c->stream>>>(x, n, shift, hist, nb, total, y);
    std::swap(x, y);
  }
  return x;
}
size_t grouping_bytes(const xrl_batch *b, Distinct *q, bool fold) {
  const GroupArgs a = groupings(b, q, fold);
  return sort_bytes_of(a.item0[a.n]);
}
int make_groupings(xrl_ctx *c, const xrl_batch *b, Distinct *q, bool fold) {
  const GroupArgs a = groupings(b, q, fold);
  const dim3 per_item((unsigned)((a.item0[a.n] + 255) / 256));
  const uint2 *x = sort_items(c, c->bws, a.item0[a.n], a.key0[a.n], [&](uint2 *items) {
    group_items_kernel<<<per_item, dim3(256), 0, c->stream>>>(a, items);
  });
  group_write_kernel<<<per_item, dim3(256), 0, c->stream>>>(a, x);
  HIP_TRY(hipGetLastError());
  // (while a stream is being captured nothing runs: eager calls make them for themselves)
  q->grouped_fold = fold;
  q->grouped = !is_capturing(c);
  return XRL_OK;
}

double encode_estimate_us(const xrl_ctx *c, const xrl_batch *b) {
  const double H = c->m.hidden, De = c->m.d_edge;
  return 2.0 * c->m.rounds * H * ((double)b->N * 3 * H + (double)b->E * (3 * H + De)) / (c->elem == 2 ? 7e8 : 7e7);   // (flops per us measured)
}
// Whether a batch's graphs look like rewrites of their state's first: half of the first 64 operators of a sample of
// graphs the same, place by place.
bool looks_like_rewrites(const xrl_ctx *c, const xrl_batch *b) {
  if (b->from_edits || c->distinct_min_us == 0) return true;
  const int32_t *sgp = b->at<int32_t>(b->o_state_graph_ptr), *gnp = b->at<int32_t>(b->o_graph_node_ptr), *op = b->at<int32_t>(b->o_node_op);
  const int64_t step = std::max<int64_t>(1, b->G / 64);
  int64_t same = 0, seen = 0, s = 0;
  for (int64_t g = 0; g < b->G; g += step) {
    while (sgp[s + 1] <= g) ++s;
    const int64_t f = sgp[s];
    if (g == f) continue;
    const int n = std::min(64, std::min(gnp[g + 1] - gnp[g], gnp[f + 1] - gnp[f]));
    for (int i = 0; i < n; ++i) same += op[gnp[g] + i] == op[gnp[f] + i];
    seen += 64;
  }
  return 2 * same >= seen;
}

// Whether a batch's levels are worth finding: its encode is estimated from the products' flops, and its
// graphs have to look like rewrites of their state's first (half of the first 64 operators of a sample of
// graphs the same, place by place). Finding the levels and the groupings takes 0.4 to 0.6 ms (70 k to
// 700 k nodes), two waits included. Measured, us per step without / with, by the estimate (update
// with a fresh minibatch, so that every step pays for it; 5 rounds, H = 128): 30 us 1008 / 1410, 108 us
// 1912 / 1721, 216 us 3115 / 3874, 430 us 5380 / 3779; fp32 200 us 2265 / 2587. A batch kept over
// the steps pays once: 430 us 622 / 337 forward only.
// A smaller batch, from a tenth of that estimate on (fp32: a quarter), pays over several encodes: it is reduced once as much has
// been spent for want of it (three times the estimate for a step that is differentiated, 0.8 for another) as it takes. But
// not one of less than kReduceNodes, up to two thirds of that estimate: its launches are a tile or less per compute unit, and
// few tiles take as long as that. Kept batches, us per step whole / reduced, residual networks' and transformers' states:
// update bf16 H = 128, 31 us 637 / 579, 46 us 718 / 584, 67 us 817 / 598; H = 64, 31 us 667 / 452, 67 us 1110 / 465; H = 256, 8.8 k nodes 51 us
// 1054 / 991, 82 us 1156 / 1006, 154 us 1373 / 1015 (but 7.1 k nodes 809 / 994); fp32 H = 64, 77 us 652 / 440; H = 128, 8.8 k nodes 128 us
// 831 / 599 (7.1 k 646 / 597); H = 256, 196 us 1531 / 1441 (119 us 1441 / 1439); forward only in the same order 213 / 189, 245 / 189, 259 / 192; 170 / 127,
// 232 / 137; 448 / 419, 464 / 429, 528 / 432 (418 / 431); 186 / 151; 256 / 225 (215 / 225); 623 / 630 (619 / 632). An inception-shaped state, 64 to 75 % of
// whose edges are left, least: bf16 H = 128, 26 us 608 / 613, 210 / 201; H = 256, 60 us 1087 / 1062, 452 / 439.
constexpr double kReduceUs = 450;
constexpr int64_t kReduceNodes = 8192;
bool distinct_pays(const xrl_ctx *c, xrl_batch *b, bool save) {
  const int R = c->m.rounds;
  if (c->distinct_min_us < 0 || c->captured || c->m.round_kind != XRL_ROUND_MLP || R < 1 || R + 1 > kMaxLevels || b->G <= b->S || b->N < 1 || b->E < 1 || b->n_split_tiles > 0 ||
      b->N + b->E > (int64_t)1 << kNodeBits)                // (table slots hold node numbers of so many bits)
    return false;
  const double us = encode_estimate_us(c, b), min_us = (double)c->distinct_min_us;
  if (us >= min_us) return (save || b->encodes > 0) && looks_like_rewrites(c, b);
  if (us < min_us / (c->elem == 2 ? 10 : 4) || (b->N < kReduceNodes && us < min_us * 2 / 3)) return false;
  if (b->forgone_us < kReduceUs) {
    b->forgone_us += us * (save ? 3.0 : 0.8);
    return false;
  }
  if (looks_like_rewrites(c, b)) return true;
  b->encodes = -1;                          // (not asked again)
  return false;
}

// Whether nodes that stand at the same place of a graph and of its state's first are alike in all that level 0 goes by: five
// of eight, of the first and last sixteen places of eight graphs as far as the operators are the same (a rewrite moves what is behind
// it; sixteen graphs and 32 places took 18 us of host time, these 3). Rewrites 0.76 to 0.97 (what is missing are nodes of three and more
// in-edges, listed in another order); noise on every edge's attributes 0.41 to 0.60, a dense attribute changed at every third node 0.29 to
// 0.48, at every tenth 0.63 to 0.79. Encodes of 91 k nodes, H = 256, us, whole / by levels, in this order: 519 / 324, 527 / 681, 531 / 688, 537 / 537.
bool attributes_alike(const xrl_ctx *c, const xrl_batch *b) {
  if (b->from_edits || c->distinct_min_us == 0) return true;
  const int32_t *sgp = b->at<int32_t>(b->o_state_graph_ptr), *gnp = b->at<int32_t>(b->o_graph_node_ptr), *op = b->at<int32_t>(b->o_node_op);
  const int32_t *in_ptr = b->at<int32_t>(b->o_in_ptr);
  const float *dense = b->at<float>(b->o_node_dense), *feat = b->at<float>(b->o_edge_feat);
  const size_t De = c->m.d_edge, Dd = c->m.n_node_dense;
  auto same_edges = [&](int64_t x, int64_t y, int64_t n) { return memcmp(feat + x * De, feat + y * De, n * De * sizeof(float)) == 0; };
  auto alike = [&](int64_t u, int64_t v) {
    const int64_t e = in_ptr[u], f = in_ptr[v], d = in_ptr[u + 1] - e;
    if (in_ptr[v + 1] - f != d || memcmp(dense + u * Dd, dense + v * Dd, Dd * sizeof(float)) != 0) return false;
    return same_edges(e, f, d) || (d >= 2 && same_edges(e, f + 1, 1) && same_edges(e + 1, f, 1) && same_edges(e + 2, f + 2, d - 2));
  };
  constexpr int kGraphs = 8, kPlaces = 16;
  int64_t same = 0, seen = 0, s = 0;
  for (int k = 0; k < kGraphs; ++k) {
    int64_t g = k * b->G / kGraphs;
    while (sgp[s + 1] <= g) ++s;
    const int64_t f = sgp[s];
    if (g == f && ++g == sgp[s + 1]) continue;
    const int n = std::min(kPlaces, std::min(gnp[g + 1] - gnp[g], gnp[f + 1] - gnp[f]));
    auto walk = [&](int64_t u, int64_t v, int step) {
      for (int i = 0; i < n && op[u] == op[v]; ++i, u += step, v += step) { ++seen; same += alike(u, v); }
    };
    if (n > 0) { walk(gnp[g], gnp[f], 1); walk(gnp[g + 1] - 1, gnp[f + 1] - 1, -1); }
  }
  return seen > 0 && 8 * same >= 5 * seen;
}

// The same for one forward-only encode (see OnceArgs): no wait and nothing kept, so it pays for the classes alone. There is no way
// out once it has begun, so a batch known to have too many distinct nodes is left whole, and the sample goes by the attributes too.
// us of an encode as it is / by levels, H = 256, by the estimate: one inception-shaped state 110 us 210 / 337, 217 289 / 368,
// 417 444 / 454, 828 736 / 563; a transformer-shaped one 216 288 / 289, 429 439 / 309, 715 632 / 332; states of residual networks
// 505 508 / 353, 2008 1800 / 587. At H <= 128 a round costs a third of that and finding its level as much; in fp32 the
// kernels of a round take their sizes from the host.
constexpr int kOnceMinUs = 430;
bool once_pays(const xrl_ctx *c, const xrl_batch *b) {
  const xrl_model_desc &m = c->m;
  if (c->elem != 2 || m.hidden != 256 || c->distinct_min_us < 0 || c->captured || m.round_kind != XRL_ROUND_MLP || m.rounds < 1 ||
      m.rounds + 1 > kMaxLevels || b->G <= b->S || b->n_split_tiles > 0 || b->E < 1 || std::max(b->N, b->E) > kOnceMax || b->few_alike)
    return false;
  Mlp2Args t;
  memset(&t, 0, sizeof(t));
  t.De = m.d_edge; t.Tn = m.n_op_types; t.Dd = m.n_node_dense; t.n_rows = std::min(b->N, b->E);
  t.nslabx = c->embed.nslabx;
  if (!mlp2p_applies(c, KIND_EMBED, t)) return false;
  for (int r = 0; r < m.rounds; ++r) {
    t.nslab1 = c->edge[r].nslab1;
    if (!mlp2r_applies(c, KIND_EDGE, t)) return false;
  }
  return (c->distinct_min_us == 0 || encode_estimate_us(c, b) >= (double)std::max<int64_t>(kOnceMinUs, c->distinct_min_us)) && looks_like_rewrites(c, b) && attributes_alike(c, b);
}
struct OnceLevels {
  OnceArgs o;
  int32_t *cls[2];
  unsigned long long *counts;              // [levels]
  unsigned blocks_per_graph;
  const int32_t *classes(int l) const { return cls[l & 1]; }
};
// Lays the levels' memory out at base and returns its size.
size_t once_plan(const xrl_ctx *c, const xrl_batch *b, char *base, OnceLevels &q) {
  const int64_t N = b->N, E = b->E;
  const int De = c->m.d_edge, Dd = c->m.n_node_dense;
  memset(&q, 0, sizeof(q));
  uint32_t slots = 1024;
  while (slots < (uint64_t)N + N / 2) slots *= 2;
  const int64_t max_tiles = 2 * E / 33 + 2 * ((N + kOnceNodes - 1) / kOnceNodes) + 2;
  Bump m{base};
  ClassArgs &a = q.o.k;
  a.mask = slots - 1;
  a.table = m.take<unsigned long long>(slots);
  q.counts = m.take<unsigned long long>(kMaxLevels);
  q.o.num = m.take<int32_t>(slots);
  a.swapped = m.take<uint8_t>((size_t)N);
  a.slot = m.take<int32_t>((size_t)N);
  for (int i = 0; i < 2; ++i) q.cls[i] = m.take<int32_t>((size_t)N);
  q.o.o_ptr = m.take<int32_t>((size_t)N + 1);
  q.o.o_agg_src = m.take<int32_t>((size_t)N);
  q.o.o_self = m.take<int32_t>((size_t)N);
  q.o.o_op = m.take<int32_t>((size_t)N);
  q.o.o_src = m.take<int32_t>((size_t)E);
  q.o.o_dst = m.take<int32_t>((size_t)E);
  q.o.o_hrow = m.take<int32_t>((size_t)E);
  q.o.o_tile = m.take<int32_t>((size_t)max_tiles);
  q.o.o_feat = m.take<float>((size_t)E * De);
  q.o.o_dense = m.take<float>((size_t)N * Dd);
  return m.off;
}
int once_begin(xrl_ctx *c, const xrl_batch *b, OnceLevels &q) {
  const int64_t N = b->N;
  const xrl_batch_device &d = b->dev;
  ClassArgs &a = q.o.k;
  a.N = N; a.in_ptr = d.in_ptr; a.in_src = d.in_src; a.node_op = d.node_op;
  a.edge_feat = (const uint32_t *)d.edge_feat; a.node_dense = (const uint32_t *)d.node_dense; a.De = c->m.d_edge; a.Dd = c->m.n_node_dense;
  a.state_graph_ptr = d.state_graph_ptr; a.graph_node_ptr = d.graph_node_ptr;
  q.blocks_per_graph = (unsigned)std::max<int64_t>(1, (b->max_graph_nodes + 255) / 256);
  once_clear_kernel<<<dim3(a.mask / 256 + 1), dim3(256), 0, c->stream>>>(a.table, a.mask + 1, q.counts);
  first_two_kernel<<<dim3((unsigned)((N + 255) / 256)), dim3(256), 0, c->stream>>>(a, (uint8_t *)a.swapped);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}
// the classes and the graph of level l; `a`: as the kernels of the round take it
int once_level(xrl_ctx *c, const xrl_batch *b, OnceLevels &q, int l, Mlp2Args &a) {
  const dim3 per_node((unsigned)((b->N + 255) / 256)), b256(256);
  q.o.k.prev = l > 0 ? q.cls[(l - 1) & 1] : nullptr;
  q.o.k.cls = q.cls[l & 1];
  q.o.counts = q.counts + l;
  once_insert_first_kernel<<<dim3((unsigned)b->S * q.blocks_per_graph), b256, 0, c->stream>>>(q.o.k, (int)q.blocks_per_graph);
  once_insert_kernel<<<per_node, b256, 0, c->stream>>>(q.o.k);
  once_fill_kernel<<<dim3((unsigned)((b->N + kOnceNodes - 1) / kOnceNodes)), b256, 0, c->stream>>>(q.o);
  once_class_kernel<<<per_node, b256, 0, c->stream>>>(q.o.k, q.o.num);
  HIP_TRY(hipGetLastError());
  a.level_counts = q.o.counts;
  a.in_ptr = q.o.o_ptr; a.in_src = q.o.o_src; a.in_dst = q.o.o_dst; a.agg_src = q.o.o_agg_src; a.edge_feat = q.o.o_feat;
  a.node_op = q.o.o_op; a.node_dense = q.o.o_dense; a.tile_ptr = q.o.o_tile;
  a.n_tiles = b->n_tiles;                  // (of the whole batch: the grid)
  return XRL_OK;
}

// Finds the levels' classes, reads back how many there are, and, if that is few enough, makes the levels'
// graphs. Two waits for the stream (the counts of classes, then of tiles).
int find_distinct(xrl_ctx *c, xrl_batch *b) {
  RelaxedCapture relaxed;               // (an encode that neither allocated nor waited before must not end another stream's capture)
  const int R = c->m.rounds, L = R + 1, De = c->m.d_edge, Dd = c->m.n_node_dense;
  const int64_t N = b->N, E = b->E;
  const xrl_batch_device &d = b->dev;
  uint32_t slots = 1024;
  while (slots < (uint64_t)N + N / 2) slots *= 2;
  const int nb = (int)((N + kScanItems - 1) / kScanItems);
  auto q = std::make_shared<Distinct>();
  q->levels = L;
  auto take = [&](int i, size_t bytes) -> char * {
    if (c->blocks->take(bytes, true, &q->block[i]) == hipSuccess) return (char *)q->block[i].p;
    q->block[i] = DeviceBlock();
    return nullptr;
  };
  auto drop = [&]() {
    for (DeviceBlock &x : q->block) c->blocks->give(x);
  };
  const size_t n_bytes = align_up((size_t)N * 4);
  char *cls_block = take(0, n_bytes * L);
  if (!cls_block) return XRL_OK;                            // (no memory for it: the batch is used as it is)
  const size_t scratch = align_up((size_t)slots * 8) + 2 * n_bytes + align_up((size_t)nb * 8) +
                         (n_bytes + align_up((size_t)(N + 1) * 4)) * L + align_up((size_t)N);
  int rc = ensure_bws(c, scratch);
  if (rc) { drop(); return rc == XRL_ERR_OOM ? XRL_OK : rc; }
  Bump bump{c->bws};
  ClassArgs a;
  memset(&a, 0, sizeof(a));
  a.N = N; a.in_ptr = d.in_ptr; a.in_src = d.in_src; a.node_op = d.node_op;
  a.edge_feat = (const uint32_t *)d.edge_feat; a.node_dense = (const uint32_t *)d.node_dense; a.De = De; a.Dd = Dd;
  a.table = bump.take<unsigned long long>(slots); a.mask = slots - 1;
  a.state_graph_ptr = d.state_graph_ptr; a.graph_node_ptr = d.graph_node_ptr;
  a.slot = bump.take<int32_t>((size_t)N); a.rep = bump.take<int32_t>((size_t)N); a.block_sum = bump.take<int2>((size_t)nb);
  uint8_t *swapped = bump.take<uint8_t>((size_t)N);
  a.swapped = swapped;
  std::vector<int32_t *> reps(L), ptr(L);
  const dim3 per_node((unsigned)((N + 255) / 256)), per_block((unsigned)nb), b256(256);
  first_two_kernel<<<per_node, b256, 0, c->stream>>>(a, swapped);
  for (int l = 0; l < L; ++l) {
    a.prev = l > 0 ? q->cls[l - 1] : nullptr;
    a.cls = q->cls[l] = (int32_t *)(cls_block + n_bytes * l);
    a.reps = reps[l] = bump.take<int32_t>((size_t)N);
    a.ptr = ptr[l] = bump.take<int32_t>((size_t)N + 1);
    a.totals = c->d_counts + 2 * l;
    a.receivers = c->d_counts + 2 * kMaxLevels + l;
    class_clear_kernel<<<dim3((slots + 255) / 256), b256, 0, c->stream>>>(a.table, slots);
    class_insert_first_kernel<<<dim3((unsigned)b->S), b256, 0, c->stream>>>(a);
    class_insert_kernel<<<per_node, b256, 0, c->stream>>>(a);
    class_verify_kernel<<<per_block, b256, 0, c->stream>>>(a);
    class_scan_kernel<<<dim3(1), b256, 0, c->stream>>>(a, nb);
    class_number_kernel<<<per_block, b256, 0, c->stream>>>(a);
    class_of_kernel<<<per_node, b256, 0, c->stream>>>(a);
  }
  auto read_counts = [&](int n) -> int {
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(c->h_counts, c->d_counts, sizeof(int32_t) * n, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return XRL_OK;
  };
  if ((rc = read_counts(2 * L))) { drop(); return rc; }
  int64_t sumE = 0, sumN = 0, items = N;
  for (int l = 0; l < L; ++l) {
    q->lv[l].N = c->h_counts[2 * l];
    q->lv[l].E = c->h_counts[2 * l + 1];
    if (l > 0) {
      sumE += q->lv[l].E; sumN += q->lv[l].N;
      items += std::max(level_rows(q->lv[l], false), level_rows(q->lv[l], true));
    }
  }
  // (the sort that makes the groupings counts the items of all levels in 32 bits)
  if (items > INT32_MAX - kSortItems) { drop(); return XRL_OK; }
  // (a level costs a copy of its states more, so a quarter of the edges has to go)
  if (4 * (sumE + sumN) > 3 * R * (E + N) && c->distinct_min_us != 0) {
    b->few_alike = true;
    drop();
    return XRL_OK;
  }
  // ---- the levels' graphs
  size_t off = 0;
  auto plan = [&](size_t bytes) { const size_t o = off; off += align_up(bytes + 16); return o; };
  struct Off { size_t ptr, src, dst, agg, self, op, dense, feat, tile, dptr, down, dseg, bsrc, bdst; } o[kMaxLevels];
  TileLevels tl;
  memset(&tl, 0, sizeof(tl));
  tl.n_levels = R;
  int chunks = 0;
  for (int l = 0; l < L; ++l) {
    const int64_t n = q->lv[l].N, e = q->lv[l].E;
    o[l].ptr = plan((n + 1) * 4);
    o[l].agg = plan(n * 4);
    o[l].feat = plan((size_t)e * De * 4);
    if (l == 0) {
      o[l].op = plan(n * 4);
      o[l].dense = plan((size_t)n * Dd * 4);
      continue;
    }
    const int nc = (int)((e + kTileChunk - 1) / kTileChunk);
    tl.chunk0[l - 1] = chunks;
    tl.n_edges[l - 1] = (int32_t)e;
    chunks += nc;
    tl.chunk0[l] = chunks;
    o[l].src = plan(e * 4); o[l].dst = plan(e * 4); o[l].self = plan(n * 4);
    if (c->elem == 4) { o[l].bsrc = plan(e * 4); o[l].bdst = plan(e * 4); }
    o[l].tile = plan((e / 16 + 2 * nc + 4) * 4);
    o[l].dptr = plan((q->lv[l - 1].N + 1) * 4); o[l].down = plan((e + n + std::max(e, n) + kSumRows) * 4); o[l].dseg = plan((e + n + std::max(e, n) + kSumRows) * 4);   // (level_rows)
  }
  const size_t o_mptr = plan((q->lv[R].N + 1) * 4), o_mgraph = plan((N + kSumRows) * 4), o_mseg = plan((N + kSumRows) * 4);
  const size_t o_cuts = plan((size_t)chunks * kTileChunkMax * 4), o_count = plan((size_t)(chunks + 1) * 4);
  char *blk = take(1, off);
  if (!blk) { drop(); return XRL_OK; }
  for (int l = 0; l < L; ++l) {
    LevelGraph &g = q->lv[l];
    LevelFillArgs f;
    memset(&f, 0, sizeof(f));
    auto at = [&](size_t x) { return (int32_t *)(blk + x); };
    f.n_cls = g.N; f.reps = reps[l]; f.ptr = ptr[l]; f.cls = q->cls[l]; f.prev = l > 0 ? q->cls[l - 1] : nullptr;
    f.in_ptr = d.in_ptr; f.in_src = d.in_src; f.node_op = d.node_op; f.edge_feat = d.edge_feat; f.node_dense = d.node_dense;
    f.De = De; f.Dd = Dd; f.receivers = c->d_counts + 2 * kMaxLevels + l;
    f.o_ptr = at(o[l].ptr); f.o_agg_src = at(o[l].agg); f.o_feat = (float *)(blk + o[l].feat);
    if (l == 0) { f.o_op = at(o[l].op); f.o_dense = (float *)(blk + o[l].dense); }
    else { f.o_src = at(o[l].src); f.o_dst = at(o[l].dst); f.o_self = at(o[l].self); }
    if (l > 0 && c->elem == 4) { g.below_src = f.o_below_src = at(o[l].bsrc); g.below_dst = f.o_below_dst = at(o[l].bdst); }
    level_fill_kernel<<<dim3((unsigned)((g.N + 255) / 256)), b256, 0, c->stream>>>(f);
    g.in_ptr = f.o_ptr; g.in_src = f.o_src; g.in_dst = f.o_dst; g.agg_src = f.o_agg_src; g.edge_feat = f.o_feat;
    g.node_op = f.o_op; g.node_dense = f.o_dense; g.self = f.o_self;
    if (l == 0) continue;
    g.down_ptr = at(o[l].dptr); g.down = at(o[l].down); g.down_seg = at(o[l].dseg);
    g.tile_ptr = at(o[l].tile);
    tl.ptr[l - 1] = g.in_ptr; tl.dst[l - 1] = g.in_dst; tl.tile_ptr[l - 1] = at(o[l].tile);
  }
  q->mem_ptr = (int32_t *)(blk + o_mptr); q->mem_graph = (int32_t *)(blk + o_mgraph); q->mem_seg = (int32_t *)(blk + o_mseg);
  tl.cuts = (int32_t *)(blk + o_cuts); tl.count = (int32_t *)(blk + o_count); tl.totals = c->d_counts;
  tile_cut_kernel<<<dim3((unsigned)chunks), b256, 0, c->stream>>>(tl);
  tile_scan_kernel<<<dim3((unsigned)R), b256, 0, c->stream>>>(tl);
  tile_write_kernel<<<dim3((unsigned)chunks), b256, 0, c->stream>>>(tl);
  if ((rc = read_counts(kCounts))) { drop(); return rc; }
  for (int l = 0; l < L; ++l) {
    if (l > 0) q->lv[l].n_tiles = c->h_counts[l - 1];
    q->lv[l].receivers = c->h_counts[2 * kMaxLevels + l];
  }
  b->distinct = q;
  return XRL_OK;
}

// The sender index of a batch: out_ptr, and the receiver-order positions of the edges grouped by sender, ascending.
// A block per graph: a counting sort of the graph's edges in which each of four waves takes a quarter of them,
// counted per wave and node in LDS. Where a graph has more nodes than that holds, the batch's edges are sorted by sender as
// one list: with one block and its counters in memory a graph of 200 k nodes and 400 k edges took 5.6 ms, so 0.09.
constexpr int kOutLdsNodes = 8192;
__global__ __launch_bounds__(256) void out_index_kernel(const int32_t *graph_node_ptr, const int32_t *in_ptr, const int32_t *in_src,
                                                        int32_t *out_ptr, int32_t *out_pos) {
  extern __shared__ __align__(16) int32_t out_cnt[];
  __shared__ int2 ws[4];
  const int g = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int base = graph_node_ptr[g], n = graph_node_ptr[g + 1] - base;
  if (n == 0) {
    if (g == (int)gridDim.x - 1 && t == 0) out_ptr[base] = in_ptr[base];
    return;
  }
  const int a = in_ptr[base], z = in_ptr[base + n];
  volatile int32_t *cnt = out_cnt;                                     // [4][n]
  for (int i = t; i < 4 * n; i += 256) cnt[i] = 0;
  __syncthreads();
  const int quarter = ((z - a + 3) / 4 + 63) / 64 * 64, e0 = a + w * quarter, e1 = e0 + quarter < z ? e0 + quarter : z;
  for (int e = e0 + lane; e < e1; e += 64) atomicAdd((int32_t *)&cnt[w * n + in_src[e] - base], 1);
  __threadfence_block();
  __syncthreads();
  int next = a;
  for (int i0 = 0; i0 < n; i0 += 256) {
    const int i = i0 + t;
    int c[4] = {0, 0, 0, 0};
    if (i < n)
      for (int k = 0; k < 4; ++k) c[k] = cnt[k * n + i];
    int2 sum;
    int at = next + block_scan_pair(make_int2(c[0] + c[1] + c[2] + c[3], 0), ws, sum).x;
    if (i < n) {
      out_ptr[base + i] = at;
      for (int k = 0; k < 4; ++k) {          // node i's first place for each wave
        cnt[k * n + i] = at;
        at += c[k];
      }
    }
    next += sum.x;
  }
  if (g == (int)gridDim.x - 1 && t == 0) out_ptr[base + n] = z;
  __threadfence_block();
  __syncthreads();
  const int bits = 32 - __builtin_clz(n);
  volatile int32_t *mine = cnt + w * n;
  for (int e = e0; e < e1; e += 64) {
    const bool in = e + lane < e1;
    const int s = in ? in_src[e + lane] - base : 0;
    unsigned long long same = __ballot(in);
    for (int b = 0; b < bits; ++b) {
      const unsigned long long m = __ballot((s >> b) & 1);
      same &= (s >> b) & 1 ? m : ~m;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1)), place = mine[s] + rank;
    __builtin_amdgcn_wave_barrier();
    if (in && rank == 0) mine[s] = place + __popcll(same);
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
    if (in) out_pos[place] = e + lane;
  }
}
__global__ __launch_bounds__(256) void out_items_kernel(const int32_t *in_src, int64_t E, uint2 *items) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < E) items[e] = make_uint2((uint32_t)in_src[e], (uint32_t)e);
}
// From the sorted items: the position of each, and each sender's first, by search (a sender may have none).
__global__ __launch_bounds__(256) void out_write_kernel(const uint2 *items, int64_t E, int64_t N, int32_t *out_ptr, int32_t *out_pos) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < E) out_pos[i] = (int32_t)items[i].y;
  if (i > N) return;
  int64_t lo = 0, hi = E;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (items[mid].x < (uint32_t)i) lo = mid + 1;
    else hi = mid;
  }
  out_ptr[i] = (int32_t)lo;
}
size_t out_index_bytes(const xrl_batch *b) { return b->max_graph_nodes > kOutLdsNodes ? sort_bytes_of(b->E) : 0; }
// Makes the batch's sender index on the context's stream unless it is there. Whichever context first needs it makes it; the others
// wait for that (the block's event marks the end of it). A graph makes it in every replay unless it was there
// before: the same values. scratch: out_index_bytes.
int make_out_index(xrl_ctx *c, const xrl_batch *cb, char *scratch) {
  xrl_batch *b = const_cast<xrl_batch *>(cb);
  if (b->G == 0) return XRL_OK;
  std::lock_guard<std::mutex> lk(b->out_mu);
  xrl_batch_device &d = b->dev;
  if (b->out_maker) {
    if (b->out_maker == c->id) return XRL_OK;
    RelaxedCapture relaxed;              // (this stream or another may be under capture: the wait is no part of it)
    HIP_TRY(hipEventSynchronize((hipEvent_t)d.used));
    return XRL_OK;
  }
  if (b->max_graph_nodes <= kOutLdsNodes) {
    static bool attr_set = false;
    if (!attr_set) {
      HIP_TRY(hipFuncSetAttribute((const void *)out_index_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 16 * kOutLdsNodes));
      attr_set = true;
    }
    out_index_kernel<<<dim3((unsigned)b->G), dim3(256), (size_t)16 * std::max(b->max_graph_nodes, 1), c->stream>>>(
        d.graph_node_ptr, d.in_ptr, d.in_src, d.out_ptr, d.out_pos);
  } else {
    const dim3 per_edge((unsigned)((b->E + 255) / 256)), per_item((unsigned)((std::max(b->E, b->N + 1) + 255) / 256));
    const uint2 *x = nullptr;
    if (b->E > 0)
      x = sort_items(c, scratch, b->E, (uint32_t)b->N, [&](uint2 *items) {
        out_items_kernel<<<per_edge, dim3(256), 0, c->stream>>>(d.in_src, b->E, items);
      });
    out_write_kernel<<<per_item, dim3(256), 0, c->stream>>>(x, b->E, b->N, d.out_ptr, d.out_pos);
  }
  HIP_TRY(hipGetLastError());
  if (is_capturing(c)) return XRL_OK;
  RelaxedCapture relaxed;
  hipEvent_t made = (hipEvent_t)d.used;
  if (made || went_well(hipEventCreateWithFlags(&made, hipEventDisableTiming))) {
    d.used = made;
    if (went_well(hipEventRecord(made, c->stream))) b->out_maker = c->id;
  }
  return XRL_OK;
}

template <typename T>
int encode_backward_impl(xrl_ctx *c, const xrl_batch *b, const float *d_demb, float *dweights) {
  const xrl_model_desc &m = c->m;
  const int H = m.hidden, R = m.rounds, De = m.d_edge, Dg = m.d_global;
  const int64_t N = b->N, E = b->E, G = b->G;
  const xrl_batch_device &d = b->dev;
  Distinct *q = distinct_of(c, b);
  const LevelGraph whole = batch_graph(b);
  auto lev = [&](int l) -> const LevelGraph & { return q ? q->lv[l] : whole; };
  int64_t maxN = 0, maxE = 0;
  for (int l = 0; l <= R; ++l) { maxN = std::max(maxN, lev(l).N); maxE = std::max(maxE, lev(l).E); }
  const int64_t M = std::max(maxN, maxE), N0 = lev(0).N;
  // ---- scratch plan
  size_t need = 0;
  auto acc = [&](size_t bytes) { need += align_up(bytes); };
  const bool gat = m.round_kind == XRL_ROUND_GAT;
  const bool kept = c->fwd_kept;                                   // the forward kept z1 and the ReLU masks
  // the per-edge gradients w.r.t. h_receiver leave the edge kernel already summed per receiver
  // (edge tiles end at receiver boundaries unless a receiver has more than 32 in-edges)
  const bool fold = kept && b->n_split_tiles == 0;
  const bool embed_kept = c->embed_kept, recompute = gat ? !embed_kept : !kept;
  // What the weight gradients of an MLP read -- dz1, dz2 and, where the forward kept none, z1 [rows, H] -- stays
  // until their launch, which takes as many MLPs as there is room for: all of them up to kGradRoom, else
  // the largest at least. (2 GiB: 12.5 ms step of 4.3 M nodes, H = 256, three launches; one launch of all would gain 2 x 30 us.)
  auto unit_bytes = [&](int64_t rows, int n) { return n * align_up((size_t)rows * H * sizeof(T)); };
  const int per_mlp = recompute ? 3 : 2;
  size_t room_all = unit_bytes(N0, per_mlp), room_one = room_all;
  for (int r = 1; r <= R; ++r)
    for (int64_t rows : {lev(r).N, gat ? 0 : lev(r).E}) {
      const size_t bytes = unit_bytes(rows, gat ? 1 : per_mlp);
      room_all += bytes;
      room_one = std::max(room_one, bytes);
    }
  if (gat) acc((size_t)maxN * H * sizeof(T));                      // dpre
  // per-edge d h_sender; d h_receiver: per edge, or summed per receiver (a reduced batch: d h_sender, the
  // classes' own dh and d h_receiver one behind the other, see GroupArgs)
  int64_t max_rows = 0;
  for (int l = 1; q && l <= R; ++l) max_rows = std::max(max_rows, level_rows(lev(l), fold));
  acc((size_t)(q ? max_rows : maxE) * H * sizeof(T));
  if (!q) acc((size_t)M * H * sizeof(T));
  for (int i = 0; i < 3; ++i) acc((size_t)maxN * H * sizeof(T));   // dh (two buffers), dagg
  // the node-update layer's input rows are written out for its weight gradient, Kp columns
  const int Kx = De + m.n_op_types + m.n_node_dense, Kp = (Kx + 7) / 8 * 8;
  acc((size_t)N0 * Kp * sizeof(T));
  const size_t part = std::max(wgrad_partial_floats(c), small_wgrad_partial_floats(c->L.readout, G));
  acc(part * 4);
  for (int i = 0; i < 3; ++i) acc((size_t)G * H * 4);
  if (gat) {                                                       // softmax weights and score gradients
    for (int i = 0; i < 2; ++i) acc((size_t)maxE * 4);
    for (int i = 0; i < 4; ++i) acc((size_t)maxN * 4);
    for (int r = 0; r < R; ++r) acc((size_t)kAvecChunks * 2 * H * 4);   // chunk sums of the attention vectors' gradients
  }
  if (!q) acc(out_index_bytes(b));
  // a reduced batch: the pieces of sums per class, the pool's gradient per graph; and, the first
  // time, the sort that makes the groupings these sums go by (in the same place)
  size_t sort_bytes = 0;
  const size_t o_reduced = need;
  const bool pool_windows = q && H == kPoolWidth && N >= c->pool_window_nodes * c->n_cu;      // (see pool_class_sum_kernel)
  const size_t pool_rows = (size_t)(pool_windows ? kWindows : 1) * G * H;
  if (q) {
    acc((size_t)((std::max(N, max_rows) + kSumRows - 1) / kSumRows) * 2 * H * 4);
    acc(pool_rows * 4);
    sort_bytes = q->grouped && q->grouped_fold == fold ? 0 : grouping_bytes(b, q, fold);
    need = std::max(need, sort_bytes);
  }
  const size_t o_room = align_up(need);
  size_t room = 0;
  int rc = fit_room(c->bws_bytes, o_room, room_one, std::min(room_all, std::max(room_one, c->grad_room)), c->captured, XRL_ERR_OOM,
                    &c->room_refused, &room, [&](size_t bytes) { return ensure_bws(c, bytes); });
  if (rc) return rc;
  if (q && !(q->grouped && q->grouped_fold == fold) && (rc = make_groupings(c, b, q, fold))) return rc;
  Bump bump{c->bws};
  T *dpre = gat ? bump.take<T>((size_t)maxN * H) : nullptr;
  T *dsrc = bump.take<T>((size_t)(q ? max_rows : maxE) * H), *ddst = q ? nullptr : bump.take<T>((size_t)M * H);
  T *dhA = bump.take<T>((size_t)maxN * H), *dhB = bump.take<T>((size_t)maxN * H);
  T *dagg = bump.take<T>((size_t)maxN * H);
  T *xrows = bump.take<T>((size_t)N0 * Kp);
  float *partial = bump.take<float>(part);
  float *rdz[3] = {bump.take<float>((size_t)G * H), bump.take<float>((size_t)G * H), nullptr};
  float *rdx = bump.take<float>((size_t)G * H);
  float *g_avec = nullptr, *g_ale = nullptr, *g_due = nullptr, *g_als = nullptr, *g_dus = nullptr, *g_dss = nullptr, *g_dsd = nullptr;
  if (gat) {
    g_ale = bump.take<float>((size_t)maxE); g_due = bump.take<float>((size_t)maxE);
    g_als = bump.take<float>((size_t)maxN); g_dus = bump.take<float>((size_t)maxN);
    g_dss = bump.take<float>((size_t)maxN); g_dsd = bump.take<float>((size_t)maxN);
    g_avec = bump.take<float>((size_t)R * kAvecChunks * 2 * H);
  }
  if (!q) {
    const size_t n = out_index_bytes(b);
    char *scratch = bump.take<char>(n);
    if ((rc = make_out_index(c, b, scratch))) return rc;
  }
  bump.off = o_reduced;
  float *ccarry = q ? bump.take<float>((size_t)((std::max(N, max_rows) + kSumRows - 1) / kSumRows) * 2 * H) : nullptr;
  float *dpool_rows = q ? bump.take<float>(pool_rows) : nullptr;
  WgradQueue wq;
  wq.partial = partial; wq.partial_floats = part;
  char *const room_base = c->bws + o_room;
  size_t room_used = 0;
  // memory for an MLP's gradients; what waits is launched first when there is none left (every one given out
  // so far is complete then: the next is asked for behind the kernels that fill the last)
  struct MlpGrads { T *z1 = nullptr, *dz1 = nullptr, *dz2 = nullptr; };
  auto next_grads = [&](int64_t rows, MlpGrads *m, int n) -> int {
    const size_t one = unit_bytes(rows, 1);
    if (room_used + n * one > room) {
      if (int rc2 = flush_wgrads<T>(c, wq)) return rc2;
      room_used = 0;
    }
    T *p = (T *)(room_base + room_used);
    room_used += n * one;
    m->dz1 = p;
    m->dz2 = n > 1 ? (T *)((char *)p + one) : nullptr;
    m->z1 = n > 2 ? (T *)((char *)p + 2 * one) : nullptr;
    return XRL_OK;
  };
  constexpr int PV = 16 / sizeof(T);
  // the gradients of the rows `vals`, summed per class (fp32) and stored: masked, as the dz2 of the layer
  // that produced the classes' states, or as their dh
  auto contract = [&](auto tag, const void *vals, const int32_t *perm, const int32_t *ptr, const int32_t *seg, int64_t rows,
                      const uint16_t *ymask, T *out, size_t table_bytes) -> int {
    using TIn = decltype(tag);
    constexpr int VEC = 16 / sizeof(TIn);
    ClassSumArgs s;
    s.vals = vals; s.zero_row = c->zero_row; s.perm = perm; s.seg = seg; s.ptr = ptr; s.n_rows = rows; s.D = H;
    s.ymask = ymask; s.out = out; s.carry = ccarry;
    const int64_t blocks = ((rows + kSumRows - 1) / kSumRows * (H / VEC) + 255) / 256;   // of one step a group
    s.slices = table_bytes >= kSliceBytes && H / VEC >= 64 ? 8 : 1;
    auto go = [&](auto steps) {
      constexpr int STEPS = decltype(steps)::value;
      s.group = STEPS * kSumRows;
      const int64_t groups = (rows + s.group - 1) / s.group;
      class_sum_kernel<TIn, T, VEC, STEPS><<<dim3((unsigned)((groups * (H / VEC / s.slices) + 255) / 256 * s.slices)), dim3(256), 0, c->stream>>>(s);
      class_sum_carried_kernel<T><<<dim3((unsigned)((groups + 4 * kCarryGroups - 1) / (4 * kCarryGroups))), dim3(256), 0, c->stream>>>(s);
    };
    // (the classes in several pieces, and their way to memory and back, against lanes to hide the gathers with: see class_sum_kernel)
    const int steps = c->sum_steps > 0 ? c->sum_steps : blocks >= 16 * c->n_cu ? 4 : blocks >= 3 * c->n_cu ? 2 : 1;
    if (steps >= 4) go(std::integral_constant<int, 4>());
    else if (steps >= 2) go(std::integral_constant<int, 2>());
    else go(std::integral_constant<int, 1>());
    HIP_TRY(hipGetLastError());
    return XRL_OK;
  };

  MlpGrads node_grads, edge_grads;         // of the MLP at hand; node_grads: then of the node-side layer below
  if (!gat && (rc = next_grads(R > 0 ? lev(R).N : N0, &node_grads, per_mlp))) return rc;
  // ---- global-update layer backward
  float *ract[3] = {c->ro_act[0], c->ro_act[1], nullptr};
  if ((rc = launch_readout_backward(c, row_bwd_args(c, c->L.readout, true, ract, d_demb, G, rdz, rdx)))) return rc;
  const SmallWgradMlp readout = {&c->L.readout, c->pool, d.graph_global, H, Dg, ract, rdz, G};
  if ((rc = launch_small_wgrads(c, &readout, 1, dweights, partial, part))) return rc;
  // The gradient w.r.t. the last node states is the pool's, the same row for every node of a graph.
  // From the kept forward, the first backward kernel reads it through the nodes' graph ids from a
  // [G, H] table (the kernel below with the graphs as its "nodes"); otherwise it is written out per node.
  const bool dpool_table = kept && !gat && !q;
  bool dz2_given = false;                  // dz2 of the next node-side layer down is in place already
  if (q) {
    // (a reduced batch: summed over each class's nodes of all graphs)
    const uint16_t *mask = kept ? c->ym_node[R - 1] : nullptr;
    dz2_given = mask != nullptr;
    T *const out = mask ? node_grads.dz2 : dhA;
    if (pool_windows) {
      pool_windows_kernel<<<dim3((unsigned)(((G + kWindowStrip - 1) / kWindowStrip * (H / 4) + 255) / 256)), dim3(256), 0, c->stream>>>(
          rdx, d.graph_node_ptr, m.readout == XRL_READOUT_MEAN, G, H, dpool_rows);
      ClassSumArgs s;
      s.vals = dpool_rows; s.zero_row = c->zero_row; s.perm = q->mem_graph; s.seg = q->mem_seg; s.ptr = q->mem_ptr; s.n_rows = N; s.D = H;
      s.ymask = mask; s.out = out; s.carry = ccarry; s.slices = 1; s.group = kPoolPlaces;
      const int64_t groups = (N + s.group - 1) / s.group;
      const dim3 grid((unsigned)((groups + 3) / 4));
      pool_class_sum_kernel<T><<<grid, dim3(256), 0, c->stream>>>(s, G);
      class_sum_carried_kernel<T><<<dim3((unsigned)((groups + 4 * kCarryGroups - 1) / (4 * kCarryGroups))), dim3(256), 0, c->stream>>>(s);
      HIP_TRY(hipGetLastError());
    } else {
      broadcast_dpool_kernel<float><<<dim3((unsigned)((G * (H / 4) + 255) / 256)), dim3(256), 0, c->stream>>>(
          rdx, H, nullptr, d.graph_node_ptr, m.readout == XRL_READOUT_MEAN, G, H, dpool_rows);
      if ((rc = contract(float(), dpool_rows, q->mem_graph, q->mem_ptr, q->mem_seg, N, mask, out, (size_t)G * H * 4))) return rc;
    }
  } else if (N > 0) {
    if (dpool_table)
      broadcast_dpool_kernel<T><<<dim3((unsigned)((G * (H / 4) + 255) / 256)), dim3(256), 0, c->stream>>>(
          rdx, H, nullptr, d.graph_node_ptr, m.readout == XRL_READOUT_MEAN, G, H, dhA);
    else
      broadcast_dpool_kernel<T><<<dim3((unsigned)((N * (H / 4) + 255) / 256)), dim3(256), 0, c->stream>>>(
          rdx, H, d.node_graph, d.graph_node_ptr, m.readout == XRL_READOUT_MEAN, N, H, dhA);
  }
  bool dy_by_graph = dpool_table;          // until the first backward kernel has consumed the table

  Mlp2BwdArgs a;
  memset(&a, 0, sizeof(a));
  a.De = De; a.Dd = m.n_node_dense;
  // (after a forward of one launch per layer the received sums of nodes without in-edges were never written)
  a.zero_row = c->zero_row;
  auto set_w = [&](const EncMlp &e) {
    a.W1s = e.W1s; a.W2s = e.W2s; a.W2bt = e.W2bt; a.W1bt = e.W1bt; a.b1 = e.b1; a.b2 = e.b2; a.nslab1 = e.nslab1;
    a.W1x = e.W1x; a.nslabx = e.nslabx; a.table = e.table;
  };
  // both layers' weight gradients of an MLP whose gradients have been computed; x: the first layer's input
  auto wgrads = [&](WgradJob x, const MlpRef &r, const MlpGrads &mg, const void *z1) -> int {
    x.dZ = mg.dz1; x.dW = dweights + r.w[0]; x.db = dweights + r.b[0];
    if (int rc2 = queue_wgrad<T>(c, wq, x)) return rc2;
    WgradJob y = {};
    y.kind = WG_PLAIN; y.A = z1; y.Ka = H; y.n_rows = x.n_rows;
    y.dZ = mg.dz2; y.dW = dweights + r.w[1]; y.db = dweights + r.b[1];
    return queue_wgrad<T>(c, wq, y);
  };
  // gradients through one fused MLP: from what the forward kept, else with its first layer recomputed
  Mlp2BwdzArgs za;
  memset(&za, 0, sizeof(za));
  auto set_graph = [&](const LevelGraph &g) {
    a.in_ptr = g.in_ptr; a.in_src = g.in_src; a.in_dst = za.in_dst = g.in_dst;
    a.edge_feat = g.edge_feat; a.node_op = g.node_op; a.node_dense = g.node_dense;
    za.agg_src = g.agg_src;
    a.agg_src = c->agg_skip ? g.agg_src : nullptr;
    za.tile_ptr = g.tile_ptr; za.n_tiles = g.n_tiles;
  };
  auto mlp_bwd = [&](int kind, const EncMlp &e, const MlpGrads &mg, const uint16_t *z1mask, const uint16_t *ymask) -> int {
    a.z1 = mg.z1; a.dz1 = za.dz1 = mg.dz1; a.dz2 = za.dz2 = mg.dz2;
    if constexpr (sizeof(T) == 2) {
      if (kept || (embed_kept && kind == KIND_EMBED)) {
        za.n_rows = a.n_rows; za.W2bt = e.W2bt; za.W1bt = e.W1bt; za.dy = a.dy;
        za.z1mask = z1mask; za.ymask = ymask; za.dx_a = a.dx_a; za.dx_b = a.dx_b;
        za.dy_index = (dy_by_graph && kind != KIND_EDGE) ? d.node_graph : nullptr;
        dy_by_graph = false;
        const bool given = dz2_given && kind != KIND_EDGE;   // (the gather of the round above left dz2 in place)
        if (given) za.dy = mg.dz2;
        if (kind != KIND_EDGE) dz2_given = false;
        return launch_mlp2_bwdz(c, kind, za, fold, given);
      }
    }
    return launch_mlp2_bwd<T>(c, kind, a);
  };
  for (int r = R - 1; r >= 0 && gat; --r) {
    // attention round r+1: input h[r], saved z (in the agg slot) and scores, output h[r+1]; upstream dhA
    if (N == 0) break;
    Timed t(c, TK_GAT_BWD);
    GatBwdArgs ga;
    memset(&ga, 0, sizeof(ga));
    ga.n_rows = N; ga.z = c->agg[r + 1]; ga.hout = c->h[r + 1]; ga.dout = dhA;
    ga.s_src = c->gat_ss[r]; ga.s_dst = c->gat_sd[r];
    ga.a_src = c->d_w + c->L.gat[r].a_src; ga.a_dst = c->d_w + c->L.gat[r].a_dst;
    ga.in_ptr = d.in_ptr; ga.in_src = d.in_src; ga.in_dst = d.in_dst; ga.out_ptr = d.out_ptr; ga.out_pos = d.out_pos; ga.zero_row = c->zero_row;
    ga.alpha_e = g_ale; ga.du_e = g_due; ga.alpha_s = g_als; ga.du_s = g_dus; ga.d_ss = g_dss; ga.d_sd = g_dsd;
    MlpGrads mg;
    if ((rc = next_grads(N, &mg, 1))) return rc;
    ga.dpre = dpre; ga.dz = mg.dz1;
    const int64_t threads = N * (H / PV);
    const dim3 grid_n((unsigned)((threads + 255) / 256));
    gat_bwd_scores_kernel<T, PV><<<grid_n, dim3(256), 0, c->stream>>>(ga, H);
    gat_bwd_dz_kernel<T, PV><<<grid_n, dim3(256), 0, c->stream>>>(ga, H);
    // d a_src, d a_dst (neighbours in the weight vector): sums of chunks of rows, added up with the weight gradients
    const int64_t chunks = std::min<int64_t>(kAvecChunks, (N + 63) / 64);
    const int rpc = (int)((N + chunks - 1) / chunks);
    WgradJob av = {};
    av.ny = (int)((N + rpc - 1) / rpc); av.KaP = 2; av.k_rows = 2; av.bias_row = -1; av.n_rows = N;
    av.partial = g_avec + (size_t)r * kAvecChunks * 2 * H;
    av.dW = dweights + c->L.gat[r].a_src;
    gat_avec_grad_kernel<T, PV><<<dim3((unsigned)av.ny), dim3(256), (size_t)(256 / (H / PV)) * 2 * H * sizeof(float), c->stream>>>(
        (const T *)c->agg[r + 1], g_dss, g_dsd, N, rpc, H, av.partial);
    if ((rc = queue_wgrad<T>(c, wq, av))) return rc;
    // dW = h^T dz (no bias), dh = dz W^T
    WgradJob x = {};
    x.kind = WG_PLAIN; x.A = c->h[r]; x.Ka = H; x.n_rows = N; x.dZ = mg.dz1; x.dW = dweights + c->L.gat[r].W;
    if ((rc = queue_wgrad<T>(c, wq, x))) return rc;
    GatArgs gl;
    memset(&gl, 0, sizeof(gl));
    gl.n_rows = N;
    gl.h = mg.dz1; gl.Ws = c->gatWt[r]; gl.a_src = ga.a_src; gl.a_dst = ga.a_dst; gl.z = dhB;
    if ((rc = launch_gat_linear<T>(c, gl))) return rc;
    std::swap(dhA, dhB);
  }
  for (int r = R - 1; r >= 0 && !gat; --r) {
    // node MLP of round r+1: inputs h[r], agg[r+1]; output h[r+1]; upstream dhA
    const LevelGraph &g = lev(r + 1);
    const int64_t N = g.N, E = g.E;
    const void *h_in = q ? c->hx[r + 1] : c->h[r];
    set_graph(g);
    if (q) { dhB = dsrc + (size_t)E * H; ddst = dhB + (size_t)N * H; }
    set_w(c->node[r]);
    a.n_rows = N; a.h = h_in; a.agg = c->agg[r + 1]; a.y = c->h[r + 1]; a.dy = dhA;
    a.dx_a = dhB; a.dx_b = dagg;
    { Timed t(c, TK_BWD_NODE); rc = mlp_bwd(KIND_NODE, c->node[r], node_grads, kept ? c->zm_node[r] : nullptr, kept ? c->ym_node[r] : nullptr); }
    if (rc) return rc;
    WgradJob x = {};
    x.kind = WG_NODE; x.A = h_in; x.agg = c->agg[r + 1]; x.dst = g.agg_src; x.Ka = 2 * H; x.n_rows = N;
    if ((rc = wgrads(x, c->L.node[r], node_grads, kept ? c->z1_node[r] : node_grads.z1))) return rc;
    // edge MLP of round r+1: upstream = dagg gathered by receiver
    set_w(c->edge[r]);
    a.n_rows = E; a.h = h_in; a.agg = nullptr; a.y = nullptr; a.dy = dagg;
    a.dx_a = dsrc; a.dx_b = ddst;
    if ((rc = next_grads(E, &edge_grads, per_mlp))) return rc;
    { Timed t(c, TK_BWD_EDGE); rc = mlp_bwd(KIND_EDGE, c->edge[r], edge_grads, kept ? c->zm_edge[r] : nullptr, kept ? c->ym_edge[r] : nullptr); }
    if (rc) return rc;
    x.kind = WG_EDGE; x.agg = nullptr; x.src = g.in_src; x.dst = g.in_dst; x.edge_feat = g.edge_feat; x.De = De; x.n_rows = E;
    if ((rc = wgrads(x, c->L.edge[r], edge_grads, kept ? c->z1_edge[r] : edge_grads.z1))) return rc;
    if ((rc = next_grads(lev(r).N, &node_grads, per_mlp))) return rc;
    // dh[r] = d(node MLP)/dh + sum over in-edges of d h_receiver + sum over out-edges of d h_sender
    const uint16_t *below = kept ? (r > 0 ? c->ym_node[r - 1] : c->ym_embed) : nullptr;
    Timed timed(c, TK_GRAD_GATHER);
    if (q) {
      // ... of all the classes that split one of the level below, masked as below
      dz2_given = below != nullptr;
      if ((rc = contract(T(), dsrc, g.down, g.down_ptr, g.down_seg, level_rows(g, fold), below, below ? node_grads.dz2 : dhA, 0))) return rc;
      continue;
    }
    if (E > 0) {
      const int64_t threads = N * (H / PV);
      // from the kept forward: the sum leaves multiplied by the output mask of the layer that
      // produced h[r] (the node MLP of the round below, or the node-update layer), as that layer's
      // dz2 -- its backward kernel then neither reads the mask nor stores dz2
      T *masked_out = nullptr;
      const uint16_t *mask = nullptr;
      if constexpr (sizeof(T) == 2) {
        if (kept) { masked_out = node_grads.dz2; mask = below; }
      }
      node_grad_gather_kernel<T, PV><<<dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, c->stream>>>(
          ddst, dsrc, g.in_ptr, g.out_ptr, g.out_pos, N, H, dhB, fold ? 1 : 0, masked_out, mask);
      dz2_given = masked_out != nullptr;
    }
    std::swap(dhA, dhB);
  }
  // ---- node-update layer backward (weights only: its inputs are data)
  const LevelGraph &g0 = lev(0);
  set_graph(g0);
  set_w(c->embed);
  a.n_rows = N0; a.h = nullptr; a.agg = nullptr; a.y = c->h[0]; a.dy = dhA; a.dx_a = nullptr; a.dx_b = nullptr;
  if (gat && (rc = next_grads(N0, &node_grads, per_mlp))) return rc;
  { Timed t(c, TK_BWD_EMBED); rc = mlp_bwd(KIND_EMBED, c->embed, node_grads, embed_kept ? c->zm_embed : nullptr, embed_kept ? c->ym_embed : nullptr); }
  if (rc) return rc;
  // first layer: dW1 = X^T dz1, X written out once, its Kx real columns padded to Kp
  if (N0 > 0)
    embed_input_rows_kernel<T><<<dim3((unsigned)((N0 * (Kp / 8) + 255) / 256)), dim3(256), 0, c->stream>>>(
        g0.edge_feat, g0.in_ptr, g0.node_op, g0.node_dense, N0, De, m.n_op_types, m.n_node_dense, Kp, xrows);
  WgradJob x = {};
  x.kind = WG_PLAIN; x.A = xrows; x.Ka = Kp; x.k_rows = Kx; x.n_rows = N0;
  if ((rc = wgrads(x, c->L.embed, node_grads, embed_kept ? c->z1_embed : node_grads.z1))) return rc;
  if ((rc = flush_wgrads<T>(c, wq))) return rc;
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

template <typename T>
int encode_impl(xrl_ctx *c, const xrl_batch *b, float *d_emb, int save) {
  const xrl_model_desc &m = c->m;
  const int H = m.hidden, R = m.rounds, De = m.d_edge;
  const int64_t N = b->N, E = b->E, G = b->G;
  const Distinct *q = distinct_of(c, b);
  const LevelGraph whole = batch_graph(b);
  auto lev = [&](int l) -> const LevelGraph & { return q ? q->lv[l] : whole; };
  c->min_rows_now = !save ? c->p_min_rows_forward : (q && c->p_min_rows <= kPersistentMinRows ? 1 : c->p_min_rows);
  // A level's classes split those of the level below. fp32 kernels read the states there by index; others, and the backward
  // pass, go by a copy of the state each. (Re-evaluation of 73 k nodes in five levels, H = 128: 217 -> 203 us.)
  const bool below = q && !save && sizeof(T) == 4;
  // ---- workspace plan
  const int nh = save ? R + 1 : (R > 0 ? 2 : 1), nagg = save ? R : (R > 0 ? 1 : 0);
  int64_t maxN = 0, max_tiles = 0;
  for (int l = 0; l <= R; ++l) { maxN = std::max(maxN, lev(l).N); max_tiles = std::max(max_tiles, lev(l).n_tiles); }
  auto h_rows = [&](int i) { return (size_t)(save ? lev(i).N : maxN); };         // i-th buffer of h
  auto a_rows = [&](int i) { return (size_t)(save ? lev(i + 1).N : maxN); };     // ... of the received sums and of hx
  size_t need = 0;
  auto acc = [&](size_t bytes) { need += align_up(bytes); };
  constexpr int PV = 16 / sizeof(T);
  const bool gat = m.round_kind == XRL_ROUND_GAT;
  for (int i = 0; i < nh; ++i) acc(h_rows(i) * H * sizeof(T));
  for (int i = 0; i < nagg; ++i) acc(a_rows(i) * H * sizeof(T));        // (GAT: the agg slot holds z)
  for (int i = 0; q && !below && i < nagg; ++i) acc(a_rows(i) * H * sizeof(T));
  const xrl_batch_device &d = b->dev;
  const bool resident_ok = !gat && !q && H * sizeof(T) <= 256 && d.graph_tile_ptr && R <= kResidentMaxRounds;
  const int64_t resident_max = save ? c->resident_max_graphs : c->resident_max_forward;
  const int64_t cluster_max = save ? c->cluster_max_graphs : c->cluster_max_forward;
  const int64_t graph_tiles = std::max<int64_t>((b->max_graph_nodes + 31) / 32, b->max_graph_tiles);
  // blocks per graph of the one-launch encoder: one while a graph's phase is a single pass of a
  // block's four waves; otherwise as many as give every tile of a phase a wave of its own, if
  // that many are resident at once (at most one block per CU; graphs padded to a multiple of 8)
  int cluster_k = 0;
  if (resident_ok && c->resident_max_graphs > 0 && G <= cluster_max && G > 0 &&
      graph_tiles > c->resident_max_tiles) {
    const int64_t slots = c->n_cu / (8 * ((G + 7) / 8));
    cluster_k = (int)((graph_tiles + 3) / 4);
    if (cluster_k > slots) cluster_k = 0;   // a phase would take a second pass: the launch-per-phase path is as fast
  }
  const bool resident_batch = resident_ok && ((G <= resident_max && graph_tiles <= c->resident_max_tiles) ||
                                              cluster_k > 0);
  // Large bf16 batches run on kernels that can keep z1 and the ReLU masks of every fused MLP for
  // the backward pass (a row of H elements and 2 H / 32 words per node or edge and MLP): kept when
  // every launch of this encode is one of them.
  bool keep = false;
  if constexpr (sizeof(T) == 2) {
    if (save && !gat && !resident_batch && N > 0) {
      Mlp2Args t;
      memset(&t, 0, sizeof(t));
      t.De = De; t.Tn = m.n_op_types; t.Dd = m.n_node_dense;
      t.n_rows = lev(0).N; t.nslabx = c->embed.nslabx;
      keep = mlp2p_applies(c, KIND_EMBED, t);
      for (int r = 0; r < R && keep; ++r) {
        t.n_rows = lev(r + 1).E; t.nslab1 = c->edge[r].nslab1;
        keep = keep && (mlp2r_applies(c, KIND_EDGE, t) || mlp2p_applies(c, KIND_EDGE, t));
        t.n_rows = lev(r + 1).N; t.nslab1 = c->node[r].nslab1;
        keep = keep && (mlp2r_applies(c, KIND_NODE, t) || mlp2p_applies(c, KIND_NODE, t));
      }
    }
  }
  bool keep_embed = keep;
  if constexpr (sizeof(T) == 2) {
    // (attention rounds: the embed MLP's backward from what its forward kept; recomputing it took 81 us at 148 k
    // nodes, H = 128, from mask bits half of that)
    if (save && gat && N > 0) {
      Mlp2Args t;
      memset(&t, 0, sizeof(t));
      t.De = De; t.Tn = m.n_op_types; t.Dd = m.n_node_dense; t.n_rows = N; t.nslabx = c->embed.nslabx;
      keep_embed = mlp2p_applies(c, KIND_EMBED, t);
    }
  }
  auto ym_words = [&](int l) { return (size_t)lev(l).n_tiles * (H / 32) * 64; };          // 16-bit words of one edge MLP's mask bits (z1 or y)
  auto nm_words = [&](int l) { return (size_t)((lev(l).N + 31) / 32) * (H / 32) * 64; };  // ... of a node-side MLP's
  if (keep_embed && !keep) {
    acc((size_t)N * H * sizeof(T));
    acc(nm_words(0) * 2); acc(nm_words(0) * 2);
  }
  if (keep) {
    for (int l = 0; l <= R; ++l) {
      acc((size_t)lev(l).N * H * sizeof(T));
      acc(nm_words(l) * 2); acc(nm_words(l) * 2);
      if (l > 0) { acc((size_t)lev(l).E * H * sizeof(T)); acc(ym_words(l) * 2); acc(ym_words(l) * 2); }
    }
  }
  const int n_gs = gat ? (save ? R : std::min(R, 2)) : 0;               // saved per round for the backward; or in turn
  for (int i = 0; i < 2 * n_gs; ++i) acc((size_t)N * 4);
  // (a reduced batch has few huge graphs at most: the carries of the readout's segment sum are not needed)
  const size_t carry_floats = std::max(std::max(segsum_carry_floats(E, De), q && N <= 4096 * G ? 0 : segsum_carry_floats(N, H)),
                                       (size_t)max_tiles * 2 * H);
  acc(carry_floats * 4);
  acc((size_t)G * H * 4);
  acc((size_t)G * H * 4);
  acc((size_t)G * H * 4);
  // (the levels of a batch reduced for this encode lie behind the rest, so that there is one allocation and wait at most: a context's
  // first call, 287 k nodes at H = 256, held its caller 846 us with a second one, 557 so. RelaxedCapture: an encode that neither
  // allocated nor waited before must not end another stream's capture)
  OnceLevels once;
  bool by_levels = false;
  int rc = XRL_OK;
  const size_t o_levels = need;
  if constexpr (sizeof(T) == 2) by_levels = !save && !q && once_pays(c, b);
  if (by_levels) {
    RelaxedCapture relaxed;
    const size_t bytes = o_levels + once_plan(c, b, nullptr, once);
    rc = bytes < c->levels_refused ? ensure_ws(c, bytes) : XRL_ERR_OOM;
    if (rc && rc != XRL_ERR_OOM) return rc;
    by_levels = rc == XRL_OK;          // (no memory for them: the batch is encoded as it is, and as much is not asked for again)
    if (!by_levels) c->levels_refused = std::min(c->levels_refused, bytes);
  }
  if (!by_levels && (rc = ensure_ws(c, need))) return rc;
  Bump bump{c->ws};
  c->h.assign(R + 1, nullptr);
  c->agg.assign(R + 1, nullptr);
  std::vector<T *> hb(nh), ab(std::max(nagg, 1), nullptr);
  std::vector<T *> xb(std::max(nagg, 1), nullptr);
  c->hx.assign(R + 1, nullptr);
  for (int i = 0; i < nh; ++i) hb[i] = bump.take<T>(h_rows(i) * H);
  for (int i = 0; i < nagg; ++i) ab[i] = bump.take<T>(a_rows(i) * H);
  for (int i = 0; q && !below && i < nagg; ++i) xb[i] = bump.take<T>(a_rows(i) * H);
  c->gat_ss.assign(R, nullptr);
  c->gat_sd.assign(R, nullptr);
  for (int i = 0; i < n_gs; ++i) {
    c->gat_ss[i] = bump.take<float>((size_t)N);
    c->gat_sd[i] = bump.take<float>((size_t)N);
  }
  c->carry = bump.take<float>(carry_floats);
  c->pool = bump.take<float>((size_t)G * H);
  c->ro_act[0] = bump.take<float>((size_t)G * H);
  c->ro_act[1] = bump.take<float>((size_t)G * H);
  c->fwd_kept = keep;
  c->embed_kept = keep_embed;
  c->z1_edge.assign(R, nullptr); c->z1_node.assign(R, nullptr);
  c->ym_edge.assign(R, nullptr); c->zm_edge.assign(R, nullptr);
  c->ym_node.assign(R, nullptr); c->zm_node.assign(R, nullptr);
  c->z1_embed = nullptr; c->ym_embed = c->zm_embed = nullptr;
  if (keep_embed) {
    c->z1_embed = bump.take<T>((size_t)lev(0).N * H);
    c->zm_embed = bump.take<uint16_t>(nm_words(0));
    c->ym_embed = bump.take<uint16_t>(nm_words(0));
  }
  if (keep) {
    for (int r = 0; r < R; ++r) {
      c->z1_node[r] = bump.take<T>((size_t)lev(r + 1).N * H);
      c->z1_edge[r] = bump.take<T>((size_t)lev(r + 1).E * H);
      c->zm_edge[r] = bump.take<uint16_t>(ym_words(r + 1));
      c->ym_edge[r] = bump.take<uint16_t>(ym_words(r + 1));
      c->zm_node[r] = bump.take<uint16_t>(nm_words(r + 1));
      c->ym_node[r] = bump.take<uint16_t>(nm_words(r + 1));
    }
  }
  c->enc_batch = b->id;
  c->enc_saved = save != 0;

  // ---- global-update layer: per-graph sum (or mean) of the last states (with cls: of each node's class), then the readout MLP
  auto readout = [&](const T *hlast, const int32_t *cls) -> int {
    int rc = XRL_OK;
    if (N <= 4096 * G) {
      // Many graphs of moderate size: a block per graph. The readout MLP follows in the same launch where two blocks lie on a compute unit at
      // most, of the narrower rows three come one after the other; beyond, in a launch of its own, where sixteen graphs share the weights' way from L2.
      // us of a bf16 encode of one round, graphs of 50 nodes, in one launch / two: H = 64, 257 graphs 17.6 / 21.1, 512 24.1 / 26.9, 768 30.4 / 30.9,
      // 1040 36.4 / 34.8; H = 128 24.1 / 27.4, 37.9 / 40.6, 47.9 / 47.9, 56.7 / 52.8; H = 256 59.6 / 63.4, 74.6 / 77.1, 98.1 / 94.2, 123 / 110.
      const RowFwdArgs ra = row_fwd_args(c, c->L.readout, true, c->pool, H, d.graph_global, m.d_global, G, d_emb, c->ro_act);
      const int mean = m.readout == XRL_READOUT_MEAN ? 1 : 0;
      if (G > (H == 256 ? 2 : 3) * c->n_cu) {
        { Timed t(c, TK_POOL);
          rc = with_readout_widths(c, [&](auto fwd, auto) -> int {
            constexpr int HH = decltype(fwd)::w[1];
            auto kern = cls ? graph_pool_kernel<T, PV, HH, true> : graph_pool_kernel<T, PV, HH, false>;
            kern<<<dim3((unsigned)G), dim3(kPoolThreads), 0, c->stream>>>(hlast, d.graph_node_ptr, cls, mean, c->pool);
            HIP_TRY(hipGetLastError());
            return XRL_OK;
          }); }
        if (rc) return rc;
        Timed t(c, TK_READOUT);
        return launch_readout(c, ra);
      }
      if (G == 0) return XRL_OK;
      Timed t(c, TK_POOL);
      return with_readout_widths(c, [&](auto fwd, auto) -> int {
        constexpr int HH = decltype(fwd)::w[1];
        auto kern = cls ? graph_readout_kernel<T, PV, HH, true> : graph_readout_kernel<T, PV, HH, false>;
        kern<<<dim3((unsigned)G), dim3(kRowThreads), 0, c->stream>>>(hlast, d.graph_node_ptr, cls, mean, c->pool, ra);
        HIP_TRY(hipGetLastError());
        return XRL_OK;
      });
    }
    { Timed t(c, TK_POOL);
      rc = launch_segsum<T, float, PV>(c, hlast, cls, d.graph_node_ptr, d.node_graph, N, G, H, c->pool, c->carry); }
    if (rc) return rc;
    if (m.readout == XRL_READOUT_MEAN && G > 0)
      mean_scale_kernel<<<dim3((unsigned)((G * H + 255) / 256)), dim3(256), 0, c->stream>>>(c->pool, d.graph_node_ptr, G, H, 0);
    { Timed t(c, TK_READOUT);
      rc = launch_readout(c, row_fwd_args(c, c->L.readout, true, c->pool, H, d.graph_global, m.d_global, G, d_emb, c->ro_act)); }
    if (rc) return rc;
    HIP_TRY(hipGetLastError());
    return XRL_OK;
  };
  // ---- node-update layer: the embed MLP (it sums each node's incoming edge attrs itself)
  Mlp2Args a;
  memset(&a, 0, sizeof(a));
  a.De = De; a.Tn = m.n_op_types; a.Dd = m.n_node_dense;
  auto set_graph = [&](const LevelGraph &g) {
    a.in_ptr = g.in_ptr; a.in_src = g.in_src; a.in_dst = g.in_dst;
    a.edge_feat = g.edge_feat; a.node_op = g.node_op; a.node_dense = g.node_dense;
    a.tile_ptr = g.tile_ptr; a.n_tiles = g.n_tiles;
  };
  set_graph(lev(0));
  a.carry = c->carry; a.zero_row = c->zero_row;
  auto set_w = [&](const EncMlp &e) {
    const bool parts = c->parts() && &e != &c->embed;
    a.W1s = parts ? e.W1p : e.W1s; a.W2s = parts ? e.W2p : e.W2s; a.W1 = e.W1; a.W2 = e.W2; a.b1 = e.b1; a.b2 = e.b2;
    a.nslab1 = parts ? (e.nslab1 + 1) / 2 : e.nslab1;       // (in parts: slabs of sixteen columns)
    a.W1x = e.W1x; a.nslabx = e.nslabx; a.table = e.table;
  };
  set_w(c->embed);
  a.n_rows = lev(0).N; a.out = hb[0];
  a.agg0 = ab[0]; a.n_agg = gat ? 0 : nagg; a.agg_stride = nagg > 1 ? (size_t)((char *)ab[1] - (char *)ab[0]) : 0;
  if (resident_batch) {
    // small batch: the whole encoder in one launch, one block per graph (rows of at most 256
    // bytes: the three inlined tile routines of wider ones do not fit the register file)
    ResidentArgs ra;
    memset(&ra, 0, sizeof(ra));
    c->agg_skip = false;               // (the node-update layer zeroes the rows nobody else writes)
    ra.base = a;
    ra.rounds = R; ra.E = E;
    ra.graph_node_ptr = d.graph_node_ptr; ra.graph_tile_ptr = d.graph_tile_ptr; ra.gtile_ptr = d.gtile_ptr;
    ra.h[0] = hb[0];
    c->h[0] = hb[0];
    for (int r = 0; r < R; ++r) {
      ra.edge[r] = ResidentMlp{c->edge[r].W1s, c->edge[r].W2s, c->edge[r].b1, c->edge[r].b2, c->edge[r].nslab1};
      ra.node[r] = ResidentMlp{c->node[r].W1s, c->node[r].W2s, c->node[r].b1, c->node[r].b2, c->node[r].nslab1};
      ra.agg[r] = save ? ab[r] : ab[0];
      ra.h[r + 1] = save ? hb[r + 1] : hb[(r + 1) & 1];
      c->h[r + 1] = ra.h[r + 1];
      c->agg[r + 1] = ra.agg[r];
    }
    const int MB = H / 32;
    int w1 = c->embed.nslabx;
    for (int r = 0; r < R; ++r) w1 = std::max(w1, std::max(c->edge[r].nslab1, c->node[r].nslab1));
    ra.w1_bytes_max = w1 * MB * 1024;
    const size_t w2_bytes = (size_t)MB * (32 / (2 * PV)) * MB * 1024;
    const size_t lds = (size_t)4 * RowStage<T, 128>::BYTES + ra.w1_bytes_max + w2_bytes + (size_t)m.n_op_types * H * 4;
    ra.K = cluster_k; ra.G = (int)G; ra.arrived = c->d_arrived; ra.fault = c->d_fault; ra.spin_limit = c->cluster_spin_limit;
    if (lds <= (size_t)c->max_lds) {
      const unsigned grid = cluster_k > 0 ? (unsigned)(8 * ((G + 7) / 8) * cluster_k) : (unsigned)G;
      auto launch = [&](auto kern) -> int {
        if (lds > 65536) HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        { Timed t(c, TK_RESIDENT);
          kern<<<dim3(grid), dim3(256), lds, c->stream>>>(ra); }
        HIP_TRY(hipGetLastError());
        return readout((const T *)ra.h[R], nullptr);
      };
      if (cluster_k > 0) {   // (grid <= number of CUs and a block fits a CU: every block is resident)
        if (H == 64) return launch(encode_cluster_kernel<T, 64>);
        if constexpr (sizeof(T) == 2) return launch(encode_cluster_kernel<T, 128>);
      } else {
        if (H == 64) return launch(encode_resident_kernel<T, 64>);
        if constexpr (sizeof(T) == 2) return launch(encode_resident_kernel<T, 128>);
      }
    }
  }
  // one launch per layer: the node MLPs (and whatever reads the received sums afterwards) take
  // zeros for nodes without in-edges through agg_src, so nobody has to write those rows
  a.n_agg = 0; a.agg_src = lev(0).agg_src;
  c->agg_skip = !gat;
  if constexpr (sizeof(T) == 2) {
    if (by_levels) {
      once_plan(c, b, c->ws + o_levels, once);
      { Timed t(c, TK_LEVELS); rc = once_begin(c, b, once); }
      if (rc) return rc;
      { Timed t(c, TK_LEVELS); rc = once_level(c, b, once, 0, a); }
      if (rc) return rc;
      { Timed t(c, TK_EMBED); rc = launch_embedp_s<256, false, true>(c, a); }
      if (rc) return rc;
      T *hcur = hb[0];
      for (int r = 0; r < R; ++r) {
        T *hnext = hb[(r + 1) & 1];
        { Timed t(c, TK_LEVELS); rc = once_level(c, b, once, r + 1, a); }
        if (rc) return rc;
        set_w(c->edge[r]);
        a.n_rows = E; a.h = hcur; a.out = ab[0]; a.h_row = once.o.o_hrow;
        { Timed t(c, TK_EDGE); rc = launch_mlp2r_ks<256, KIND_EDGE, false, true>(c, a); }
        if (rc) return rc;
        set_w(c->node[r]);
        a.n_rows = N; a.agg = ab[0]; a.out = hnext; a.h_row = once.o.o_self;
        { Timed t(c, TK_NODE); rc = launch_mlp2r_ks<256, KIND_NODE, false, true>(c, a); }
        if (rc) return rc;
        hcur = hnext;
      }
      return readout(hcur, once.classes(R));
    }
  }
  a.z1 = c->z1_embed; a.z1mask = c->zm_embed; a.ymask = c->ym_embed;
  { Timed t(c, TK_EMBED); rc = launch_mlp2<T>(c, KIND_EMBED, a); }
  if (rc) return rc;
  c->h[0] = hb[0];
  T *hcur = hb[0];
  // ---- message-passing rounds
  bool one_launch = false;             // a whole round in one launch
  for (int r = 0; r < R; ++r) {
    T *aggb = save ? ab[r] : ab[0];
    T *hnext = save ? hb[r + 1] : hb[(r + 1) & 1];
    const LevelGraph &g = lev(r + 1);
    const int64_t N = g.N, E = g.E;
    if (q && !below) {
      T *x = save ? xb[r] : xb[0];
      const int pieces = H / PV;
      expand_states_kernel<<<dim3((unsigned)((N * pieces + 255) / 256)), dim3(256), 0, c->stream>>>(
          (const f32x4 *)hcur, g.self, N, pieces, (f32x4 *)x);
      c->hx[r + 1] = x;
      hcur = x;
    }
    if (gat) {                         // graph-attention reading of the round
      if (N > 0) {
        const bool fused = gat_round_applies<T>(c, N);
        // (not saved, z of one round is read while that of the next is written: in turn in ab[0] and, once the first
        // product has read h from there, hb[0])
        if (!save && fused) { aggb = r % 2 ? hb[0] : ab[0]; hnext = hb[1]; }
        GatArgs ga;
        ga.n_rows = N;
        ga.h = hcur; ga.Ws = c->gatW[r];
        ga.a_src = c->d_w + c->L.gat[r].a_src; ga.a_dst = c->d_w + c->L.gat[r].a_dst;
        ga.z = aggb; ga.s_src = c->gat_ss[save ? r : r % n_gs]; ga.s_dst = c->gat_sd[save ? r : r % n_gs];
        ga.in_ptr = d.in_ptr; ga.in_src = d.in_src; ga.out = hnext; ga.zero_row = c->zero_row;
        if (r == 0 || !fused) { Timed t(c, TK_GAT_LINEAR); if ((rc = launch_gat_linear<T>(c, ga))) return rc; }
        if (fused && r + 1 < R) {
          if (!save) ga.out = nullptr;
          const GatNext next = {c->gatW[r + 1], c->d_w + c->L.gat[r + 1].a_src, c->d_w + c->L.gat[r + 1].a_dst,
                                save ? ab[r + 1] : r % 2 ? ab[0] : hb[0], c->gat_ss[save ? r + 1 : (r + 1) % n_gs],
                                c->gat_sd[save ? r + 1 : (r + 1) % n_gs]};
          Timed t(c, TK_ROUND);
          if ((rc = launch_gat_round<T>(c, ga, next))) return rc;
        } else { Timed t(c, TK_GAT_AGGREGATE);
          const int64_t threads = N * (H / PV);
          gat_aggregate_kernel<T, PV><<<dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, c->stream>>>(ga, H); }
        HIP_TRY(hipGetLastError());
      }
      c->h[r + 1] = hnext;
      c->agg[r + 1] = aggb;            // (z of this round)
      hcur = hnext;
      continue;
    }
    set_graph(g);
    a.agg_src = g.agg_src;
    if (!q && r == 0 && !save) one_launch = b->n_split_tiles == 0 && round_applies<T>(c, g, b->at<int32_t>(b->o_in_ptr));
    if (q && !save) one_launch = !below && round_applies<T>(c, g, nullptr);     // (a round in one launch reads copied states)
    if (one_launch) {
      RoundArgs ra;
      set_w(c->edge[r]);
      a.n_rows = E; a.h = hcur;
      ra.edge = a;
      set_w(c->node[r]);
      a.n_rows = N; a.out = hnext;
      ra.node = a;
      { Timed t(c, TK_ROUND); rc = launch_round<T>(c, ra); }
      if (rc) return rc;
      c->h[r + 1] = hnext;
      hcur = hnext;
      continue;
    }
    set_w(c->edge[r]);
    a.n_rows = E; a.h = hcur; a.out = aggb;
    if (below) { a.in_src = g.below_src; a.h_row = g.below_dst; }
    a.z1 = c->z1_edge[r]; a.z1mask = c->zm_edge[r]; a.ymask = c->ym_edge[r];
    { Timed t(c, TK_EDGE); rc = launch_mlp2<T>(c, KIND_EDGE, a); }
    if (rc) return rc;
    if (b->n_split_tiles > 0) {         // only a receiver with more than 32 in-edges spans tiles
      Timed t(c, TK_EDGE_FIXUP);
      const int64_t n_tiles = g.n_tiles, fthreads = n_tiles * (H / 4);
      edge_tile_fixup<T><<<dim3((unsigned)((fthreads + 255) / 256)), dim3(256), 0, c->stream>>>(
          d.tile_ptr, n_tiles, d.in_ptr, d.in_dst, H, c->carry, aggb);
    }
    set_w(c->node[r]);
    a.n_rows = N; a.h = hcur; a.agg = aggb; a.out = hnext;
    if (below) a.h_row = g.self;
    a.z1 = c->z1_node[r]; a.z1mask = c->zm_node[r]; a.ymask = c->ym_node[r];
    { Timed t(c, TK_NODE); rc = launch_mlp2<T>(c, KIND_NODE, a); }
    if (rc) return rc;
    c->h[r + 1] = hnext;
    c->agg[r + 1] = aggb;
    hcur = hnext;
  }
  return readout(hcur, q ? q->cls[R] : nullptr);
}

}  // namespace

extern "C" {

int xrl_create(const xrl_model_desc *model, const float *weights_host, void *hip_stream,
               xrl_ctx **out) {
  if (!model || !weights_host || !out) return fail(XRL_ERR_NULL, "xrl_create: NULL argument");
  *out = nullptr;
  Layout L, Lu;
  int rc = build_layout(*model, Lu);
  if (rc) return rc;
  if (model->hidden != 64 && model->hidden != 128 && model->hidden != 256)
    return fail(XRL_ERR_UNSUPPORTED, "hidden = %d: the kernels cover 64, 128 and 256", model->hidden);
  if (model->mlp_layers != 1 && model->mlp_layers != 2)
    return fail(XRL_ERR_UNSUPPORTED, "mlp_layers = %d: the kernels cover 1 and 2", model->mlp_layers);
  xrl_model_desc model_int = *model;
  model_int.mlp_layers = 2;
  if ((rc = build_layout(model_int, L))) return rc;
  const bool single_layer = model->mlp_layers == 1;
  model = &model_int;
  if (model->d_edge % 4 != 0)
    return fail(XRL_ERR_UNSUPPORTED, "d_edge = %d: the kernels need a multiple of 4", model->d_edge);
  if (model->head_hidden[0] > 512 || model->head_hidden[1] > 512 || model->d_global > 256 ||
      model->d_edge > 256 || model->n_op_types + model->n_node_dense > 1024)
    return fail(XRL_ERR_UNSUPPORTED, "head/global/edge/node attribute width beyond the kernels' range");
  int ndev = 0;
  hipError_t e = hipGetDeviceCount(&ndev);
  if (e != hipSuccess || ndev < 1) {
    (void)hipGetLastError();
    return fail(XRL_ERR_HIP, "no usable GPU: %s", e != hipSuccess ? hipGetErrorString(e) : "0 devices");
  }
  xrl_ctx *c = new (std::nothrow) xrl_ctx();
  if (!c) return fail(XRL_ERR_OOM, "xrl_create: out of host memory");
  static std::atomic<uint64_t> next_ctx{1};
  c->id = next_ctx++;
  c->blocks = std::make_shared<DevicePool>();
  c->blocks->stream = (hipStream_t)hip_stream;
  if (hipGetDevice(&c->device) != hipSuccess) (void)hipGetLastError();
  c->blocks->device = c->device;
  host_pool_context(1, c->device);
  c->m = *model;
  c->L = L;
  c->single_layer = single_layer;
  if (single_layer) c->Lu = Lu;
  c->stream = (hipStream_t)hip_stream;
  c->elem = model->precision == XRL_PREC_BF16 ? 2 : 4;
  // Row count from which the persistent kernels replace the split one (tuning knob; the
  // default is where they start to win; 0 = always, a huge value = never)
  c->p_min_rows = kPersistentMinRows;
  if (const char *e = getenv("XRL_DISTINCT_MIN_US")) c->distinct_min_us = atoll(e);
  // Saving from these on keeps the forward for the backward pass. Without that, H <= 128, five rounds, us per
  // encode, persistent / split kernels: 10.5 k nodes 120 / 74, 17.5 k 128 / 96, 34.5 k 141 / 140, 73 k 188 / 232
  // (H = 64: 17.5 k 73 / 59, 73 k 105 / 113); H = 256: 17.5 k 194 / 215
  c->p_min_rows_forward = model->hidden <= 128 ? 4 * kPersistentMinRows : kPersistentMinRows;
  if (const char *e = getenv("XRL_PERSISTENT_MIN_ROWS")) c->p_min_rows = c->p_min_rows_forward = atoll(e);
  if (const char *e = getenv("XRL_WGRAD_WIDE_MIN_ROWS")) c->wide_min_rows = atoll(e);
  c->round_blocks = model->hidden == 64 ? 4 : 2;
  if (const char *e = getenv("XRL_ROUND_BLOCKS")) { c->round_blocks = atoll(e); c->round_any = true; }
  if (const char *e = getenv("XRL_SUM_STEPS")) c->sum_steps = atoi(e);
  if (const char *e = getenv("XRL_POOL_WINDOW_NODES")) c->pool_window_nodes = atoll(e);
  if (const char *e = getenv("XRL_GRAD_ROOM")) c->grad_room = (size_t)std::max<long long>(0, atoll(e));
  // Largest batches of the one-launch encoders (0 graphs = never). A forward-only encode takes them up to a
  // limit that the variable of that form states, and by default never: since a tile of the
  // launch-per-layer path is split over H / 32 waves that path is the faster one at every size they
  // cover (us per encode, one launch / a launch per layer: nine 50-node graphs, fp32, H = 64, two
  // rounds 50 / 38; bf16, H = 128, five rounds: the same graphs 79 / 57, 200 of them 81 / 76, 15 graphs of 338
  // nodes 97 / 61, of 565 nodes 106 / 76). Saving for the backward pass, where from 8192 rows on the other path
  // is the persistent kernels': the nine graphs 51 / 39, 79 / 63, the 200 (10 k nodes) 88 / 167, 338 nodes 101 / 68,
  // 565 nodes (8.5 k) 117 / 160; with the backward pass, which starts from more there, 295 / 284, 488 / 466,
  // 659 / 669, 619 / 576, 657 / 630.
  // (one block of four waves per graph while every phase of a graph is a single pass of its waves)
  c->resident_max_graphs = 256;
  c->resident_max_tiles = 4;
  if (const char *e = getenv("XRL_RESIDENT_MAX_GRAPHS")) c->resident_max_graphs = c->resident_max_forward = atoll(e);
  if (const char *e = getenv("XRL_RESIDENT_MAX_TILES")) c->resident_max_tiles = atoll(e);
  // ... and with several blocks per graph, for the few dozen larger graphs of one rewriting step
  c->cluster_max_graphs = 48;
  if (const char *e = getenv("XRL_CLUSTER_MAX_GRAPHS"))
    c->cluster_max_graphs = c->cluster_max_forward = std::min<int64_t>(atoll(e), kClusterMaxGraphs);
  if (const char *e = getenv("XRL_CLUSTER_SPIN_LIMIT")) c->cluster_spin_limit = (unsigned)std::max<long long>(0, std::min<long long>(atoll(e), kClusterSpinLimit));
  {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, c->device) == hipSuccess && v > 0) c->n_cu = v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, c->device) == hipSuccess && v > 0) c->max_lds = v;
  }
  // the weights, followed by 1 KB of zeros (16-byte aligned) that kernels read in place of absent rows
  const size_t w_bytes = align_up(sizeof(float) * L.total);
  // zero row, heads' counters, the one-launch encoder's counters
  const size_t tail_bytes = kZeroRow + sizeof(int32_t) * kMaxFusedStates + sizeof(unsigned) * kClusterMaxGraphs + sizeof(int32_t) * kCounts;
  e = hipMalloc((void **)&c->d_w, w_bytes + tail_bytes);
  if (e != hipSuccess) {
    xrl_destroy(c);
    return fail(XRL_ERR_OOM, "device weights: %s", hipGetErrorString(e));
  }
  c->zero_row = (char *)c->d_w + w_bytes;
  c->d_counter = (int32_t *)((char *)c->zero_row + kZeroRow);
  c->d_arrived = (unsigned *)(c->d_counter + kMaxFusedStates);
  c->d_counts = (int32_t *)(c->d_arrived + kClusterMaxGraphs);
  e = hipMemset(c->zero_row, 0, tail_bytes);
  if (e != hipSuccess) {
    xrl_destroy(c);
    return fail(XRL_ERR_HIP, "hipMemset: %s", hipGetErrorString(e));
  }
  const uint32_t one = c->elem == 2 ? 0x3f80u : 0x3f800000u;       // 1 in the operand type, zeros behind it
  e = hipMemcpy((char *)c->zero_row + 1024, &one, sizeof(one), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    xrl_destroy(c);
    return fail(XRL_ERR_HIP, "hipMemcpy: %s", hipGetErrorString(e));
  }
  e = hipHostMalloc((void **)&c->h_counts, sizeof(int32_t) * kCounts, hipHostMallocDefault);
  if (e == hipSuccess) e = hipHostMalloc((void **)&c->h_fault, sizeof(unsigned), hipHostMallocMapped);
  if (e == hipSuccess) {
    *c->h_fault = 0;
    e = hipHostGetDevicePointer((void **)&c->d_fault, c->h_fault, 0);
  }
  if (e != hipSuccess) {
    xrl_destroy(c);
    return fail(XRL_ERR_HIP, "pinned status word: %s", hipGetErrorString(e));
  }
  rc = plan_weights(c);
  if (!rc) rc = upload_weights(c, weights_host);
  if (!rc && c->single_layer) {
    std::vector<int32_t> wmap((size_t)c->Lu.total);
    for (const WeightTensor &t : c->Lu.tensors) {
      const int64_t n = t.cols > 0 ? t.rows * t.cols : t.rows, o = internal_offset(c, t);
      for (int64_t i = 0; i < n; ++i) wmap[(size_t)(t.offset + i)] = (int32_t)(o + i);
    }
    e = hipMalloc((void **)&c->d_dw_int, sizeof(float) * (size_t)c->L.total);
    if (e == hipSuccess) e = hipMalloc((void **)&c->d_wmap, sizeof(int32_t) * wmap.size());
    if (e == hipSuccess) e = hipMemcpy(c->d_wmap, wmap.data(), sizeof(int32_t) * wmap.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) rc = fail(XRL_ERR_OOM, "internal gradient vector: %s", hipGetErrorString(e));
  }
  if (!rc) rc = static_scratch(c->device, &c->static_ws);
  if (rc) {
    xrl_destroy(c);
    return rc;
  }
  *out = c;
  return XRL_OK;
}

int xrl_set_weights(xrl_ctx *c, const float *weights_host) {
  if (!c || !weights_host) return fail(XRL_ERR_NULL, "xrl_set_weights: NULL argument");
  return upload_weights(c, weights_host);
}

int xrl_destroy(xrl_ctx *c) {
  if (!c) return XRL_OK;
  (void)hipStreamSynchronize(c->stream);
  if (c->d_w) (void)hipFree(c->d_w);
  if (c->h_fault) (void)hipHostFree(c->h_fault);
  if (c->h_counts) (void)hipHostFree(c->h_counts);
  if (c->d_dw_int) (void)hipFree(c->d_dw_int);
  if (c->d_wmap) (void)hipFree(c->d_wmap);
  if (c->d_swz) (void)hipFree(c->d_swz);
  if (c->d_wstage) (void)hipFree(c->d_wstage);
  if (c->h_wstage) (void)hipHostFree(c->h_wstage);
  if (c->wstage_free) (void)hipEventDestroy(c->wstage_free);
  if (c->ws) (void)hipFree(c->ws);
  if (c->hws) (void)hipFree(c->hws);
  if (c->bws) (void)hipFree(c->bws);
  for (auto &sp : c->spans) { (void)hipEventDestroy(sp.a); (void)hipEventDestroy(sp.b); }
  for (auto &e : c->free_events) (void)hipEventDestroy(e);
  c->blocks->close();
  if (c->copy_stream) {
    (void)hipStreamSynchronize(c->copy_stream);
    (void)hipStreamDestroy(c->copy_stream);
  }
  host_pool_context(-1);
  delete c;
  return XRL_OK;
}

namespace {
// out[i, :] = from[i] >= 0 ? base[from[i], :] : added[-1 - from[i], :], rows of `width` 4-byte words:
// the per-node and per-edge attribute arrays of a batch packed from edits, filled on the device
// from the current graphs' attributes and the new items'.
__global__ void expand_rows_kernel(const int32_t *from, int64_t n, int width, const uint32_t *base, const uint32_t *added,
                                   uint32_t *out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * width) return;
  const int64_t r = i / width;
  const int j = (int)(i - r * width);
  const int32_t f = from[r];
  out[i] = f >= 0 ? base[(size_t)f * width + j] : added[(size_t)(-1 - f) * width + j];
}
// What follows from a batch's in-edge ranges and its graphs' node ranges, one thread per node: agg_src (n for a
// node with in-edges, -1 for one without), the receiver of every edge and the graph of every node. Packing and
// sending them and the sender index instead took a fifth of a batch's bytes (half of one packed from edits):
// us per step, four alternating runs each (the host's part varies): 129 graphs of 565 nodes 365 to 388 / 322 to 384 without, from
// edits 417 to 448 / 365 to 379, 2080 graphs of 338 nodes 1929 to 2191 / 1536 to 1713.
__global__ __launch_bounds__(256) void derive_index_kernel(const int32_t *in_ptr, const int32_t *graph_node_ptr, int64_t N, int G,
                                                           int32_t *agg_src, int32_t *in_dst, int32_t *node_graph) {
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  constexpr int kFew = 8;                    // in-edges a thread writes itself
  int e0 = 0, e1 = 0;
  if (n < N) {
    e0 = in_ptr[n];
    e1 = in_ptr[n + 1];
    agg_src[n] = e1 > e0 ? (int32_t)n : -1;
    node_graph[n] = seg_of_row(graph_node_ptr, G, n);
    if (e1 - e0 <= kFew)
      for (int e = e0; e < e1; ++e) in_dst[e] = (int32_t)n;
  }
  for (unsigned long long many = __ballot(e1 - e0 > kFew); many; many &= many - 1) {   // the others' by the wave together
    const int l = __builtin_ctzll(many), a = __shfl(e0, l), z = __shfl(e1, l);
    for (int e = a + lane; e < z; e += 64) in_dst[e] = (int32_t)(n - lane + l);
  }
}
}  // namespace

int xrl_batch_upload(xrl_ctx *c, xrl_batch *b) {
  if (!c || !b) return fail(XRL_ERR_NULL, "xrl_batch_upload: NULL argument");
  if (b->uploaded) return XRL_OK;
  const int Dd = b->model.n_node_dense, De = b->model.d_edge;
  const int64_t N = b->N, E = b->E;
  if (int rc = refuse_capture(c, "xrl_batch_upload")) return rc;
  // the device block: what the host sends, then what the device writes itself
  size_t off = b->send_bytes;
  auto plan = [&](size_t bytes) { size_t o = off; off += align_up(bytes + 16); return o; };
  const bool ed = b->from_edits;
  const size_t o_as = plan(N * 4), o_dst = plan(E * 4), o_ng = plan(N * 4), o_optr = plan((N + 1) * 4), o_opos = plan(E * 4);
  const size_t o_op = ed ? plan(N * 4) : b->o_node_op, o_nd = ed ? plan((size_t)N * Dd * 4) : b->o_node_dense,
               o_ef = ed ? plan((size_t)E * De * 4) : b->o_edge_feat;
  xrl_batch_release_device(b);           // (of an upload that failed)
  char *blk = nullptr;
  xrl_batch_device &d = b->dev;
  // A large batch travels on a stream of its own, so that it arrives while the context's stream is still at
  // work on the batch before. us per step, one stream / two, calls queued back to back: 55 MB 2199 / 1713,
  // 24 MB 2012 / 1496, 14 MB 1768 / 1561; but 6.6 MB 341 / 470 and 4 MB 391 / 536: below 8 MB the hand-over
  // between the streams and the further blocks in rotation cost more than the transfer.
  hipStream_t up = c->stream;
  if (b->mem.pinned && b->send_bytes >= kCopyStreamBytes) {
    if (!c->copy_stream) HIP_TRY(hipStreamCreateWithFlags(&c->copy_stream, hipStreamNonBlocking));
    up = c->copy_stream;
  }
  DeviceBlock got;
  hipError_t e = c->blocks->take(off, up == c->stream, &got);
  if (e != hipSuccess) return fail(XRL_ERR_OOM, "device copy of the batch (%zu bytes): %s", off, hipGetErrorString(e));
  blk = (char *)got.p;
  d.block = blk;
  d.bytes = got.cap;
  d.used = got.used;
  b->pool = c->blocks;
  b->owner = c->id;
  b->shared = false;
  auto queue = [&]() -> int {
    if (up != c->stream && got.used) HIP_TRY(hipStreamWaitEvent(up, got.used, 0));
    HIP_TRY(hipMemcpyAsync(blk, b->mem.p, b->send_bytes, hipMemcpyHostToDevice, up));
    if (N > 0)
      derive_index_kernel<<<dim3((unsigned)((N + 255) / 256)), dim3(256), 0, up>>>(
          (const int32_t *)(blk + b->o_in_ptr), (const int32_t *)(blk + b->o_graph_node_ptr), N, (int)b->G, (int32_t *)(blk + o_as),
          (int32_t *)(blk + o_dst), (int32_t *)(blk + o_ng));
    if (ed) {
      auto expand = [&](size_t o_from, int64_t n, int width, size_t o_base, size_t o_new, size_t o_out) {
        const int64_t total = n * width;
        if (total > 0)
          expand_rows_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, up>>>(
              (const int32_t *)(blk + o_from), n, width, (const uint32_t *)(blk + o_base), (const uint32_t *)(blk + o_new),
              (uint32_t *)(blk + o_out));
      };
      expand(b->o_node_from, N, 1, b->o_base_op, b->o_new_op, o_op);
      expand(b->o_node_from, N, Dd, b->o_base_dense, b->o_new_dense, o_nd);
      expand(b->o_edge_from, E, De, b->o_base_feat, b->o_new_feat, o_ef);
    }
    HIP_TRY(hipGetLastError());
    if (!b->mem.pinned) {                // (read while this call runs, or soon after: wait for it)
      HIP_TRY(hipStreamSynchronize(c->stream));
      return XRL_OK;
    }
    // A pinned block is read after this call returns: an event marks the end of it (and of the kernels
    // above), which the block's next user waits for, and other contexts that are given the batch.
    if (b->mem.copied && b->mem.device != c->device) {
      (void)hipEventDestroy((hipEvent_t)b->mem.copied);
      b->mem.copied = nullptr;
    }
    if (!b->mem.copied) {
      hipEvent_t ev = nullptr;
      HIP_TRY(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
      b->mem.copied = ev;
      b->mem.device = c->device;
    }
    HIP_TRY(hipEventRecord((hipEvent_t)b->mem.copied, up));
    if (up != c->stream) HIP_TRY(hipStreamWaitEvent(c->stream, (hipEvent_t)b->mem.copied, 0));
    return XRL_OK;
  };
  const int rc = queue();
  if (rc) {
    (void)hipStreamSynchronize(up);
    return rc;
  }
  d.state_graph_ptr = (int32_t *)(blk + b->o_state_graph_ptr);
  d.graph_node_ptr = (int32_t *)(blk + b->o_graph_node_ptr);
  d.node_op = (int32_t *)(blk + o_op);
  d.in_ptr = (int32_t *)(blk + b->o_in_ptr);
  d.in_src = (int32_t *)(blk + b->o_in_src);
  d.in_dst = (int32_t *)(blk + o_dst);
  d.out_ptr = (int32_t *)(blk + o_optr);
  d.out_pos = (int32_t *)(blk + o_opos);
  d.node_graph = (int32_t *)(blk + o_ng);
  d.node_dense = (float *)(blk + o_nd);
  d.edge_feat = (float *)(blk + o_ef);
  d.graph_global = (float *)(blk + b->o_graph_global);
  d.mask = (uint8_t *)(blk + b->o_mask);
  d.tile_ptr = (int32_t *)(blk + b->o_tile);
  d.gtile_ptr = b->has_graph_tiles ? (int32_t *)(blk + b->o_gtile) : nullptr;
  d.graph_tile_ptr = b->has_graph_tiles ? (int32_t *)(blk + b->o_graph_tile) : nullptr;
  d.agg_src = (int32_t *)(blk + o_as);
  b->encodes = 0;
  b->forgone_us = 0;
  b->few_alike = false;
  b->out_maker = 0;
  b->uploaded = true;
  return XRL_OK;
}

int xrl_encode(xrl_ctx *c, const xrl_batch *b, float *d_emb, int save_for_backward) {
  int rc = check_batch(c, b, "xrl_encode");
  if (rc) return rc;
  if (!d_emb && b->G > 0) return fail(XRL_ERR_NULL, "xrl_encode: d_emb is NULL");
  if (b->G == 0) return XRL_OK;
  if (*(volatile unsigned *)c->h_fault) {
    // an earlier one-launch encode gave up a wait between its blocks: its embeddings were wrong.
    // Its counters are put back to zero (after everything queued so far) before anything else runs.
    (void)hipStreamSynchronize(c->stream);
    (void)hipMemsetAsync(c->d_arrived, 0, sizeof(unsigned) * kClusterMaxGraphs, c->stream);
    *c->h_fault = 0;
    return fail(XRL_ERR_HIP, "xrl_encode: an earlier xrl_encode on this context did not complete (a wait between the "
                             "blocks of its one-launch form ran out); its embeddings are invalid");
  }
  if (b->owner == c->id && b->encodes >= 0) {
    // Reduced to its distinct nodes when it is first saved for a backward pass, or encoded again (a smaller one: several
    // times): a batch encoded once and forward only would not earn back what finding them takes. Not in a capture, nor
    // once the context has been through one: a reduced batch's buffers may be larger than those it was
    // encoded whole in, and to grow them would free what the graphs write to.
    xrl_batch *mb = const_cast<xrl_batch *>(b);
    if (distinct_pays(c, mb, save_for_backward != 0)) {
      mb->encodes = -1;
      if ((rc = find_distinct(c, mb))) return rc;
    } else if (!save_for_backward && mb->encodes >= 0) {
      ++mb->encodes;
    }
  }
  return c->elem == 2 ? encode_impl<bf16_t>(c, b, d_emb, save_for_backward)
                      : encode_impl<float>(c, b, d_emb, save_for_backward);
}

int xrl_batch_level(xrl_ctx *c, const xrl_batch *b, int32_t level, int64_t counts[4]) {
  const int rc = check_batch(c, b, "xrl_batch_level");
  if (rc) return rc;
  if (!counts) return fail(XRL_ERR_NULL, "xrl_batch_level: counts is NULL");
  if (level < 0 || level > c->m.rounds) return fail(XRL_ERR_INDEX, "xrl_batch_level: level %d outside [0, %d]", level, c->m.rounds);
  if (const Distinct *q = distinct_of(c, b)) {
    const LevelGraph &g = q->lv[level];
    counts[0] = g.N; counts[1] = g.E; counts[2] = g.receivers; counts[3] = g.n_tiles;
    return XRL_OK;
  }
  const int32_t *in_ptr = b->at<int32_t>(b->o_in_ptr);
  counts[0] = b->N; counts[1] = b->E; counts[2] = 0; counts[3] = b->n_tiles;
  for (int64_t n = 0; n < b->N; ++n) counts[2] += in_ptr[n + 1] > in_ptr[n];
  return XRL_OK;
}

int xrl_policy_value(xrl_ctx *c, const xrl_batch *b, const float *d_emb, float *d_logp,
                     float *d_value, float *d_entropy, int32_t *d_action, float *d_logit) {
  int rc = check_batch(c, b, "xrl_policy_value");
  if (rc) return rc;
  if (b->S == 0) return XRL_OK;
  if (!d_emb || !d_logp || !d_value || !d_entropy || !d_action)
    return fail(XRL_ERR_NULL, "xrl_policy_value: NULL device pointer");
  if ((uintptr_t)d_emb & 15) return fail(XRL_ERR_SHAPE, "xrl_policy_value: d_emb must be 16-byte aligned");
  const int H = c->m.hidden;
  rc = ensure_hws(c, align_up((size_t)b->G * 4) + align_up((size_t)b->S * H * 4));
  if (rc) return rc;
  float *logit = d_logit ? d_logit : (float *)c->hws;
  float *zmean = (float *)(c->hws + align_up((size_t)b->G * 4));
  Timed t(c, TK_HEADS);
  return launch_heads(c, b, d_emb, logit, d_logp, d_entropy, d_action, zmean, d_value, nullptr, nullptr, c->d_counter);
}

int xrl_policy_value_static(xrl_ctx *c, const xrl_batch *b, const float *d_emb, float *d_logp,
                            float *d_value, float *d_entropy, int32_t *d_action, float *d_logit) {
  int rc = check_batch(c, b, "xrl_policy_value_static");
  if (rc) return rc;
  if (b->S == 0) return XRL_OK;
  if (!d_emb || !d_logp || !d_value || !d_entropy || !d_action)
    return fail(XRL_ERR_NULL, "xrl_policy_value_static: NULL device pointer");
  if ((uintptr_t)d_emb & 15) return fail(XRL_ERR_SHAPE, "xrl_policy_value_static: d_emb must be 16-byte aligned");
  const int H = c->m.hidden;
  if (b->G > kStaticMaxSlots || b->S * H > kStaticMaxStateFloats)
    return fail(XRL_ERR_UNSUPPORTED,
                "xrl_policy_value_static: %lld slots, %lld states x hidden %d exceed the fixed scratch "
                "(at most %lld slots and %lld state floats)",
                (long long)b->G, (long long)b->S, H, (long long)kStaticMaxSlots, (long long)kStaticMaxStateFloats);
  int32_t *counter = (int32_t *)(c->static_ws + kStaticCounterOff);
  float *logit = d_logit ? d_logit : (float *)(c->static_ws + kStaticLogitOff);
  float *zmean = (float *)(c->static_ws + kStaticZmeanOff);
  // the array keeps the last call's contents: the counters must start at zero
  fill_zero_kernel<<<dim3((unsigned)((b->S + 255) / 256)), dim3(256), 0, c->stream>>>((float *)counter, b->S);
  return launch_heads(c, b, d_emb, logit, d_logp, d_entropy, d_action, zmean, d_value, nullptr, nullptr, counter);
}

int xrl_ppo_objective(xrl_ctx *c, const xrl_batch *b, const float *d_logp, const float *d_value,
                      const float *d_entropy, const int32_t *d_action, const float *d_old_logp,
                      const float *d_advantage, const float *d_v_target, float eps, float c1,
                      float c2, float *d_J, float *d_dlogp, float *d_dvalue, float *d_dentropy) {
  int rc = check_batch(c, b, "xrl_ppo_objective");
  if (rc) return rc;
  if (!d_J) return fail(XRL_ERR_NULL, "xrl_ppo_objective: d_J is NULL");
  if (b->S > 0 && (!d_logp || !d_value || !d_entropy || !d_action || !d_old_logp || !d_advantage ||
                   !d_v_target || !d_dlogp || !d_dvalue || !d_dentropy))
    return fail(XRL_ERR_NULL, "xrl_ppo_objective: NULL device pointer");
  if (b->G > 0)
    fill_zero_kernel<<<dim3((unsigned)((b->G + 255) / 256)), dim3(256), 0, c->stream>>>(d_dlogp, b->G);
  ppo_objective_kernel<<<dim3(1), dim3(256), 0, c->stream>>>(
      d_logp, d_value, d_entropy, b->dev.state_graph_ptr, b->dev.mask, d_action, d_old_logp, d_advantage, d_v_target,
      (int)b->S, eps, c1, c2, d_J, d_dlogp, d_dvalue, d_dentropy);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

}  // extern "C"

namespace {
// user[i] += internal[map[i]]: the real tensors of a single-layer context's internal gradient vector,
// added to the caller's
__global__ void add_mapped_kernel(float *user, const float *internal, const int32_t *map, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) user[i] += internal[map[i]];
}

// Runs a backward pass that adds weight gradients into a vector of the context's own layout: the
// caller's vector itself, or (single-layer contexts) the internal one, zeroed first and folded
// into the caller's afterwards.
template <typename Run>
int with_weight_gradients(xrl_ctx *c, float *d_dweights, Run run) {
  if (!c->single_layer) return run(d_dweights);
  const int64_t n = c->L.total, nu = c->Lu.total;
  fill_zero_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream>>>(c->d_dw_int, n);
  HIP_TRY(hipGetLastError());
  const int rc = run(c->d_dw_int);
  if (rc) return rc;
  add_mapped_kernel<<<dim3((unsigned)((nu + 255) / 256)), dim3(256), 0, c->stream>>>(d_dweights, c->d_dw_int, c->d_wmap, nu);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

int policy_value_backward_run(xrl_ctx *c, const xrl_batch *b, const float *d_emb, const float *d_dlogp,
                              const float *d_dvalue, const float *d_dentropy, float *d_demb, float *d_dweights);
}  // namespace

extern "C" {

int xrl_policy_value_backward(xrl_ctx *c, const xrl_batch *b, const float *d_emb,
                              const float *d_dlogp, const float *d_dvalue,
                              const float *d_dentropy, float *d_demb, float *d_dweights) {
  int rc = check_batch(c, b, "xrl_policy_value_backward");
  if (rc) return rc;
  if (b->S == 0) return XRL_OK;
  if (!d_emb || !d_dlogp || !d_dvalue || !d_dentropy || !d_demb || !d_dweights)
    return fail(XRL_ERR_NULL, "xrl_policy_value_backward: NULL device pointer");
  return with_weight_gradients(c, d_dweights, [&](float *dw) {
    return policy_value_backward_run(c, b, d_emb, d_dlogp, d_dvalue, d_dentropy, d_demb, dw);
  });
}

}  // extern "C"

namespace {
int policy_value_backward_run(xrl_ctx *c, const xrl_batch *b, const float *d_emb, const float *d_dlogp,
                              const float *d_dvalue, const float *d_dentropy, float *d_demb, float *d_dweights) {
  int rc = XRL_OK;
  if ((uintptr_t)d_emb & 15)
    return fail(XRL_ERR_SHAPE, "xrl_policy_value_backward: d_emb must be 16-byte aligned");
  const int H = c->m.hidden, h0 = c->m.head_hidden[0], h1 = c->m.head_hidden[1];
  const int64_t G = b->G, S = b->S;
  size_t need = 0;
  auto acc = [&](size_t n) { need += align_up(n * 4); };
  acc(G); acc(S * H); acc(S);                                         // logit zmean value
  acc(G * h0); acc(G * h1); acc(G);                                   // policy activations
  acc(S * h0); acc(S * h1); acc(S);                                   // value activations
  acc(G); acc(S);                                                     // dlogit, 1/|valid|
  acc(G * h0); acc(G * h1); acc(G);                                   // policy dz
  acc(S * h0); acc(S * h1); acc(S); acc(S * H);                       // value dz, dz_mean
  const size_t spart_floats = small_wgrad_partial_floats(c->L.policy, G) + small_wgrad_partial_floats(c->L.value, S);
  acc(spart_floats);                                                  // chunk partials of the heads' weight gradients
  if ((rc = ensure_hws(c, need))) return rc;
  Bump bump{c->hws};
  float *logit = bump.take<float>(G), *zmean = bump.take<float>(S * H);
  float *value = bump.take<float>(S);
  float *pact[3] = {bump.take<float>(G * h0), bump.take<float>(G * h1), bump.take<float>(G)};
  float *vact[3] = {bump.take<float>(S * h0), bump.take<float>(S * h1), bump.take<float>(S)};
  float *dlogit = bump.take<float>(G), *inv_n = bump.take<float>(S);
  float *pdz[3] = {bump.take<float>(G * h0), bump.take<float>(G * h1), bump.take<float>(G)};
  float *vdz[3] = {bump.take<float>(S * h0), bump.take<float>(S * h1), bump.take<float>(S)};
  float *dzs = bump.take<float>(S * H);
  float *spart = spart_floats ? bump.take<float>(spart_floats) : nullptr;
  const xrl_batch_device &d = b->dev;
  // forward of the heads, keeping every layer's output
  if ((rc = launch_heads(c, b, d_emb, logit, nullptr, nullptr, nullptr, zmean, value, pact, vact, c->d_counter))) return rc;
  // backward: the softmax of each state, both heads' MLPs, then their weight gradients and the slots' share of the mean embedding's gradient
  HeadsSoftmaxBwdArgs sb;
  sb.logit = logit; sb.mask = d.mask; sb.state_graph_ptr = d.state_graph_ptr; sb.dlogp = d_dlogp; sb.dentropy = d_dentropy;
  sb.dlogit = dlogit; sb.inv_valid = inv_n; sb.S = (int)S; sb.states_per_block = value_rows(c, S);
  const int64_t state_blocks = (S + sb.states_per_block - 1) / sb.states_per_block;
  heads_softmax_bwd_kernel<<<dim3((unsigned)state_blocks), dim3(kRowThreads), 0, c->stream>>>(sb);
  HeadsBwdArgs hb;
  hb.value = row_bwd_args(c, c->L.value, false, vact, d_dvalue, S, vdz, dzs);
  hb.policy = row_bwd_args(c, c->L.policy, false, pact, dlogit, G, pdz, d_demb);
  hb.value_rows = sb.states_per_block; hb.value_blocks = (int)state_blocks;
  rc = with_head_widths(c, [&](auto, auto bwd) {
    return launch_rows<heads_backward_kernel<decltype(bwd)>>(kRowBackwardMost, state_blocks + row_blocks(G), row_bwd_lds_floats(hb.policy), c->stream, hb);
  });
  if (rc) return rc;
  const SmallWgradMlp heads[2] = {{&c->L.policy, d_emb, nullptr, H, 0, pact, pdz, G}, {&c->L.value, zmean, nullptr, H, 0, vact, vdz, S}};
  MeanShareArgs mean;
  mean.demb = d_demb; mean.dmean = dzs; mean.inv_valid = inv_n; mean.mask = d.mask; mean.state_graph_ptr = d.state_graph_ptr;
  mean.G = (int)G; mean.S = (int)S; mean.H = H;
  if ((rc = launch_small_wgrads(c, heads, 2, d_dweights, spart, spart_floats, &mean))) return rc;
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}
}  // namespace

extern "C" {

int xrl_encode_backward(xrl_ctx *c, const xrl_batch *b, const float *d_demb, float *d_dweights) {
  int rc = check_batch(c, b, "xrl_encode_backward");
  if (rc) return rc;
  if (b->G == 0) return XRL_OK;
  if (!d_demb || !d_dweights) return fail(XRL_ERR_NULL, "xrl_encode_backward: NULL device pointer");
  if (!c->enc_saved || c->enc_batch != b->id)
    return fail(XRL_ERR_STATE, "xrl_encode_backward: the batch's last xrl_encode did not save for backward");
  return with_weight_gradients(c, d_dweights, [&](float *dw) {
    return c->elem == 2 ? encode_backward_impl<bf16_t>(c, b, d_demb, dw) : encode_backward_impl<float>(c, b, d_demb, dw);
  });
}

int xrl_set_timing(xrl_ctx *c, int enabled) {
  if (!c) return fail(XRL_ERR_NULL, "xrl_set_timing: ctx is NULL");
  c->timing = enabled != 0;
  return XRL_OK;
}

int xrl_read_timing(xrl_ctx *c, const char *kernel, double *total_ms, int64_t *launches) {
  if (!c || !kernel || !total_ms || !launches) return fail(XRL_ERR_NULL, "xrl_read_timing: NULL argument");
  int kind = -1;
  for (int k = 0; k < TK_COUNT; ++k)
    if (!strcmp(kernel, kTimedNames[k])) kind = k;
  if (kind < 0) return fail(XRL_ERR_INDEX, "xrl_read_timing: unknown kernel '%s'", kernel);
  HIP_TRY(hipStreamSynchronize(c->stream));
  double tot = 0.0;
  int64_t n = 0;
  std::vector<xrl_ctx::Span> keep;
  for (const auto &sp : c->spans) {
    if (sp.kind != kind) { keep.push_back(sp); continue; }
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, sp.a, sp.b));
    tot += ms;
    ++n;
    c->free_events.push_back(sp.a);
    c->free_events.push_back(sp.b);
  }
  c->spans.swap(keep);
  *total_ms = tot;
  *launches = n;
  return XRL_OK;
}

namespace {
// 4 independent accumulator tiles per wave, operands never change: nothing but the matrix pipe
__global__ __launch_bounds__(256) void mfma_peak_kernel(float *out, int iters) {
  bf16x8 a = Operand<bf16_t>::zero(), b = Operand<bf16_t>::zero();
  a[threadIdx.x & 7] = (bf16_t)1.0f;
  b[(threadIdx.x >> 3) & 7] = (bf16_t)0.5f;
  f32x16 acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) s += acc[i][r];
  out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}
__global__ __launch_bounds__(256) void copy_peak_kernel(const f32x4 *src, f32x4 *dst, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}
}  // namespace

int xrl_measure_peaks(xrl_ctx *c, int64_t copy_bytes, double *mfma_tflops, double *copy_gbs) {
  if (!c || !mfma_tflops || !copy_gbs) return fail(XRL_ERR_NULL, "xrl_measure_peaks: NULL argument");
  if (copy_bytes < 16) return fail(XRL_ERR_SHAPE, "xrl_measure_peaks: copy_bytes = %lld", (long long)copy_bytes);
  const int64_t n16 = copy_bytes / 16;
  const int blocks = c->n_cu * 4;                              // 16 waves per CU
  char *buf = nullptr;
  hipError_t e = hipMalloc((void **)&buf, (size_t)n16 * 32 + (size_t)blocks * 256 * 4);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(XRL_ERR_OOM, "xrl_measure_peaks: %s", hipGetErrorString(e));
  }
  f32x4 *src = (f32x4 *)buf, *dst = src + n16;
  float *out = (float *)(dst + n16);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = XRL_OK;
  auto run = [&]() -> int {
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    HIP_TRY(hipMemsetAsync(buf, 0, (size_t)n16 * 32, c->stream));
    const int iters = 20000;
    mfma_peak_kernel<<<dim3(blocks), dim3(256), 0, c->stream>>>(out, 100);          // warm-up
    HIP_TRY(hipEventRecord(e0, c->stream));
    mfma_peak_kernel<<<dim3(blocks), dim3(256), 0, c->stream>>>(out, iters);
    HIP_TRY(hipEventRecord(e1, c->stream));
    HIP_TRY(hipEventSynchronize(e1));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
    *mfma_tflops = (double)blocks * 4 * iters * 4 * (2.0 * 32 * 32 * 16) / (ms * 1e-3) / 1e12;
    copy_peak_kernel<<<dim3(c->n_cu * 8), dim3(256), 0, c->stream>>>(src, dst, n16);   // warm-up
    HIP_TRY(hipEventRecord(e0, c->stream));
    for (int i = 0; i < 5; ++i) copy_peak_kernel<<<dim3(c->n_cu * 8), dim3(256), 0, c->stream>>>(src, dst, n16);
    HIP_TRY(hipEventRecord(e1, c->stream));
    HIP_TRY(hipEventSynchronize(e1));
    HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
    *copy_gbs = 5.0 * (double)n16 * 32 / (ms * 1e-3) / 1e9;
    return XRL_OK;
  };
  rc = run();
  (void)hipStreamSynchronize(c->stream);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(buf);
  return rc;
}

int xrl_segment_sum(xrl_ctx *c, const float *d_values, const int32_t *d_ptr, int64_t n_rows,
                    int64_t n_seg, int32_t width, float *d_out) {
  if (!c || !d_ptr || !d_out || (n_rows > 0 && !d_values))
    return fail(XRL_ERR_NULL, "xrl_segment_sum: NULL argument");
  if (n_rows < 0 || n_seg < 0 || width < 4 || width > 256 || width % 4)
    return fail(XRL_ERR_SHAPE, "xrl_segment_sum: n_rows/n_seg negative or width not a multiple of 4 in [4, 256]");
  int rc = ensure_ws(c, align_up(segsum_carry_floats(n_rows, width) * 4));
  if (rc) return rc;
  c->enc_batch = 0;   // the workspace no longer holds an encode's activations
  c->enc_saved = false;
  return launch_segsum<float, float, 4>(c, d_values, nullptr, d_ptr, nullptr, n_rows, n_seg, width, d_out,
                                        (float *)c->ws);
}

int xrl_weight_gradient(xrl_ctx *c, const xrl_batch *b, int32_t kind, const void *d_x, const void *d_x2,
                        const void *d_dZ, int64_t n_rows, float *d_dW, float *d_db) {
  int rc = check_batch(c, b, "xrl_weight_gradient");
  if (rc) return rc;
  if (kind != XRL_WG_PLAIN && kind != XRL_WG_EDGE && kind != XRL_WG_NODE)
    return fail(XRL_ERR_INDEX, "xrl_weight_gradient: unknown kind %d", kind);
  const int H = c->m.hidden, De = c->m.d_edge;
  if (kind == XRL_WG_EDGE) n_rows = b->E;
  if (kind == XRL_WG_NODE) n_rows = b->N;
  if (n_rows < 0) return fail(XRL_ERR_SHAPE, "xrl_weight_gradient: n_rows is negative");
  if (n_rows == 0) return XRL_OK;
  if (!d_x || !d_dZ || !d_dW || !d_db || (kind == XRL_WG_NODE && !d_x2))
    return fail(XRL_ERR_NULL, "xrl_weight_gradient: NULL device pointer");
  const size_t part = wgrad_partial_floats(c);
  if ((rc = ensure_bws(c, align_up(part * 4)))) return rc;
  const xrl_batch_device &d = b->dev;
  WgradQueue q;
  q.partial = (float *)c->bws; q.partial_floats = part;
  WgradJob j = {};
  j.kind = kind == XRL_WG_PLAIN ? WG_PLAIN : (kind == XRL_WG_EDGE ? WG_EDGE : WG_NODE);
  j.A = d_x; j.agg = d_x2; j.Ka = kind == XRL_WG_PLAIN ? H : 2 * H; j.n_rows = n_rows;
  j.src = d.in_src; j.dst = kind == XRL_WG_EDGE ? d.in_dst : d.agg_src; j.edge_feat = d.edge_feat; j.De = De;
  j.dZ = d_dZ; j.dW = d_dW; j.db = d_db;
  auto run = [&](auto tag) -> int {
    using T = decltype(tag);
    const int rc2 = queue_wgrad<T>(c, q, j);
    return rc2 ? rc2 : flush_wgrads<T>(c, q);
  };
  return c->elem == 2 ? run(bf16_t()) : run(float());
}

int xrl_mlp_backward(xrl_ctx *c, const xrl_batch *b, int32_t kind, int32_t round, const void *d_h,
                     const void *d_agg, const void *d_y, const void *d_dy, void *d_z1, void *d_dz1,
                     void *d_dz2, void *d_dxa, void *d_dxb) {
  int rc = check_batch(c, b, "xrl_mlp_backward");
  if (rc) return rc;
  if (c->m.round_kind != XRL_ROUND_MLP) return fail(XRL_ERR_UNSUPPORTED, "xrl_mlp_backward: MLP rounds only");
  if (kind != XRL_WG_EDGE && kind != XRL_WG_NODE) return fail(XRL_ERR_INDEX, "xrl_mlp_backward: unknown kind %d", kind);
  if (round < 0 || round >= c->m.rounds) return fail(XRL_ERR_INDEX, "xrl_mlp_backward: round %d outside [0, %d)", round, c->m.rounds);
  const int64_t rows = kind == XRL_WG_EDGE ? b->E : b->N;
  if (rows == 0) return XRL_OK;
  if (!d_h || !d_dy || !d_z1 || !d_dz1 || !d_dz2 || !d_dxa || !d_dxb || (kind == XRL_WG_NODE && (!d_agg || !d_y)))
    return fail(XRL_ERR_NULL, "xrl_mlp_backward: NULL device pointer");
  const xrl_batch_device &d = b->dev;
  Mlp2BwdArgs a;
  memset(&a, 0, sizeof(a));
  a.De = c->m.d_edge; a.Dd = c->m.n_node_dense;
  a.in_ptr = d.in_ptr; a.in_src = d.in_src; a.in_dst = d.in_dst;
  a.edge_feat = d.edge_feat; a.node_op = d.node_op; a.node_dense = d.node_dense;
  const EncMlp &e = kind == XRL_WG_EDGE ? c->edge[round] : c->node[round];
  a.W1s = e.W1s; a.W2s = e.W2s; a.W2bt = e.W2bt; a.W1bt = e.W1bt; a.b1 = e.b1; a.b2 = e.b2; a.nslab1 = e.nslab1;
  a.n_rows = rows; a.h = d_h; a.agg = d_agg; a.y = d_y; a.dy = d_dy;
  a.z1 = d_z1; a.dz1 = d_dz1; a.dz2 = d_dz2; a.dx_a = d_dxa; a.dx_b = d_dxb;
  const int k = kind == XRL_WG_EDGE ? KIND_EDGE : KIND_NODE;
  return c->elem == 2 ? launch_mlp2_bwd<bf16_t>(c, k, a) : launch_mlp2_bwd<float>(c, k, a);
}

int xrl_get_activation(xrl_ctx *c, const xrl_batch *b, const char *what, int32_t round, float *d_out) {
  int rc = check_batch(c, b, "xrl_get_activation");
  if (rc) return rc;
  if (!what || !d_out) return fail(XRL_ERR_NULL, "xrl_get_activation: NULL argument");
  if (!c->enc_saved || c->enc_batch != b->id)
    return fail(XRL_ERR_STATE, "xrl_get_activation: no saved forward of this batch");
  const int H = c->m.hidden, R = c->m.rounds;
  const int64_t N = b->N, G = b->G;
  const void *src = nullptr;
  int64_t rows = N;
  int D = H;
  bool typed = true;
  const int32_t *row_src = nullptr, *cls = nullptr;   // (a reduced batch: the node's class at the level)
  const Distinct *q = distinct_of(c, b);
  if (!strcmp(what, "a0")) {   // not kept by the forward pass: recomputed with the segment-sum kernel
    return launch_segsum<float, float, 4>(c, b->dev.edge_feat, nullptr, b->dev.in_ptr, b->dev.in_dst, b->E, N,
                                          c->m.d_edge, d_out, c->carry);
  }
  else if (!strcmp(what, "pool")) { src = c->pool; rows = G; typed = false; }
  else if (!strcmp(what, "h")) {
    if (round < 0 || round > R) return fail(XRL_ERR_INDEX, "h: round %d outside [0, %d]", round, R);
    src = c->h[round];
    if (q) cls = q->cls[round];
  } else if (!strcmp(what, "agg")) {
    if (round < 1 || round > R) return fail(XRL_ERR_INDEX, "agg: round %d outside [1, %d]", round, R);
    if (c->m.round_kind == XRL_ROUND_GAT)
      return fail(XRL_ERR_UNSUPPORTED, "agg: the graph-attention rounds keep no received sums");
    src = c->agg[round];
    if (q) cls = q->cls[round];
    if (c->agg_skip) row_src = b->dev.agg_src;   // rows of nodes without in-edges were never written
  } else return fail(XRL_ERR_INDEX, "xrl_get_activation: unknown tensor '%s'", what);
  if (rows * D == 0) return XRL_OK;
  const unsigned blocks = (unsigned)((rows * D + 255) / 256);
  if (typed && c->elem == 2)
    export_rows_kernel<bf16_t><<<dim3(blocks), dim3(256), 0, c->stream>>>((const bf16_t *)src, rows, D, row_src, cls, d_out);
  else
    export_rows_kernel<float><<<dim3(blocks), dim3(256), 0, c->stream>>>((const float *)src, rows, D, row_src, cls, d_out);
  HIP_TRY(hipGetLastError());
  return XRL_OK;
}

}  // extern "C"
