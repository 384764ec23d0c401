// Internal declarations shared by the host-side packer and the device-side runtime.
#pragma once
#include <atomic>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "xrl.h"

namespace xrl {

void set_error(const char *fmt, ...);
int fail(int code, const char *fmt, ...);

// One tensor of the flat weight vector (order documented in xrl.h).
struct WeightTensor {
  std::string name;
  int64_t offset, rows, cols;  // cols == 0 for a bias vector of length rows
};

// Offsets of one MLP inside the flat vector: per layer (W offset, b offset, in, out).
struct MlpRef {
  int n_layers = 0;
  int64_t w[3] = {0, 0, 0}, b[3] = {0, 0, 0};
  int32_t d_in[3] = {0, 0, 0}, d_out[3] = {0, 0, 0};
};

struct Layout {
  std::vector<WeightTensor> tensors;
  int64_t total = 0;
  MlpRef embed, readout, policy, value;
  std::vector<MlpRef> edge, node;  // per round (XRL_ROUND_MLP)
  struct GatRef { int64_t W = 0, a_src = 0, a_dst = 0; };
  std::vector<GatRef> gat;         // per round (XRL_ROUND_GAT)
};

// Validates the dimensions that every part of the library relies on (positive widths, ...)
// and fills the layout. Returns XRL_OK or an error code (message set).
int build_layout(const xrl_model_desc &m, Layout &out);

}  // namespace xrl

// Allocator whose resize() leaves new trivially-constructible elements uninitialised: the packed
// arrays are written in full by the packing threads, which then also take their page faults.
template <typename T>
struct RawAlloc : std::allocator<T> {
  template <typename U> struct rebind { typedef RawAlloc<U> other; };
  RawAlloc() = default;
  template <typename U> RawAlloc(const RawAlloc<U> &) {}
  template <typename U> void construct(U *p) { ::new ((void *)p) U; }              // default-init: no write
  template <typename U, typename... A> void construct(U *p, A &&...a) { ::new ((void *)p) U(std::forward<A>(a)...); }
};
template <typename T> using RawVec = std::vector<T, RawAlloc<T>>;

// Device-side copies of a packed batch (all owned by one hipMalloc block).
struct xrl_batch_device {
  void *block = nullptr;
  size_t bytes = 0;
  void *used = nullptr;   // event behind the block's last use before this batch, then behind the making of the sender index
  int32_t *state_graph_ptr = nullptr, *graph_node_ptr = nullptr, *node_op = nullptr;
  int32_t *in_ptr = nullptr, *in_src = nullptr, *in_dst = nullptr;
  int32_t *out_ptr = nullptr, *out_pos = nullptr, *node_graph = nullptr, *tile_ptr = nullptr;
  int32_t *gtile_ptr = nullptr, *graph_tile_ptr = nullptr;   // null unless the batch has per-graph tiles
  int32_t *agg_src = nullptr;   // [N] n for a node with in-edges, -1 for one without (filled on the device)
  float *node_dense = nullptr, *edge_feat = nullptr, *graph_global = nullptr;
  uint8_t *mask = nullptr;
};

// Host memory of one packed batch. While a context is alive it is pinned (the upload is then one
// transfer at the link's rate) and comes from a bounded pool, so that a program that packs a state
// per step pays neither for page faults nor for pinning; otherwise it is ordinary memory.
struct HostBlock {
  char *p = nullptr;
  size_t cap = 0;
  bool pinned = false;
  int device = -1;          // device of `copied`
  void *copied = nullptr;   // event behind the last transfer out of the block (pinned blocks)
};
// Implemented in the device translation unit. host_block_take leaves p null when memory ran out.
HostBlock host_block_take(size_t bytes);
void host_block_give(HostBlock &b);

struct Distinct;            // the batch's graphs reduced to distinct nodes (device translation unit)
struct DevicePool;          // idle device blocks of one context (device translation unit)

// Host copies, for views, of arrays that packing does not write.
struct PackedArrays {
  RawVec<int32_t> in_dst, out_ptr, out_pos, node_graph;
  RawVec<float> edge_feat;                     // of a batch packed from edits
};

// The packed arrays lie in one host block, those the device needs first and in the device's layout:
// array i of the device block is at the same offset in both. Behind them, in the host block, in_eid;
// in the device block, the arrays that the device writes itself: receivers, the nodes' graphs and
// (for a backward pass) the sender index follow from the others, and are neither packed nor sent.
struct xrl_batch {
  xrl_model_desc model;
  int64_t S = 0, G = 0, N = 0, E = 0;
  int32_t max_slots = 0;  // largest number of slots in one state
  HostBlock mem;
  size_t send_bytes = 0;  // transferred to the device
  size_t o_state_graph_ptr = 0, o_graph_node_ptr = 0, o_in_ptr = 0, o_node_op = 0, o_in_src = 0, o_node_dense = 0,
         o_edge_feat = 0, o_graph_global = 0, o_mask = 0, o_tile = 0, o_gtile = 0, o_graph_tile = 0, o_in_eid = 0;
  template <typename T> T *at(size_t off) const { return (T *)(mem.p + off); }
  int64_t n_tiles = 0;            // edge tiles of the message kernels (see the packer): [n_tiles + 1] at o_tile
  int64_t n_split_tiles = 0;      // tiles that end inside a receiver's in-edge range
  // Per-graph edge tiles for the one-launch encoder of small batches: the same cutting rule, but
  // a tile never spans two graphs; graph g owns tiles [graph_tile_ptr[g], graph_tile_ptr[g + 1])
  // of gtile_ptr. Absent when the batch has more than kGraphTileMaxGraphs graphs or a node
  // with more than 32 in-edges.
  bool has_graph_tiles = false;
  int64_t n_graph_tiles = 0;
  int32_t max_graph_nodes = 0;    // nodes of the largest graph
  int32_t max_graph_tiles = 0;    // most per-graph edge tiles of one graph
  // Batches packed from edits (xrl_pack_state_edits): where each node's and each receiver-order
  // edge's attributes come from -- an index into the current graphs' arrays (>= 0) or, as -1 - k,
  // into the new nodes' / edges' arrays -- and those compact attribute arrays. Such a batch has no
  // node_op, node_dense and edge_feat on the host (xrl_batch_host_view writes the last on demand).
  bool from_edits = false;
  size_t o_node_from = 0, o_edge_from = 0, o_base_op = 0, o_new_op = 0, o_base_dense = 0, o_new_dense = 0,
         o_base_feat = 0, o_new_feat = 0;
  std::atomic<PackedArrays *> view{nullptr};   // made by the first xrl_batch_host_view
  xrl_batch_device dev;
  bool uploaded = false;
  std::mutex out_mu;                       // of the sender index on the device:
  uint64_t out_maker = 0;                  // the context that made it, 0: none yet (dev.used then marks the end of that)
  // the context that uploaded it: its other users wait for its transfer, and a device block that only it
  // has used goes back to its pool (reuse on the same stream is ordered), any other is freed
  uint64_t owner = 0;
  std::shared_ptr<DevicePool> pool;
  std::shared_ptr<Distinct> distinct;      // used by the owner only
  int encodes = 0;                         // the owner's calls of xrl_encode, until the batch is looked at for it
  double forgone_us = 0;                   // what they would have taken less, by an estimate, had it been reduced before
  std::atomic<bool> few_alike{false};      // its distinct nodes have been counted: too many of them
  std::atomic<bool> shared{false};
  uint64_t id = 0;  // unique per packed batch; ties saved activations to their batch
  xrl_batch() = default;
  xrl_batch(const xrl_batch &) = delete;
  ~xrl_batch() {
    host_block_give(mem);
    delete view.load();
  }
};

constexpr int64_t kGraphTileMaxGraphs = 4096;

// Implemented in the device translation unit; gives dev.block back if there is one.
extern "C" void xrl_batch_release_device(xrl_batch *b);
