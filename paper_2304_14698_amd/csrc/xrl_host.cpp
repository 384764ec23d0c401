// Host side of the library: weight layout, validation and packing of states into the
// receiver-sorted meta-batch. Nothing in this file calls the GPU runtime.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <system_error>
#include <thread>

#include "xrl_internal.h"

namespace xrl {

static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}

int fail(int code, const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

static void add_mlp(Layout &L, MlpRef &ref, const std::string &prefix, int d_in,
                    const std::vector<int> &widths) {
  ref.n_layers = (int)widths.size();
  int d = d_in;
  for (size_t i = 0; i < widths.size(); ++i) {
    int w = widths[i];
    ref.d_in[i] = d;
    ref.d_out[i] = w;
    ref.w[i] = L.total;
    L.tensors.push_back({prefix + ".W" + std::to_string(i), L.total, d, w});
    L.total += (int64_t)d * w;
    ref.b[i] = L.total;
    L.tensors.push_back({prefix + ".b" + std::to_string(i), L.total, w, 0});
    L.total += w;
    d = w;
  }
}

int build_layout(const xrl_model_desc &m, Layout &L) {
  if (m.n_op_types < 1 || m.n_node_dense < 0 || m.d_edge < 1 || m.d_global < 0 || m.hidden < 1 ||
      m.rounds < 0 || m.mlp_layers < 1 || m.mlp_layers > 3 || m.head_hidden[0] < 1 ||
      m.head_hidden[1] < 1)
    return fail(XRL_ERR_SHAPE, "model: non-positive or out-of-range dimension");
  if (m.n_op_types > 4096 || m.n_node_dense > 4096 || m.d_edge > 4096 || m.d_global > 4096 ||
      m.hidden > 4096 || m.rounds > 1024 || m.head_hidden[0] > 4096 || m.head_hidden[1] > 4096)
    return fail(XRL_ERR_SHAPE, "model: dimension above 4096 (rounds above 1024)");
  if (m.readout != XRL_READOUT_SUM && m.readout != XRL_READOUT_MEAN)
    return fail(XRL_ERR_SHAPE, "model: readout must be XRL_READOUT_SUM or XRL_READOUT_MEAN");
  if (m.precision != XRL_PREC_FP32 && m.precision != XRL_PREC_BF16)
    return fail(XRL_ERR_SHAPE, "model: precision must be XRL_PREC_FP32 or XRL_PREC_BF16");
  if (m.round_kind != XRL_ROUND_MLP && m.round_kind != XRL_ROUND_GAT)
    return fail(XRL_ERR_SHAPE, "model: round_kind must be XRL_ROUND_MLP or XRL_ROUND_GAT");
  L = Layout();
  const int H = m.hidden;
  std::vector<int> enc(m.mlp_layers, H);
  add_mlp(L, L.embed, "embed", m.d_edge + m.n_op_types + m.n_node_dense, enc);
  if (m.round_kind == XRL_ROUND_GAT) {
    L.gat.resize(m.rounds);
    for (int r = 0; r < m.rounds; ++r) {
      const std::string p = "gat" + std::to_string(r);
      L.gat[r].W = L.total;
      L.tensors.push_back({p + ".W", L.total, H, H});
      L.total += (int64_t)H * H;
      L.gat[r].a_src = L.total;
      L.tensors.push_back({p + ".a_src", L.total, H, 0});
      L.total += H;
      L.gat[r].a_dst = L.total;
      L.tensors.push_back({p + ".a_dst", L.total, H, 0});
      L.total += H;
    }
  } else {
    L.edge.resize(m.rounds);
    L.node.resize(m.rounds);
    for (int r = 0; r < m.rounds; ++r) {
      add_mlp(L, L.edge[r], "edge" + std::to_string(r), 2 * H + m.d_edge, enc);
      add_mlp(L, L.node[r], "node" + std::to_string(r), 2 * H, enc);
    }
  }
  add_mlp(L, L.readout, "readout", H + m.d_global, enc);
  std::vector<int> head = {m.head_hidden[0], m.head_hidden[1], 1};
  add_mlp(L, L.policy, "policy", H, head);
  add_mlp(L, L.value, "value", H, head);
  return XRL_OK;
}

}  // namespace xrl

using namespace xrl;

namespace {
// Packing works graph by graph (a graph's nodes, and its edges in receiver order, occupy the same
// index ranges before and after), so large batches are cut into contiguous graph ranges of about
// equal nodes + edges, one per thread. XRL_PACK_THREADS overrides the thread count (1 = serial).
struct PackIssue {
  int code = 0;
  char msg[200] = "";
  void set(int c, const char *fmt, ...) {
    if (code) return;                                   // keep the first one of this range
    code = c;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(msg, sizeof(msg), fmt, ap);
    va_end(ap);
  }
};

int pack_thread_count(int64_t work) {
  if (const char *e = getenv("XRL_PACK_THREADS")) {
    const int v = atoi(e);
    if (v >= 1) return v > 64 ? 64 : v;
  }
  int hw = (int)std::thread::hardware_concurrency();
  if (hw < 1) hw = 1;
  // About 4.5 ns per node or edge against 12 us to start a thread: the best number is the square root of
  // their quotient. Measured, one thread / the best number / what this picks, us: 36 k nodes and edges
  // 154 / 125 / 125, 152 k 451 / 163 / 163, 620 k 3640 / 822 / 880; at 1.4 M (8.3 / 1.9 / 1.9 ms) eight
  // threads already take what the memory gives.
  if (hw > 12) hw = 12;
  const int t = (int)std::sqrt((double)work / 4096.0);
  return t < 1 ? 1 : (t > hw ? hw : t);
}

// graph range boundaries [T + 1], balanced by nodes + edges
std::vector<int64_t> graph_ranges(const xrl_state_desc *st, int64_t G, int T) {
  std::vector<int64_t> cut(T + 1, G);
  cut[0] = 0;
  const int64_t total = (int64_t)st->graph_node_ptr[G] + st->graph_edge_ptr[G];
  int64_t g = 0;
  for (int t = 1; t < T; ++t) {
    const int64_t want = total * t / T;
    while (g < G && (int64_t)st->graph_node_ptr[g] + st->graph_edge_ptr[g] < want) ++g;
    cut[t] = g;
  }
  return cut;
}

// fn(t, g_begin, g_end) for every range; returns false if a range ran out of memory. Ranges whose
// thread cannot be started run on the calling thread.
template <typename F>
bool run_ranges(const std::vector<int64_t> &cut, F fn) {
  const int T = (int)cut.size() - 1;
  std::atomic<bool> ok{true};
  auto guarded = [&](int t) {
    try {
      fn(t, cut[t], cut[t + 1]);
    } catch (const std::bad_alloc &) {
      ok = false;
    }
  };
  std::vector<std::thread> th;
  th.reserve(T > 1 ? T - 1 : 0);
  int started = 1;
  for (; started < T; ++started) {
    try {
      th.emplace_back(guarded, started);
    } catch (const std::system_error &) {
      break;
    }
  }
  guarded(0);
  for (int t = started; t < T; ++t) guarded(t);
  for (auto &x : th) x.join();
  return ok;
}

// Edge tiles of the message kernels: consecutive receiver-order edges, at most 32 per tile, cut at
// receiver boundaries so that a receiver's in-edges share a tile. Only a receiver with more than
// 32 in-edges is split (into full tiles plus a remainder that later receivers may join); its
// pieces are recombined by the carry fix-up. cut_tiles goes over the receivers
// [n0, n1), whose edges begin at `first`, with `fill` edges in the open tile, appends the first edge of
// every tile it opens and returns the edges in the tile open at the end.
struct TileCut {
  std::vector<int32_t> starts;
  int64_t n_split = 0;
  int32_t fill = 0;
};
int32_t cut_tiles(const int32_t *in_ptr, int64_t n0, int64_t n1, int32_t first, int32_t fill, TileCut &out) {
  for (int64_t n = n0; n < n1; ++n) {
    const int32_t end = in_ptr[n + 1];
    if (first == end) continue;
    if (fill == 0 || fill + (end - first) > 32) {
      out.starts.push_back(first);
      fill = 0;
    }
    while (end - first > 32) {          // fill == 0 here
      first += 32;
      out.starts.push_back(first);
      out.n_split++;
    }
    fill += end - first;
    first = end;
  }
  return fill;
}

// Ranges of nodes are cut on separate threads, each as if a tile began with it (spec). The real entry
// state of a range is known once the ranges before it are joined: they are cut again from there until a
// tile begins where one of the speculative cut does -- usually a few tiles in -- and from that tile
// on the two are the same.
void join_tiles(const int32_t *in_ptr, int64_t n0, int64_t n1, const TileCut &spec, int32_t *tiles, int64_t &nt,
                int32_t &fill, int64_t &n_split) {
  size_t k = 0;                          // next speculative start not passed yet
  for (int64_t n = n0; n < n1; ++n) {
    const int32_t first = in_ptr[n], end = in_ptr[n + 1];
    if (first == end) continue;
    const bool opens = fill == 0 || fill + (end - first) > 32;
    if (opens) {
      while (k < spec.starts.size() && spec.starts[k] < first) ++k;
      if (k < spec.starts.size() && spec.starts[k] == first) {
        // (a split receiver's pieces begin at its first edge in both, so its splits lie on one side)
        const size_t rest = spec.starts.size() - k;
        memcpy(tiles + nt, spec.starts.data() + k, sizeof(int32_t) * rest);
        nt += (int64_t)rest;
        for (int64_t q = n; spec.n_split > 0 && q < n1; ++q)
          if (in_ptr[q + 1] - in_ptr[q] > 32) n_split += (in_ptr[q + 1] - in_ptr[q] - 1) / 32;
        fill = spec.fill;
        return;
      }
    }
    TileCut one;
    fill = cut_tiles(in_ptr, n, n + 1, first, fill, one);
    for (int32_t st : one.starts) tiles[nt++] = st;
    n_split += one.n_split;
  }
}

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// Offsets of the packed arrays; every array is followed by at least 16 bytes of slack (the
// kernels' 16-byte loads of a last, partial piece). Upper bounds for the tile tables: two neighbouring
// tiles hold more than 32 edges together.
struct BlockPlan {
  size_t off = 0;
  size_t take(size_t bytes) {
    const size_t o = off;
    off += align_up(bytes + 16);
    return o;
  }
};
bool plan_block(xrl_batch *b, int64_t Nc = 0, int64_t Ec = 0, int64_t n_an = 0, int64_t n_ae = 0) {
  const size_t S = b->S, G = b->G, N = b->N, E = b->E;
  const size_t Dd = b->model.n_node_dense, De = b->model.d_edge, Dg = b->model.d_global;
  const bool ed = b->from_edits;
  BlockPlan p;
  b->o_state_graph_ptr = p.take((S + 1) * 4);
  b->o_graph_node_ptr = p.take((G + 1) * 4);
  b->o_in_ptr = p.take((N + 1) * 4);
  b->o_in_src = p.take(E * 4);
  b->o_graph_global = p.take(G * Dg * 4);
  b->o_mask = p.take(G);
  if (ed) {
    b->o_node_from = p.take(N * 4);
    b->o_edge_from = p.take(E * 4);
    b->o_base_op = p.take((size_t)Nc * 4);
    b->o_new_op = p.take((size_t)n_an * 4);
    b->o_base_dense = p.take((size_t)Nc * Dd * 4);
    b->o_new_dense = p.take((size_t)n_an * Dd * 4);
    b->o_base_feat = p.take((size_t)Ec * De * 4);
    b->o_new_feat = p.take((size_t)n_ae * De * 4);
  } else {
    b->o_node_op = p.take(N * 4);
    b->o_node_dense = p.take(N * Dd * 4);
    b->o_edge_feat = p.take(E * De * 4);
  }
  const bool gt = b->G <= kGraphTileMaxGraphs;
  b->o_tile = p.take((E / 16 + 4) * 4);
  b->o_gtile = p.take(gt ? (E / 16 + 2 * G + 4) * 4 : 0);
  b->o_graph_tile = p.take(gt ? (G + 1) * 4 : 0);
  b->send_bytes = p.off;
  b->o_in_eid = p.take(E * 4);
  b->mem = host_block_take(p.off);
  return b->mem.p != nullptr;
}

// What the packing threads find out about their graphs, besides the arrays they write.
struct RangeTiles {
  TileCut cut;                           // edge tiles of the range's nodes
  TileCut graphs;                        // per-graph edge tiles, one graph after the other
  std::vector<int32_t> graph_end;        // tiles of the range up to and with each of its graphs
  int32_t max_nodes = 0, max_tiles = 0;
};
// (the entries of in_ptr past gnp[g0] are written; that one is another thread's, so its value is given)
void range_tiles(const int32_t *in_ptr, const int32_t *gnp, int64_t g0, int64_t g1, int32_t first, bool per_graph,
                 RangeTiles &r) {
  r.cut.fill = cut_tiles(in_ptr, gnp[g0], gnp[g1], first, 0, r.cut);
  for (int64_t g = g0; g < g1; ++g) {
    r.max_nodes = std::max(r.max_nodes, gnp[g + 1] - gnp[g]);
    if (!per_graph) continue;
    const size_t before = r.graphs.starts.size();
    cut_tiles(in_ptr, gnp[g], gnp[g + 1], first, 0, r.graphs);
    if (gnp[g + 1] > gnp[g]) first = in_ptr[gnp[g + 1]];
    r.max_tiles = std::max(r.max_tiles, (int32_t)(r.graphs.starts.size() - before));
    r.graph_end.push_back((int32_t)r.graphs.starts.size());
  }
}
void join_range_tiles(xrl_batch *b, const std::vector<int64_t> &cut, const std::vector<RangeTiles> &rt) {
  const int32_t *in_ptr = b->at<int32_t>(b->o_in_ptr), *gnp = b->at<int32_t>(b->o_graph_node_ptr);
  int32_t *tiles = b->at<int32_t>(b->o_tile);
  int64_t nt = 0;
  int32_t fill = 0;
  b->n_split_tiles = 0;
  for (size_t t = 0; t < rt.size(); ++t)
    join_tiles(in_ptr, gnp[cut[t]], gnp[cut[t + 1]], rt[t].cut, tiles, nt, fill, b->n_split_tiles);
  b->n_tiles = nt;
  if (nt == 0) tiles[0] = 0;             // (no edges: one entry, no tile)
  else tiles[nt] = (int32_t)b->E;
  b->max_graph_nodes = 0;
  b->max_graph_tiles = 0;
  for (const RangeTiles &r : rt) {
    b->max_graph_nodes = std::max(b->max_graph_nodes, r.max_nodes);
    b->max_graph_tiles = std::max(b->max_graph_tiles, r.max_tiles);
  }
  b->has_graph_tiles = b->G <= kGraphTileMaxGraphs && b->n_split_tiles == 0;
  b->n_graph_tiles = 0;
  if (!b->has_graph_tiles) {
    b->max_graph_tiles = 0;
    return;
  }
  int32_t *gt = b->at<int32_t>(b->o_gtile), *gtp = b->at<int32_t>(b->o_graph_tile);
  int64_t n = 0, g = 0;
  gtp[g++] = 0;
  for (const RangeTiles &r : rt) {
    if (!r.graphs.starts.empty()) memcpy(gt + n, r.graphs.starts.data(), sizeof(int32_t) * r.graphs.starts.size());
    for (int32_t e : r.graph_end) gtp[g++] = (int32_t)n + e;
    n += (int64_t)r.graphs.starts.size();
  }
  b->n_graph_tiles = n;
  gt[n] = (int32_t)b->E;
}
}  // namespace

extern "C" {

const char *xrl_last_error(void) { return g_err; }
const char *xrl_version(void) { return "xrl 0.1 (gfx950)"; }

int64_t xrl_weight_count(const xrl_model_desc *model) {
  if (!model) return fail(XRL_ERR_NULL, "xrl_weight_count: model is NULL");
  Layout L;
  int rc = build_layout(*model, L);
  return rc ? rc : L.total;
}

int32_t xrl_weight_tensor_count(const xrl_model_desc *model) {
  if (!model) return fail(XRL_ERR_NULL, "xrl_weight_tensor_count: model is NULL");
  Layout L;
  int rc = build_layout(*model, L);
  return rc ? rc : (int32_t)L.tensors.size();
}

int xrl_weight_tensor(const xrl_model_desc *model, int32_t index, char *name, size_t name_cap,
                      int64_t *offset, int64_t *rows, int64_t *cols) {
  if (!model) return fail(XRL_ERR_NULL, "xrl_weight_tensor: model is NULL");
  Layout L;
  int rc = build_layout(*model, L);
  if (rc) return rc;
  if (index < 0 || index >= (int32_t)L.tensors.size())
    return fail(XRL_ERR_INDEX, "xrl_weight_tensor: index %d outside [0, %zu)", index,
                L.tensors.size());
  const WeightTensor &t = L.tensors[index];
  if (name && name_cap) {
    strncpy(name, t.name.c_str(), name_cap - 1);
    name[name_cap - 1] = 0;
  }
  if (offset) *offset = t.offset;
  if (rows) *rows = t.rows;
  if (cols) *cols = t.cols;
  return XRL_OK;
}

static int check_ptr(const int32_t *p, int64_t n, const char *what) {
  if (p[0] != 0) return fail(XRL_ERR_SHAPE, "%s[0] = %d, must be 0", what, p[0]);
  for (int64_t i = 0; i < n; ++i)
    if (p[i + 1] < p[i])
      return fail(XRL_ERR_SHAPE, "%s decreases at %lld (%d -> %d)", what, (long long)i, p[i],
                  p[i + 1]);
  return XRL_OK;
}

static bool all_finite(const float *p, int64_t n, int64_t *where) {
  constexpr int64_t kPiece = 4096;                   // (no early exit inside a piece: vector code)
  for (int64_t i = 0; i < n; i += kPiece) {
    const int64_t k = std::min(kPiece, n - i);
    uint32_t bad = 0;
    for (int64_t j = 0; j < k; ++j) {
      uint32_t u;
      memcpy(&u, p + i + j, 4);
      bad |= (uint32_t)((u & 0x7f800000u) == 0x7f800000u);
    }
    if (!bad) continue;
    *where = i;
    while (std::isfinite(p[*where])) ++*where;
    return false;
  }
  return true;
}

// The first of n operator ids outside [0, limit), or n.
static int64_t first_outside(const int32_t *p, int64_t n, int32_t limit) {
  uint32_t bad = 0;
  for (int64_t i = 0; i < n; ++i) bad |= (uint32_t)((uint32_t)p[i] >= (uint32_t)limit);
  if (!bad) return n;
  int64_t i = 0;
  while ((uint32_t)p[i] < (uint32_t)limit) ++i;
  return i;
}

int xrl_pack_state(const xrl_model_desc *model, const xrl_state_desc *st, xrl_batch **out) {
  if (!model || !st || !out) return fail(XRL_ERR_NULL, "xrl_pack_state: NULL argument");
  *out = nullptr;
  Layout L;
  int rc = build_layout(*model, L);
  if (rc) return rc;
  const int64_t S = st->n_states;
  if (S < 0) return fail(XRL_ERR_SHAPE, "n_states = %lld is negative", (long long)S);
  if (!st->state_graph_ptr || !st->graph_node_ptr || !st->graph_edge_ptr || !st->slot_mask)
    return fail(XRL_ERR_NULL, "xrl_pack_state: a ptr array or slot_mask is NULL");
  if ((rc = check_ptr(st->state_graph_ptr, S, "state_graph_ptr"))) return rc;
  const int64_t G = st->state_graph_ptr[S];
  for (int64_t s = 0; s < S; ++s)
    if (st->state_graph_ptr[s + 1] == st->state_graph_ptr[s])
      return fail(XRL_ERR_SHAPE, "state %lld has no graph (needs its current graph)", (long long)s);
  if ((rc = check_ptr(st->graph_node_ptr, G, "graph_node_ptr"))) return rc;
  if ((rc = check_ptr(st->graph_edge_ptr, G, "graph_edge_ptr"))) return rc;
  const int64_t N = st->graph_node_ptr[G], E = st->graph_edge_ptr[G];
  const int Dd = model->n_node_dense, De = model->d_edge, Dg = model->d_global;
  if (N > 0 && (!st->node_op || (Dd > 0 && !st->node_dense)))
    return fail(XRL_ERR_NULL, "node_op or node_dense is NULL");
  if (E > 0 && (!st->edge_src || !st->edge_dst || !st->edge_feat))
    return fail(XRL_ERR_NULL, "edge_src, edge_dst or edge_feat is NULL");
  for (int64_t s = 0; s < S; ++s)
    if (st->slot_mask[st->state_graph_ptr[s]] == 0)
      return fail(XRL_ERR_MASK, "state %lld masks its No-Op slot (its first graph)", (long long)s);
  xrl_batch *b = new (std::nothrow) xrl_batch();
  if (!b) return fail(XRL_ERR_OOM, "xrl_pack_state: out of host memory");
  // One pass of the packing threads over their graphs. Checks first, reported in the order a serial pass
  // would find them: operator ids, edge endpoints, node attributes, edge attributes; within a
  // kind, the lowest range first.
  try {
    static std::atomic<uint64_t> next_id{1};
    b->id = next_id++;
    b->model = *model;
    b->S = S; b->G = G; b->N = N; b->E = E;
    if (!plan_block(b)) throw std::bad_alloc();
    int32_t *gnp = b->at<int32_t>(b->o_graph_node_ptr), *in_ptr = b->at<int32_t>(b->o_in_ptr);
    int32_t *node_op = b->at<int32_t>(b->o_node_op);
    int32_t *in_src = b->at<int32_t>(b->o_in_src), *in_eid = b->at<int32_t>(b->o_in_eid);
    float *node_dense = b->at<float>(b->o_node_dense), *edge_feat = b->at<float>(b->o_edge_feat);
    memcpy(b->at<int32_t>(b->o_state_graph_ptr), st->state_graph_ptr, sizeof(int32_t) * (S + 1));
    memcpy(gnp, st->graph_node_ptr, sizeof(int32_t) * (G + 1));
    in_ptr[0] = 0;
    const int T = pack_thread_count(N + E);
    const std::vector<int64_t> cut = graph_ranges(st, G, T);
    std::vector<PackIssue> issue((size_t)4 * T);
    std::vector<RangeTiles> rt(T);
    const bool done = run_ranges(cut, [&](int t, int64_t g0, int64_t g1) {
      const int64_t n0 = st->graph_node_ptr[g0], n1 = st->graph_node_ptr[g1];
      const int64_t e0 = st->graph_edge_ptr[g0], e1 = st->graph_edge_ptr[g1];
      const int64_t op = n1 > n0 ? n0 + first_outside(st->node_op + n0, n1 - n0, model->n_op_types) : n1;
      if (op < n1)
        issue[0 * T + t].set(XRL_ERR_INDEX, "node %lld: op id %d outside [0, %d)", (long long)op, st->node_op[op],
                             model->n_op_types);
      for (int64_t g = g0; g < g1 && !issue[1 * T + t].code; ++g) {
        const int32_t n = st->graph_node_ptr[g + 1] - st->graph_node_ptr[g];
        const int64_t a = st->graph_edge_ptr[g], z = st->graph_edge_ptr[g + 1];
        if (a == z) continue;
        const int64_t e = a + std::min(first_outside(st->edge_src + a, z - a, n), first_outside(st->edge_dst + a, z - a, n));
        if (e < z)
          issue[1 * T + t].set(XRL_ERR_INDEX, "edge %lld of graph %lld: endpoint (%d -> %d) outside [0, %d)",
                               (long long)e, (long long)g, st->edge_src[e], st->edge_dst[e], n);
      }
      int64_t where = 0;
      if (Dd > 0 && !all_finite(st->node_dense + n0 * Dd, (n1 - n0) * Dd, &where))
        issue[2 * T + t].set(XRL_ERR_VALUE, "node_dense[%lld] is not finite", (long long)(n0 * Dd + where));
      if (!all_finite(st->edge_feat + e0 * De, (e1 - e0) * De, &where))
        issue[3 * T + t].set(XRL_ERR_VALUE, "edge_feat[%lld] is not finite", (long long)(e0 * De + where));
      for (int k = 0; k < 4; ++k)
        if (issue[k * T + t].code) return;
      if (n1 > n0) {
        memcpy(node_op + n0, st->node_op + n0, sizeof(int32_t) * (n1 - n0));
        if (Dd > 0) memcpy(node_dense + n0 * Dd, st->node_dense + n0 * Dd, sizeof(float) * (n1 - n0) * Dd);
        memset(in_ptr + n0 + 1, 0, sizeof(int32_t) * (n1 - n0));
      }
      // Receiver order: stable counting sort of each graph's edges by receiver. A graph's edges keep the index
      // range they came with, so the graph ranges are independent.
      std::vector<int32_t> cur;
      for (int64_t g = g0; g < g1; ++g) {
        const int32_t base = st->graph_node_ptr[g], n = st->graph_node_ptr[g + 1] - base;
        const int64_t a = st->graph_edge_ptr[g], z = st->graph_edge_ptr[g + 1];
        int32_t *inp = in_ptr + base + 1;                 // counts, then ends
        for (int64_t e = a; e < z; ++e) inp[st->edge_dst[e]]++;
        if (cur.size() < (size_t)n) cur.resize((size_t)n);
        int32_t ri = (int32_t)a;
        for (int32_t i = 0; i < n; ++i) {
          cur[i] = ri;                                    // first position of node i's in-edges
          ri += inp[i];
          inp[i] = ri;
        }
        auto place = [&](auto width) {
          constexpr size_t kRow = sizeof(float) * decltype(width)::value;      // 0: any width
          for (int64_t e = a; e < z; ++e) {
            const int32_t p = cur[st->edge_dst[e]]++;
            in_src[p] = base + st->edge_src[e];
            in_eid[p] = (int32_t)e;
            memcpy(edge_feat + (size_t)p * De, st->edge_feat + (size_t)e * De, kRow ? kRow : sizeof(float) * De);
          }
        };
        if (De == 8) place(std::integral_constant<int, 8>());
        else if (De == 4) place(std::integral_constant<int, 4>());
        else place(std::integral_constant<int, 0>());
      }
      range_tiles(in_ptr, gnp, g0, g1, (int32_t)e0, G <= kGraphTileMaxGraphs, rt[t]);
    });
    if (!done) throw std::bad_alloc();
    int code = 0;
    for (const PackIssue &is : issue)
      if (is.code && !code) code = fail(is.code, "%s", is.msg);
    int64_t bad = 0;
    if (!code && st->graph_global && !all_finite(st->graph_global, G * Dg, &bad))
      code = fail(XRL_ERR_VALUE, "graph_global[%lld] is not finite", (long long)bad);
    if (code) {
      delete b;
      return code;
    }
    uint8_t *mask = b->at<uint8_t>(b->o_mask);
    for (int64_t g = 0; g < G; ++g) mask[g] = st->slot_mask[g] ? 1 : 0;
    float *gg = b->at<float>(b->o_graph_global);
    if (st->graph_global && G * Dg > 0) memcpy(gg, st->graph_global, sizeof(float) * G * Dg);
    else memset(gg, 0, sizeof(float) * (size_t)(G * Dg));
    for (int64_t s = 0; s < S; ++s) {
      int32_t c = st->state_graph_ptr[s + 1] - st->state_graph_ptr[s];
      if (c > b->max_slots) b->max_slots = c;
    }
    join_range_tiles(b, cut, rt);
  } catch (const std::bad_alloc &) {
    delete b;
    return fail(XRL_ERR_OOM, "xrl_pack_state: out of host memory");
  }
  *out = b;
  return XRL_OK;
}

int xrl_pack_state_edits(const xrl_model_desc *model, const xrl_edit_state_desc *st, xrl_batch **out) {
  if (!model || !st || !out) return fail(XRL_ERR_NULL, "xrl_pack_state_edits: NULL argument");
  *out = nullptr;
  Layout L;
  int rc = build_layout(*model, L);
  if (rc) return rc;
  const int64_t S = st->n_states;
  if (S < 0) return fail(XRL_ERR_SHAPE, "n_states = %lld is negative", (long long)S);
  if (!st->cur_node_ptr || !st->cur_edge_ptr || !st->state_cand_ptr || !st->del_node_ptr || !st->del_edge_ptr ||
      !st->add_node_ptr || !st->add_edge_ptr || !st->slot_mask)
    return fail(XRL_ERR_NULL, "xrl_pack_state_edits: a ptr array or slot_mask is NULL");
  if ((rc = check_ptr(st->cur_node_ptr, S, "cur_node_ptr"))) return rc;
  if ((rc = check_ptr(st->cur_edge_ptr, S, "cur_edge_ptr"))) return rc;
  if ((rc = check_ptr(st->state_cand_ptr, S, "state_cand_ptr"))) return rc;
  const int64_t C = st->state_cand_ptr[S], G = S + C;
  if ((rc = check_ptr(st->del_node_ptr, C, "del_node_ptr"))) return rc;
  if ((rc = check_ptr(st->del_edge_ptr, C, "del_edge_ptr"))) return rc;
  if ((rc = check_ptr(st->add_node_ptr, C, "add_node_ptr"))) return rc;
  if ((rc = check_ptr(st->add_edge_ptr, C, "add_edge_ptr"))) return rc;
  const int64_t Nc = st->cur_node_ptr[S], Ec = st->cur_edge_ptr[S];
  const int64_t n_dn = st->del_node_ptr[C], n_de = st->del_edge_ptr[C], n_an = st->add_node_ptr[C], n_ae = st->add_edge_ptr[C];
  const int Dd = model->n_node_dense, De = model->d_edge, Dg = model->d_global;
  if (Nc > 0 && (!st->node_op || (Dd > 0 && !st->node_dense))) return fail(XRL_ERR_NULL, "node_op or node_dense is NULL");
  if (Ec > 0 && (!st->edge_src || !st->edge_dst || !st->edge_feat))
    return fail(XRL_ERR_NULL, "edge_src, edge_dst or edge_feat is NULL");
  if ((n_dn > 0 && !st->del_node) || (n_de > 0 && !st->del_edge) || (n_an > 0 && (!st->add_node_op || (Dd > 0 && !st->add_node_dense))) ||
      (n_ae > 0 && (!st->add_edge_src || !st->add_edge_dst || !st->add_edge_feat)))
    return fail(XRL_ERR_NULL, "xrl_pack_state_edits: an edit array is NULL");
  // graph g of the batch: state s's current graph, or candidate c
  std::vector<int32_t> sgp(S + 1), g_state(G), g_cand(G);
  for (int64_t s = 0, g = 0; s < S; ++s) {
    sgp[s] = (int32_t)g;
    g_state[g] = (int32_t)s; g_cand[g] = -1; ++g;
    for (int32_t c = st->state_cand_ptr[s]; c < st->state_cand_ptr[s + 1]; ++c, ++g) { g_state[g] = (int32_t)s; g_cand[g] = c; }
    sgp[s + 1] = (int32_t)g;
  }
  for (int64_t s = 0; s < S; ++s)
    if (st->slot_mask[sgp[s]] == 0) return fail(XRL_ERR_MASK, "state %lld masks its No-Op slot (its first graph)", (long long)s);
  // ---- the current graphs and the new items (what is validated; everything else is copied from them)
  const int64_t op = first_outside(st->node_op, Nc, model->n_op_types), new_op = first_outside(st->add_node_op, n_an, model->n_op_types);
  if (op < Nc) return fail(XRL_ERR_INDEX, "node %lld: op id %d outside [0, %d)", (long long)op, st->node_op[op], model->n_op_types);
  if (new_op < n_an)
    return fail(XRL_ERR_INDEX, "new node %lld: op id %d outside [0, %d)", (long long)new_op, st->add_node_op[new_op], model->n_op_types);
  for (int64_t s = 0; s < S; ++s) {
    const int32_t n = st->cur_node_ptr[s + 1] - st->cur_node_ptr[s];
    for (int64_t e = st->cur_edge_ptr[s]; e < st->cur_edge_ptr[s + 1]; ++e)
      if (st->edge_src[e] < 0 || st->edge_src[e] >= n || st->edge_dst[e] < 0 || st->edge_dst[e] >= n)
        return fail(XRL_ERR_INDEX, "edge %lld of state %lld's current graph: endpoint (%d -> %d) outside [0, %d)", (long long)e,
                    (long long)s, st->edge_src[e], st->edge_dst[e], n);
  }
  int64_t where = 0;
  if (Dd > 0 && !all_finite(st->node_dense, Nc * Dd, &where)) return fail(XRL_ERR_VALUE, "node_dense[%lld] is not finite", (long long)where);
  if (Dd > 0 && !all_finite(st->add_node_dense, n_an * Dd, &where)) return fail(XRL_ERR_VALUE, "add_node_dense[%lld] is not finite", (long long)where);
  if (!all_finite(st->edge_feat, Ec * De, &where)) return fail(XRL_ERR_VALUE, "edge_feat[%lld] is not finite", (long long)where);
  if (!all_finite(st->add_edge_feat, n_ae * De, &where)) return fail(XRL_ERR_VALUE, "add_edge_feat[%lld] is not finite", (long long)where);
  if (st->graph_global && !all_finite(st->graph_global, G * Dg, &where)) return fail(XRL_ERR_VALUE, "graph_global[%lld] is not finite", (long long)where);
  // ---- the current graph of every state in receiver order once: its in-edge lists (edge ids
  // ascending inside a receiver's list, i.e. the stable order); and its out-edge lists
  std::vector<int32_t> bin_ptr(Nc + S + 1, 0), bin_eid(Ec), bout_ptr(Nc + S + 1, 0), bout_eid(Ec), cursor;
  for (int64_t s = 0; s < S; ++s) {
    const int32_t nb = st->cur_node_ptr[s], n = st->cur_node_ptr[s + 1] - nb;
    const int64_t e0 = st->cur_edge_ptr[s], e1 = st->cur_edge_ptr[s + 1];
    auto lists = [&](const int32_t *end, int32_t *ip, int32_t *eid) {      // ip: [n + 1] of this state
      for (int64_t e = e0; e < e1; ++e) ip[end[e] + 1]++;
      for (int32_t i = 0; i < n; ++i) ip[i + 1] += ip[i];
      cursor.assign(ip, ip + n);
      for (int64_t e = e0; e < e1; ++e) eid[e0 + cursor[end[e]]++] = (int32_t)(e - e0);
    };
    lists(st->edge_dst, bin_ptr.data() + nb + s, bin_eid.data());
    lists(st->edge_src, bout_ptr.data() + nb + s, bout_eid.data());
  }
  // ---- the edits, and the size of every graph: an edge is gone if it is deleted or at a deleted node,
  // so only the lists of the deleted nodes are gone over
  std::vector<int32_t> gnp(G + 1, 0), gep(G + 1, 0);
  {
    int32_t n_max = 0;
    for (int64_t s = 0; s < S; ++s) n_max = std::max(n_max, st->cur_node_ptr[s + 1] - st->cur_node_ptr[s]);
    std::vector<uint8_t> dead(n_max, 0);           // per node of the state's current graph; cleared after each candidate
    for (int64_t g = 0; g < G; ++g) {
      const int64_t s = g_state[g];
      const int32_t n = st->cur_node_ptr[s + 1] - st->cur_node_ptr[s];
      const int64_t e0 = st->cur_edge_ptr[s], e1 = st->cur_edge_ptr[s + 1];
      if (g_cand[g] < 0) { gnp[g + 1] = n; gep[g + 1] = (int32_t)(e1 - e0); continue; }
      const int64_t c = g_cand[g];
      for (int32_t k = st->del_node_ptr[c]; k < st->del_node_ptr[c + 1]; ++k) {
        const int32_t v = st->del_node[k];
        if (v < 0 || v >= n || (k > st->del_node_ptr[c] && v <= st->del_node[k - 1]))
          return fail(XRL_ERR_INDEX, "candidate %lld: del_node[%d] = %d out of range or not ascending", (long long)c, k, v);
        dead[v] = 1;
      }
      const int32_t kd = st->del_edge_ptr[c], kd1 = st->del_edge_ptr[c + 1];
      int32_t kept = (int32_t)(e1 - e0) - (kd1 - kd);
      for (int32_t k = kd; k < kd1; ++k) {
        const int32_t v = st->del_edge[k];
        if (v < 0 || v >= e1 - e0 || (k > kd && v <= st->del_edge[k - 1]))
          return fail(XRL_ERR_INDEX, "candidate %lld: del_edge[%d] = %d out of range or not ascending", (long long)c, k, v);
      }
      const int32_t *ip = bin_ptr.data() + st->cur_node_ptr[s] + s, *op = bout_ptr.data() + st->cur_node_ptr[s] + s;
      auto deleted = [&](int32_t el) { return kd < kd1 && std::binary_search(st->del_edge + kd, st->del_edge + kd1, el); };
      for (int32_t k = st->del_node_ptr[c]; k < st->del_node_ptr[c + 1]; ++k) {
        const int32_t v = st->del_node[k];
        for (int32_t q = ip[v]; q < ip[v + 1]; ++q) kept -= !deleted(bin_eid[e0 + q]);
        for (int32_t q = op[v]; q < op[v + 1]; ++q) {
          const int32_t el = bout_eid[e0 + q];
          kept -= !dead[st->edge_dst[e0 + el]] && !deleted(el);    // (else counted above)
        }
      }
      const int32_t n_new = st->add_node_ptr[c + 1] - st->add_node_ptr[c];
      for (int32_t k = st->add_edge_ptr[c]; k < st->add_edge_ptr[c + 1]; ++k)
        for (const int32_t v : {st->add_edge_src[k], st->add_edge_dst[k]})
          if (v < 0 || v >= n + n_new || (v < n && dead[v]))
            return fail(XRL_ERR_INDEX, "candidate %lld: new edge %d has endpoint %d outside its graph or on a deleted node", (long long)c, k, v);
      for (int32_t k = st->del_node_ptr[c]; k < st->del_node_ptr[c + 1]; ++k) dead[st->del_node[k]] = 0;
      gnp[g + 1] = n - (st->del_node_ptr[c + 1] - st->del_node_ptr[c]) + n_new;
      gep[g + 1] = kept + (st->add_edge_ptr[c + 1] - st->add_edge_ptr[c]);
    }
    int64_t nn = 0, ee = 0;
    for (int64_t g = 0; g < G; ++g) {
      nn += gnp[g + 1]; ee += gep[g + 1];
      if (nn > INT32_MAX || ee > INT32_MAX) return fail(XRL_ERR_SHAPE, "the batch has more than 2^31 - 1 nodes or edges");
      gnp[g + 1] = (int32_t)nn; gep[g + 1] = (int32_t)ee;
    }
  }
  const int64_t N = gnp[G], E = gep[G];

  xrl_batch *b = new (std::nothrow) xrl_batch();
  if (!b) return fail(XRL_ERR_OOM, "xrl_pack_state_edits: out of host memory");
  try {
    static std::atomic<uint64_t> next_id{(uint64_t)1 << 62};
    b->id = next_id++;
    b->model = *model;
    b->S = S; b->G = G; b->N = N; b->E = E;
    b->from_edits = true;
    if (!plan_block(b, Nc, Ec, n_an, n_ae)) throw std::bad_alloc();
    memcpy(b->at<int32_t>(b->o_state_graph_ptr), sgp.data(), sizeof(int32_t) * (S + 1));
    memcpy(b->at<int32_t>(b->o_graph_node_ptr), gnp.data(), sizeof(int32_t) * (G + 1));
    uint8_t *mask = b->at<uint8_t>(b->o_mask);
    for (int64_t g = 0; g < G; ++g) mask[g] = st->slot_mask[g] ? 1 : 0;
    float *gg = b->at<float>(b->o_graph_global);
    if (st->graph_global && G * Dg > 0) memcpy(gg, st->graph_global, sizeof(float) * G * Dg);
    else memset(gg, 0, sizeof(float) * (size_t)(G * Dg));
    for (int64_t s = 0; s < S; ++s) b->max_slots = std::max(b->max_slots, sgp[s + 1] - sgp[s]);
    // (node_op, node_dense and edge_feat of the batch are not written here: the device fills its
    // copies from node_from / edge_from, and xrl_batch_host_view writes edge_feat on demand)
    int32_t *in_ptr = b->at<int32_t>(b->o_in_ptr), *in_src = b->at<int32_t>(b->o_in_src), *in_eid = b->at<int32_t>(b->o_in_eid);
    int32_t *node_from = b->at<int32_t>(b->o_node_from), *edge_from = b->at<int32_t>(b->o_edge_from);
    in_ptr[0] = 0;
    auto put = [&](size_t off, const void *src, int64_t bytes) {
      if (bytes > 0) memcpy(b->mem.p + off, src, (size_t)bytes);
    };
    put(b->o_base_op, st->node_op, Nc * 4);
    put(b->o_base_dense, st->node_dense, Nc * Dd * 4);
    put(b->o_base_feat, st->edge_feat, Ec * De * 4);
    put(b->o_new_op, st->add_node_op, n_an * 4);
    put(b->o_new_dense, st->add_node_dense, n_an * Dd * 4);
    put(b->o_new_feat, st->add_edge_feat, n_ae * De * 4);
    // ---- every graph by merging; graph ranges on separate threads
    const int T = pack_thread_count(N + E);
    std::vector<int64_t> cut(T + 1, G);
    cut[0] = 0;
    for (int t = 1, g = 0; t < T; ++t) {
      const int64_t want = (N + E) * t / T;
      while (g < G && (int64_t)gnp[g] + gep[g] < want) ++g;
      cut[t] = g;
    }
    std::vector<RangeTiles> rt(T);
    const bool merged = run_ranges(cut, [&](int t, int64_t g0, int64_t g1) {
      std::vector<int32_t> newid, erank, add_order;
      std::vector<uint8_t> dead;
      for (int64_t g = g0; g < g1; ++g) {
        const int64_t s = g_state[g], c = g_cand[g];
        const int32_t nb = st->cur_node_ptr[s], n = st->cur_node_ptr[s + 1] - nb;
        const int64_t e0 = st->cur_edge_ptr[s], e1 = st->cur_edge_ptr[s + 1];
        const int32_t *ip = bin_ptr.data() + nb + s;
        const int32_t base = gnp[g], eb = gep[g];
        const int32_t an0 = c < 0 ? 0 : st->add_node_ptr[c], n_new = c < 0 ? 0 : st->add_node_ptr[c + 1] - an0;
        const int32_t ae0 = c < 0 ? 0 : st->add_edge_ptr[c], n_ae_c = c < 0 ? 0 : st->add_edge_ptr[c + 1] - ae0;
        // surviving nodes -> new ids; surviving edges -> rank in the candidate's edge list
        dead.assign(n, 0);
        if (c >= 0)
          for (int32_t k = st->del_node_ptr[c]; k < st->del_node_ptr[c + 1]; ++k) dead[st->del_node[k]] = 1;
        newid.assign(n + n_new, -1);
        int32_t nk = 0;
        for (int32_t i = 0; i < n; ++i)
          if (!dead[i]) newid[i] = nk++;
        for (int32_t k = 0; k < n_new; ++k) newid[n + k] = nk + k;
        erank.assign(e1 - e0, -1);
        int32_t ek = 0;
        {
          int32_t kd = c < 0 ? 0 : st->del_edge_ptr[c];
          const int32_t kd1 = c < 0 ? 0 : st->del_edge_ptr[c + 1];
          for (int64_t e = e0; e < e1; ++e) {
            if (kd < kd1 && st->del_edge[kd] == e - e0) { ++kd; continue; }
            if (!dead[st->edge_src[e]] && !dead[st->edge_dst[e]]) erank[e - e0] = ek++;
          }
        }
        // new edges grouped by receiver, in their own order inside a group
        add_order.resize(n_ae_c);
        for (int32_t k = 0; k < n_ae_c; ++k) add_order[k] = k;
        std::stable_sort(add_order.begin(), add_order.end(), [&](int32_t x, int32_t y) {
          return newid[st->add_edge_dst[ae0 + x]] < newid[st->add_edge_dst[ae0 + y]];
        });
        // nodes
        for (int32_t i = 0; i < n; ++i) {
          if (dead[i]) continue;
          node_from[base + newid[i]] = nb + i;
        }
        for (int32_t k = 0; k < n_new; ++k) node_from[base + nk + k] = -1 - (an0 + k);
        // receiver order: per receiver its surviving in-edges (edge ids ascending), then its new ones
        int32_t p = eb, ka = 0;
        int32_t *inp = in_ptr + base + 1;
        int32_t vcur = 0;
        for (int32_t i = 0; i < n + n_new; ++i) {
          if (i < n && dead[i]) continue;
          const int32_t v = vcur++;                  // == newid[i]
          if (i < n) {
            for (int32_t q = ip[i]; q < ip[i + 1]; ++q) {
              const int32_t el = bin_eid[e0 + q];
              if (erank[el] < 0) continue;
              const int64_t e = e0 + el;
              in_src[p] = base + newid[st->edge_src[e]];
              in_eid[p] = eb + erank[el];
              edge_from[p] = (int32_t)e;
              ++p;
            }
          }
          for (; ka < n_ae_c && newid[st->add_edge_dst[ae0 + add_order[ka]]] == v; ++ka) {
            const int32_t k = ae0 + add_order[ka];
            in_src[p] = base + newid[st->add_edge_src[k]];
            in_eid[p] = eb + ek + add_order[ka];
            edge_from[p] = -1 - k;
            ++p;
          }
          inp[v] = p;                                // end of v's in-edges
        }
      }
      range_tiles(in_ptr, gnp.data(), g0, g1, gep[g0], G <= kGraphTileMaxGraphs, rt[t]);
    });
    if (!merged) throw std::bad_alloc();
    join_range_tiles(b, cut, rt);
  } catch (const std::bad_alloc &) {
    delete b;
    return fail(XRL_ERR_OOM, "xrl_pack_state_edits: out of host memory");
  }
  *out = b;
  return XRL_OK;
}

int xrl_edge_features_from_shapes(const int32_t *shape_ptr, const int64_t *dims, int64_t n_edges,
                                  double M, float *edge_feat) {
  if (n_edges < 0) return fail(XRL_ERR_SHAPE, "n_edges = %lld is negative", (long long)n_edges);
  if (!shape_ptr || (n_edges > 0 && !edge_feat))
    return fail(XRL_ERR_NULL, "xrl_edge_features_from_shapes: NULL argument");
  if (!(M > 0.0)) return fail(XRL_ERR_VALUE, "the normalisation constant M must be positive");
  if (shape_ptr[0] != 0) return fail(XRL_ERR_SHAPE, "shape_ptr[0] must be 0");
  for (int64_t e = 0; e < n_edges; ++e) {
    const int64_t r = (int64_t)shape_ptr[e + 1] - shape_ptr[e];
    if (r < 0 || r > 4)
      return fail(XRL_ERR_SHAPE, "edge %lld: rank %lld outside [0, 4]", (long long)e, (long long)r);
    if (r > 0 && !dims) return fail(XRL_ERR_NULL, "xrl_edge_features_from_shapes: dims is NULL");
    float *o = edge_feat + 4 * e;
    for (int k = 0; k < 4; ++k) o[k] = 0.0f;                  // leading dimensions padded with zeros
    for (int64_t k = 0; k < r; ++k) {
      const int64_t d = dims[shape_ptr[e] + k];
      if (d < 0) return fail(XRL_ERR_VALUE, "edge %lld: negative extent %lld", (long long)e, (long long)d);
      o[4 - r + k] = (float)((double)d / M);
    }
  }
  return XRL_OK;
}

int xrl_batch_dims(const xrl_batch *b, int64_t *S, int64_t *G, int64_t *N, int64_t *E) {
  if (!b) return fail(XRL_ERR_NULL, "xrl_batch_dims: batch is NULL");
  if (S) *S = b->S;
  if (G) *G = b->G;
  if (N) *N = b->N;
  if (E) *E = b->E;
  return XRL_OK;
}

// What packing left out, from what it wrote. Null: out of memory.
static PackedArrays *packed_arrays(const xrl_batch *b) {
  const int64_t N = b->N, E = b->E;
  const int De = b->model.d_edge;
  const int32_t *in_ptr = b->at<int32_t>(b->o_in_ptr), *in_src = b->at<int32_t>(b->o_in_src), *gnp = b->at<int32_t>(b->o_graph_node_ptr);
  std::unique_ptr<PackedArrays> a;
  try {
    a.reset(new PackedArrays());
    a->in_dst.resize(E); a->out_ptr.resize(N + 1); a->out_pos.resize(E); a->node_graph.resize(N);
    if (b->from_edits) a->edge_feat.resize((size_t)E * De);
  } catch (const std::bad_alloc &) {
    return nullptr;
  }
  for (int64_t g = 0; g < b->G; ++g)
    for (int32_t n = gnp[g]; n < gnp[g + 1]; ++n) a->node_graph[n] = (int32_t)g;
  for (int64_t n = 0; n < N; ++n)
    for (int32_t p = in_ptr[n]; p < in_ptr[n + 1]; ++p) a->in_dst[p] = (int32_t)n;
  // sender index: receiver-order positions grouped by sender, ascending (out_ptr[s]: next place while they are dealt
  // out, i.e. the end of s's, the beginning of s + 1's)
  std::fill(a->out_ptr.begin(), a->out_ptr.end(), 0);
  for (int64_t p = 0; p < E; ++p) a->out_ptr[in_src[p]]++;
  int32_t sum = 0;
  for (int64_t n = 0; n <= N; ++n) {
    const int32_t k = a->out_ptr[n];
    a->out_ptr[n] = sum;
    sum += k;
  }
  for (int64_t p = 0; p < E; ++p) a->out_pos[a->out_ptr[in_src[p]]++] = (int32_t)p;
  for (int64_t n = N; n > 0; --n) a->out_ptr[n] = a->out_ptr[n - 1];
  a->out_ptr[0] = 0;
  if (b->from_edits) {
    const int32_t *edge_from = b->at<int32_t>(b->o_edge_from);
    for (int64_t p = 0; p < E; ++p) {
      const int32_t f = edge_from[p];
      const float *src = f >= 0 ? b->at<float>(b->o_base_feat) + (size_t)f * De : b->at<float>(b->o_new_feat) + (size_t)(-1 - f) * De;
      memcpy(a->edge_feat.data() + (size_t)p * De, src, sizeof(float) * De);
    }
  }
  return a.release();
}

int xrl_batch_host_view(const xrl_batch *cb, xrl_packed_view *v) {
  if (!cb || !v) return fail(XRL_ERR_NULL, "xrl_batch_host_view: NULL argument");
  xrl_batch *b = const_cast<xrl_batch *>(cb);
  PackedArrays *a = b->view.load();
  if (!a) {
    // (made without a lock: of several threads that ask first, one publishes its copy, and the others drop theirs)
    PackedArrays *mine = packed_arrays(b);
    if (!mine) return fail(XRL_ERR_OOM, "xrl_batch_host_view: out of host memory");
    if (b->view.compare_exchange_strong(a, mine)) a = mine;
    else delete mine;
  }
  v->S = b->S; v->G = b->G; v->N = b->N; v->E = b->E;
  v->state_graph_ptr = b->at<int32_t>(b->o_state_graph_ptr);
  v->graph_node_ptr = b->at<int32_t>(b->o_graph_node_ptr);
  v->in_ptr = b->at<int32_t>(b->o_in_ptr);
  v->in_src = b->at<int32_t>(b->o_in_src);
  v->in_dst = a->in_dst.data();
  v->in_eid = b->at<int32_t>(b->o_in_eid);
  v->out_ptr = a->out_ptr.data();
  v->out_pos = a->out_pos.data();
  v->node_graph = a->node_graph.data();
  v->edge_feat = b->from_edits ? a->edge_feat.data() : b->at<float>(b->o_edge_feat);
  v->n_tiles = b->n_tiles;
  v->tile_ptr = b->at<int32_t>(b->o_tile);
  v->n_graph_tiles = b->n_graph_tiles;
  v->graph_tile_ptr = b->has_graph_tiles ? b->at<int32_t>(b->o_graph_tile) : nullptr;
  v->gtile_ptr = b->has_graph_tiles ? b->at<int32_t>(b->o_gtile) : nullptr;
  return XRL_OK;
}

int xrl_batch_free(xrl_batch *b) {
  if (!b) return XRL_OK;
  xrl_batch_release_device(b);
  delete b;
  return XRL_OK;
}

}  // extern "C"
