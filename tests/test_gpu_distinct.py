"""Batches reduced to distinct nodes: classes of nodes with equal histories are encoded once. Every state,
received sum and embedding has to be the same bits as without the reduction; gradients, whose sums
are taken in another order, agree to rounding and with the oracle."""
import dataclasses

import numpy as np
import pytest

import paper_2304_14698_amd as xrl
import synth

pytestmark = pytest.mark.gpu


def _edge_cases(rng, model):
    """Graphs that are the same but for one edge attribute's last bit, a node's last attribute, the order
    of a receiver's in-edges, a sender five hops up; empty and edgeless graphs; a repeated edge; a
    graph twice; receivers of 32 in-edges."""
    base = synth.layered_dag(rng, 40)
    n, e = base.n_nodes, base.n_edges

    def bump(a, i):
        a = a.copy()
        a.reshape(-1)[i] = np.nextafter(a.reshape(-1)[i], np.float32(100))
        return a

    def variant(**kw):
        return dataclasses.replace(base, **kw)
    back = np.arange(e)[::-1]
    indeg_32 = np.concatenate([np.where(base.dst == n - 1, n - 2, base.dst), np.full(32, n - 1)]).astype(np.int32)
    hub = variant(src=np.concatenate([base.src, np.arange(32) % (n - 1)]).astype(np.int32), dst=indeg_32,
                  efeat=np.concatenate([base.efeat, base.efeat[:32]]))
    assert np.bincount(hub.dst).max() == 32
    graphs = [base, base, variant(efeat=bump(base.efeat, 0)), variant(efeat=bump(base.efeat, base.efeat.size - 1)),
              variant(dense=bump(base.dense, base.dense.size - 1)),
              variant(op=np.concatenate([[(base.op[0] + 1) % 32], base.op[1:]]).astype(np.int32)),
              variant(src=base.src[back], dst=base.dst[back], efeat=base.efeat[back]),
              variant(src=base.src[:0], dst=base.dst[:0], efeat=base.efeat[:0]), hub, hub,
              variant(op=base.op[:0], dense=base.dense[:0], layer=base.layer[:0], block=base.block[:0], src=base.src[:0],
                      dst=base.dst[:0], efeat=base.efeat[:0])]
    return synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))])


def _state(kind, rng, model):
    if kind == "edges":
        return _edge_cases(rng, model), False
    if kind == "edits":
        base = synth.shuffle_edges(rng, synth.resnet_dag(rng, 3))
        return synth.make_edit_states(rng, [base, base], [9, 17], by_block=True)[0], True
    base = synth.transformer_dag(rng, 3) if kind == "transformer" else synth.resnet_dag(rng, 4)
    states = [synth.make_state(rng, base, n, by_block=True) for n in ((24,) if kind == "transformer" else (5, 60, 1))]
    return synth.concat_states(states), False


def _run(enc, batch, up, rounds):
    import torch
    out = {"emb": enc.encode(batch, save_for_backward=True)}
    for r in range(rounds + 1):
        out[f"h{r}"] = enc.get_activation(batch, "h", r)
        if r:
            out[f"agg{r}"] = enc.get_activation(batch, "agg", r)
    dw = torch.zeros(enc.n_weights, dtype=torch.float32, device="cuda")
    enc.encode_backward(batch, up, dw)
    plain = enc.encode(batch)
    again = torch.zeros_like(dw)
    enc.encode(batch, save_for_backward=True)
    enc.encode_backward(batch, up, again)
    assert torch.equal(plain, out["emb"]) and torch.equal(dw, again)
    return {k: v.cpu().numpy() for k, v in out.items()}, dw.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("kind", ["edges", "resnet", "transformer", "edits"])
@pytest.mark.parametrize("hidden,precision,layers,readout", [
    (64, "fp32", 2, "sum"), (128, "bf16", 2, "mean"), (256, "bf16", 2, "sum"),
    (128, "fp32", 1, "mean")])
def test_reduction_changes_nothing(kind, hidden, precision, layers, readout, monkeypatch):
    import torch
    rng = np.random.Generator(np.random.PCG64(5))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, mlp_layers=layers, readout=readout, rounds=3)
    state, edits = _state(kind, rng, model)
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    got = {}
    for min_us in ("-1", "0"):                      # never, always
        monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
        monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
        if precision == "bf16":                     # gradients from the kept forward on both sides
            monkeypatch.setenv("XRL_PERSISTENT_MIN_ROWS", "0")
        enc = xrl.Encoder(model, w)
        batch = enc.pack_edits(state) if edits else enc.pack(state)
        up = torch.tensor(np.random.default_rng(3).standard_normal((batch.G, hidden)), dtype=torch.float32, device="cuda")
        got[min_us] = _run(enc, batch, up, model["rounds"])
        batch.free()
        enc.close()
    (a, da), (b, db) = got["-1"], got["0"]
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    # fp32: sums of thousands of products in another order; bf16: every stored gradient row is rounded to
    # 2^-9, here per node, there per class (measured: 2e-7 to 1e-6 and 1e-3 to 5e-3)
    assert np.linalg.norm(da - db) <= (1e-5 if precision == "fp32" else 2e-2) * np.linalg.norm(da)


@pytest.mark.parametrize("hidden,precision,d_edge,n_cand", [(64, "bf16", 8, 100), (128, "bf16", 8, 100), (256, "bf16", 8, 30),
                                                            (128, "bf16", 20, 100), (64, "fp32", 8, 30)])
def test_reduction_at_default_thresholds(hidden, precision, d_edge, n_cand, monkeypatch):
    """A kept batch as a program runs it: the first forward-only encode takes the whole batch, on the persistent kernels
    where it is large enough for them, the second one its levels, on a mixture of split and persistent ones, and a
    saving encode the levels on persistent ones throughout. All give the whole batch's bits. (d_edge = 20: edge
    attributes wider than the persistent edge kernels take, and the backward pass that recomputes.)"""
    import torch
    rng = np.random.Generator(np.random.PCG64(5))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, rounds=5, d_edge=d_edge)
    state = synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 16), n_cand, by_block=True)])
    state["edge_feat"] = np.ascontiguousarray(np.tile(state["edge_feat"], (1, 3))[:, :d_edge])
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    N = len(state["node_op"])
    assert N > (8192 if hidden == 256 else 32768) or precision == "fp32"
    got = []
    for min_us in ("-1", "0"):
        monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
        enc = xrl.Encoder(model, w)
        batch = enc.pack(state)
        embs = [enc.encode(batch)]
        assert enc.batch_level(batch, 0)[0] == N
        embs.append(enc.encode(batch))
        nodes = [enc.batch_level(batch, r)[0] for r in range(6)]
        assert (max(nodes) < N and min(nodes) < 8192) if min_us == "0" else nodes == [N] * 6
        embs.append(enc.encode(batch, save_for_backward=True))
        acts = [enc.get_activation(batch, "h", r) for r in range(6)] + [enc.get_activation(batch, "agg", r) for r in range(1, 6)]
        dw = torch.zeros(enc.n_weights, device="cuda")
        enc.encode_backward(batch, torch.randn(batch.G, hidden, generator=torch.Generator().manual_seed(1)).cuda(), dw)
        got.append((embs, acts, dw.double()))
        batch.free()
        enc.close()
    (e0, a0, d0), (e1, a1, d1) = got
    assert all(torch.equal(x, e0[0]) for x in e0 + e1)
    assert all(torch.equal(x, y) for x, y in zip(a0, a1))
    # (as in test_reduction_changes_nothing)
    assert float((d1 - d0).norm() / d0.norm()) <= (1e-5 if precision == "fp32" else 2e-2)


def test_reduced_batch_against_the_oracle(monkeypatch):
    from test_gpu_backward import run_backward_case
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", "0")
    monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
    model, _ = synth.make_config(1)
    rng = np.random.Generator(np.random.PCG64(9))
    state = synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 2), n, by_block=True) for n in (12, 3)])
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    run_backward_case(xrl, model, state, w, seed=4)


def test_a_captured_context_keeps_its_buffers(monkeypatch):
    """A graph of a batch encoded whole holds addresses in the context's buffers: neither that batch nor a later one is
    reduced after the capture, as its buffers might have to grow, and replays among eager calls stay right."""
    import torch
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", "0")
    monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
    rng = np.random.Generator(np.random.PCG64(6))
    model, _ = synth.make_config(1)
    model.update(hidden=128, precision="bf16", rounds=3)
    states = [synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 3), n, by_block=True)]) for n in (20, 5)]
    w = [synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1) for _ in range(2)]
    side = torch.cuda.Stream()
    enc = xrl.Encoder(model, w[0], stream=side)
    batch, other = (enc.pack(s) for s in states)
    first = enc.encode(batch)
    out = torch.empty_like(first)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
        enc.encode(batch, out=out)
    for weights in (w[0], w[1]):
        enc.set_weights(weights)
        for _ in range(3):
            eager = enc.encode(batch)
            enc.encode(other)
            torch.cuda.synchronize()
            out.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager)
    assert enc.batch_level(batch, 0)[0] == batch.N and enc.batch_level(other, 0)[0] == other.N
    fresh = xrl.Encoder(model, w[1])                # (the same batch is reduced where nothing was captured)
    again = fresh.pack(states[0])
    fresh.encode(again)
    assert torch.equal(fresh.encode(again), eager) and fresh.batch_level(again, 0)[0] < again.N
    for x in (batch, other, again):
        x.free()
    fresh.close()
    enc.close()


def _tags(dense):
    """Tags of level-0 keys of nodes without in-edges, operator 0, one attribute: the hash of the class table restated."""
    def mix(h, v):
        h = (h ^ v) * np.uint64(0x9E3779B97F4A7C15)
        return h ^ (h >> np.uint64(29))
    h = mix(np.zeros(len(dense), np.uint64), np.uint64(0))
    h = mix(h, dense.view(np.uint32).astype(np.uint64))
    return mix(h, h >> np.uint64(32)) >> np.uint64(28)


def test_keys_of_one_tag(monkeypatch):
    """Two keys of one tag share a table slot: the one of the smallest node is a class, every node of the other a class of
    its own, in every run; values are those of the whole batch."""
    import torch
    dense = np.arange(1 << 21, dtype=np.float32)
    tags = _tags(dense)
    order = np.argsort(tags, kind="stable")
    twins = np.flatnonzero(tags[order][1:] == tags[order][:-1])
    assert len(twins) > 0
    a, b = dense[order[twins[0]]], dense[order[twins[0] + 1]]
    model, _ = synth.make_config(1)
    model.update(hidden=64, precision="fp32", rounds=1, n_node_dense=1)
    rng = np.random.Generator(np.random.PCG64(5))
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    G = 700                                         # graphs p -> q, p of the first key and of the second by turns
    value = np.where(np.arange(G) % 2 == 0, a, b)
    state = dict(n_states=1, state_graph_ptr=np.array([0, G], np.int32), graph_node_ptr=np.arange(0, 2 * G + 1, 2, dtype=np.int32),
                 graph_edge_ptr=np.arange(G + 1, dtype=np.int32), node_op=np.zeros(2 * G, np.int32),
                 node_dense=np.stack([value, np.zeros(G)], 1).astype(np.float32).reshape(-1, 1), edge_src=np.zeros(G, np.int32),
                 edge_dst=np.ones(G, np.int32), edge_feat=np.zeros((G, model["d_edge"]), np.float32),
                 graph_global=np.zeros((G, model["d_global"]), np.float32), slot_mask=np.ones(G, np.uint8))
    got = []
    for min_us in ("-1", "0", "0", "0"):
        monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
        monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
        enc = xrl.Encoder(model, w)
        batch = enc.pack(state)
        emb = enc.encode(batch, save_for_backward=True).cpu()
        dw = torch.zeros(enc.n_weights, device="cuda")
        enc.encode_backward(batch, torch.ones(G, 64, device="cuda"), dw)
        got.append((emb, dw.cpu(), [enc.batch_level(batch, r)[0] for r in (0, 1)]))
        batch.free()
        enc.close()
    assert got[0][2] == [2 * G, 2 * G]
    assert float((got[1][1] - got[0][1]).norm() / got[0][1].norm()) < 1e-5
    for emb, dw, nodes in got[1:]:
        assert nodes == [2 + G // 2, 2 + 2 * (G // 2)]      # first key, q, every node of the second key; and its q
        assert torch.equal(emb, got[0][0]) and torch.equal(dw, got[1][1])


def test_reducing_during_another_streams_capture(monkeypatch):
    """The encode that reduces a batch allocates and waits; a capture that is under way on another stream goes on."""
    import torch
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", "0")
    rng = np.random.Generator(np.random.PCG64(6))
    model, _ = synth.make_config(1)
    state = synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 3), 20, by_block=True)])
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1), stream=torch.cuda.Stream())
    batch = enc.pack(state)
    want = enc.encode(batch)
    out = torch.empty_like(want)
    x = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):       # (the mode that forbids unsafe calls)
        x += 1
        enc.encode(batch, out=out)
        x += 1
    assert enc.batch_level(batch, 0)[0] < batch.N
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, want) and float(x.sum()) == 16
    batch.free()
    enc.close()


@pytest.mark.parametrize("grouped", [True, False])
def test_reduced_step_in_a_graph(grouped, monkeypatch):
    """A saving encode and its backward pass of a reduced batch in a graph; grouped = False: the batch's first backward pass is
    the captured one, which then makes its groupings in every replay. Replays among eager steps under new weights."""
    import torch
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", "0")
    monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
    rng = np.random.Generator(np.random.PCG64(6))
    model, _ = synth.make_config(1)
    model.update(hidden=128, precision="bf16", rounds=3)
    state = synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 4), n, by_block=True) for n in (30, 9)])
    w = [synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1) for _ in range(2)]
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        enc = xrl.Encoder(model, w[0], stream=side)
        up = torch.randn(41, 128, generator=torch.Generator().manual_seed(2)).cuda()
        twin, batch = enc.pack(state), enc.pack(state)
        emb, dw = torch.empty(41, 128, device="cuda"), torch.zeros(enc.n_weights, device="cuda")

        def step(b):
            enc.encode(b, save_for_backward=True, out=emb)
            dw.zero_()
            enc.encode_backward(b, up, dw)
        step(twin)                                  # (the workspaces have their sizes)
        if grouped:
            step(batch)
        else:
            enc.encode(batch, save_for_backward=True)
        assert enc.batch_level(batch, 0)[0] < batch.N
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
            step(batch)
        for weights in w:
            enc.set_weights(weights)
            for _ in range(3):
                step(twin)
                want = emb.clone(), dw.clone()
                emb.zero_()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(emb, want[0]) and torch.equal(dw, want[1])
                step(batch)
                torch.cuda.synchronize()
                assert torch.equal(emb, want[0]) and torch.equal(dw, want[1])
        batch.free()
        twin.free()
        enc.close()
