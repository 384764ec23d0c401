"""A batch encoded once, forward only, in bf16 at H = 256: its levels are made on the device, one at a time, in
front of the round that runs on them. Embeddings have to be the bits of the whole batch's."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded ahead of the library)

import paper_2304_14698_amd as xrl
import synth
from test_gpu_distinct import _state

pytestmark = pytest.mark.gpu


def _embeddings(model, w, pack, min_us, monkeypatch):
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
    monkeypatch.setenv("XRL_PERSISTENT_MIN_ROWS", "0")
    enc = xrl.Encoder(model, w)
    enc.set_timing(True)
    got = []
    for _ in range(3):                       # (batches in turn: the levels' memory is used again)
        for state, edits in pack:
            batch = enc.pack_edits(state) if edits else enc.pack(state)
            got.append(enc.encode(batch).cpu().numpy())
            # (the memory made ready, then the level of the node-update layer and one a round)
            assert enc.read_timing("levels")[1] == (0 if min_us == "-1" else model["rounds"] + 2)
            batch.free()
    enc.close()
    return got


@pytest.mark.parametrize("readout,rounds", [("sum", 3), ("mean", 1)])
def test_levels_made_on_the_device(readout, rounds, monkeypatch):
    """Edge cases (see _edge_cases), several states, edits, and a state of one graph shape but for the order of edges:
    more nodes than a block of the level kernels takes, and fewer."""
    rng = np.random.Generator(np.random.PCG64(11))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", readout=readout, rounds=rounds)
    pack = [_state(kind, rng, model) for kind in ("edges", "resnet", "transformer", "edits")]
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    whole = _embeddings(model, w, pack, "-1", monkeypatch)
    levels = _embeddings(model, w, pack, "0", monkeypatch)
    assert all(np.array_equal(a, b) for a, b in zip(whole, levels))


@pytest.mark.parametrize("hidden,precision", [(64, "bf16"), (128, "bf16"), (64, "fp32")])
def test_a_kept_batch_is_reduced_after_some_encodes(hidden, precision):
    """Below the threshold of the first: the more an encode takes, the sooner, and sooner if it is saved for the backward pass, but not
    by the first; same bits before and after, and reduced for good."""
    rng = np.random.Generator(np.random.PCG64(12))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, rounds=5)
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1))
    per_us = 10 * hidden * (6 * hidden + 8) / (7e8 if precision == "bf16" else 7e7)
    taken = {}
    for us in ((40, 80, 160) if precision == "bf16" else (90, 130, 220)):
        for save in (False, True):
            state = synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 16), round(us / per_us / 345), by_block=True)])
            batch = enc.pack(state)
            first, whole = enc.encode(batch, save_for_backward=save).cpu().numpy(), 1
            while enc.batch_level(batch, 0)[0] == batch.N and whole < 60:
                assert np.array_equal(enc.encode(batch, save_for_backward=save).cpu().numpy(), first)
                whole += 1
            taken[us, save] = whole
            for again in (False, True):
                assert np.array_equal(enc.encode(batch, save_for_backward=again).cpu().numpy(), first)
            assert enc.batch_level(batch, 0)[0] < batch.N
            batch.free()
    for save in (False, True):
        n = [v for (us, s), v in sorted(taken.items()) if s == save]
        assert 1 < n[2] <= n[1] <= n[0] < 60 and n[2] < n[0], taken
    assert all(taken[us, True] < taken[us, False] for us, _ in taken), taken
    enc.close()


def _large_state(rng, model, kind):
    """A state of transformer-shaped graphs, large enough for the default threshold: rewrites of the first; the same with noise on
    every edge's attributes; with a dense attribute of every third node changed."""
    state = synth.concat_states([synth.make_state(rng, synth.transformer_dag(rng, 12), 150, by_block=True)])
    if kind == "edges":
        state["edge_feat"] = (state["edge_feat"] + rng.standard_normal(state["edge_feat"].shape) / 64).astype(np.float32)
    elif kind == "nodes":
        dense = state["node_dense"].copy()
        some = rng.random(len(dense)) < 1 / 3
        dense[some, 0] += rng.standard_normal(int(some.sum())).astype(np.float32)
        state["node_dense"] = dense
    us = 2 * model["rounds"] * 256 * (len(state["node_op"]) * 768 + len(state["edge_src"]) * 776) / 7e8
    assert us > 430
    return state


@pytest.mark.parametrize("kind", ["rewrites", "edges", "nodes"])
def test_a_batch_of_distinct_nodes_is_left_whole(kind):
    """Default threshold: graphs alike in their operators alone have nothing to gain from levels, neither when they are encoded
    once, nor in any encode after their distinct nodes have been counted (by the second encode), by any context."""
    rng = np.random.Generator(np.random.PCG64(13))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", rounds=5)
    state = _large_state(rng, model, kind)
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    enc, other = xrl.Encoder(model, w), xrl.Encoder(model, w)
    batch = enc.pack(state)
    levels = []
    for e in (enc, enc, enc, other):
        e.set_timing(True)
        emb = e.encode(batch).cpu().numpy()
        levels.append(e.read_timing("levels")[1])
        if len(levels) == 1:
            first = emb
        assert np.array_equal(emb, first)
    # (rewrites: by levels once, then reduced for good; the other context goes by levels)
    assert levels == ([7, 0, 0, 7] if kind == "rewrites" else [0, 0, 0, 0])
    assert (enc.batch_level(batch, 5)[0] < batch.N) == (kind == "rewrites")
    batch.free()
    enc.close()
    other.close()


def test_counted_and_left_whole():
    """A batch that passes for rewrites by its sample (first and last nodes alike) and is not: the first encode goes by levels, the
    second counts its distinct nodes, later ones take it whole."""
    rng = np.random.Generator(np.random.PCG64(14))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", rounds=5)
    state = _large_state(rng, model, "rewrites")
    dense, gnp = state["node_dense"].copy(), state["graph_node_ptr"]
    for a, b in zip(gnp[:-1], gnp[1:]):
        dense[a + 32:b - 32, 0] += rng.standard_normal(b - a - 64).astype(np.float32)
    state["node_dense"] = dense
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1))
    batch = enc.pack(state)
    levels, embs = [], []
    for _ in range(4):
        enc.set_timing(True)
        embs.append(enc.encode(batch).cpu().numpy())
        levels.append(enc.read_timing("levels")[1])
    assert levels == [7, 0, 0, 0] and enc.batch_level(batch, 5)[0] == batch.N
    assert all(np.array_equal(e, embs[0]) for e in embs)
    batch.free()
    enc.close()


def test_levels_need_no_workspace_of_their_own():
    """An encode by levels on a context whose encode workspace is large enough queues its work and returns: its levels lie there
    too, so nothing is allocated, which would wait for the stream."""
    import time
    rng = np.random.Generator(np.random.PCG64(15))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", rounds=5)
    state = _large_state(rng, model, "rewrites")
    lone = synth.concat_states([([synth.layered_dag(rng, 120000)], np.ones(1, np.uint8))])   # (no rewrites of it: not reduced)
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1))
    enc.encode(enc.pack(lone), save_for_backward=True)       # (saves more than the encode below takes)
    out = torch.empty((len(state["slot_mask"]), 256), device="cuda")
    held = []
    for _ in range(3):
        batch = enc.pack(state)
        torch.cuda.synchronize()
        enc.set_timing(True)
        torch.cuda._sleep(200_000_000)                          # about a tenth of a second
        t0 = time.perf_counter()
        enc.encode(batch, out=out)
        held.append(time.perf_counter() - t0)
        done = torch.cuda.Event()
        done.record()
        assert not done.query(), "the queue was not held long enough to tell"
        torch.cuda.synchronize()
        assert enc.read_timing("levels")[1] == 7
        batch.free()
    assert max(held) < 0.02, held
    enc.close()


@pytest.mark.parametrize("hidden,precision,n_cand,reduced", [
    (256, "bf16", 20, False), (256, "bf16", 30, True), (128, "fp32", 20, False), (128, "fp32", 26, True),
    (256, "fp32", 5, False), (256, "fp32", 12, True)])
def test_a_small_kept_batch_is_left_whole(hidden, precision, n_cand, reduced):
    """A kept batch that fills no pass of the chip gains nothing from being reduced, however often it is encoded: below 8192 nodes, up to
    two thirds of the estimate from which a batch is reduced at once."""
    rng = np.random.Generator(np.random.PCG64(16))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, rounds=5)
    state = synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 16), n_cand, by_block=True)])
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1))
    batch = enc.pack(state)
    us = 10 * hidden * (batch.N * 3 * hidden + batch.E * (3 * hidden + 8)) / (7e8 if precision == "bf16" else 7e7)
    assert (30 if precision == "bf16" else 75) < us < 300       # (a smaller kept batch, by its estimate)
    assert reduced == (batch.N >= 8192 or us >= 200)
    for _ in range(40):
        enc.encode(batch, save_for_backward=True)
    assert (enc.batch_level(batch, 0)[0] < batch.N) == reduced
    batch.free()
    enc.close()


@pytest.mark.parametrize("min_us,levels", [("300", 7), ("500", 7), ("2000", 0)])
def test_the_threshold_holds_for_one_encode_too(min_us, levels, monkeypatch):
    """A batch below the smallest one that is to be reduced is left whole when it is encoded once, as when it is kept."""
    rng = np.random.Generator(np.random.PCG64(17))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", rounds=5)
    state = _large_state(rng, model, "rewrites")
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1))
    batch = enc.pack(state)
    us = 10 * 256 * (batch.N * 768 + batch.E * 776) / 7e8
    assert 500 < us < 2000
    enc.set_timing(True)
    enc.encode(batch)
    assert enc.read_timing("levels")[1] == levels
    batch.free()
    enc.close()


@pytest.mark.parametrize("d_edge,n_dense,n_states,cand", [(8, 4, 1, 150), (4, 0, 3, 47), (8, 1, 40, 4)])
def test_levels_of_many_distinct_nodes(d_edge, n_dense, n_states, cand, monkeypatch):
    """Levels that keep far more nodes and edges than a pass of the chip's persistent blocks takes (256 of one edge or node tile at a
    time with the next two requested ahead, 1024 waves of one node tile each), and partly filled last tiles."""
    rng = np.random.Generator(np.random.PCG64(18))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", rounds=2, d_edge=d_edge, n_node_dense=n_dense)
    state = synth.concat_states([synth.make_state(rng, synth.transformer_dag(rng, 12), cand, by_block=True) for _ in range(n_states)])
    N, E = len(state["node_op"]), len(state["edge_src"])
    state["node_dense"] = np.ascontiguousarray(state["node_dense"][:, :n_dense])
    feat = np.ascontiguousarray(state["edge_feat"][:, :d_edge])
    other = rng.random(E) < 0.7                                  # (attributes that make most nodes distinct)
    feat[other, -1] += rng.standard_normal(int(other.sum())).astype(np.float32)
    state["edge_feat"] = feat
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    whole, levels = ([e for e in _embeddings(model, w, [(state, False)], us, monkeypatch)] for us in ("-1", "0"))
    assert all(np.array_equal(a, whole[0]) for a in whole + levels)
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", "0")
    enc = xrl.Encoder(model, w)
    batch = enc.pack(state)
    for _ in range(2):                                           # (the second one counts the levels)
        enc.encode(batch)
    nodes, edges, _, tiles = zip(*[enc.batch_level(batch, r) for r in range(3)])
    assert min(nodes) > 1024 * 32 + 32 and min(tiles[1:]) > 3 * 256 and max(nodes) < N, (nodes, tiles)
    assert any(n % 32 for n in nodes)
    batch.free()
    enc.close()


def test_levels_on_another_context_and_after_a_capture():
    """A context that did not upload the batch goes by its levels too; one whose calls have been captured does not, for that batch and
    later ones. The same bits all along."""
    rng = np.random.Generator(np.random.PCG64(19))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", rounds=5)
    state = _large_state(rng, model, "rewrites")
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    side = torch.cuda.Stream()
    owner, other, captured = xrl.Encoder(model, w), xrl.Encoder(model, w), xrl.Encoder(model, w, stream=side)
    batch = owner.pack(state)

    def encode(enc, b):
        enc.set_timing(True)
        emb = enc.encode(b)
        torch.cuda.synchronize()
        n = enc.read_timing("levels")[1]
        enc.set_timing(False)
        return emb, n

    first, n = encode(owner, batch)
    assert n == 7
    for _ in range(2):
        emb, n = encode(other, batch)
        assert n == 7 and torch.equal(emb, first)
    small = captured.pack(synth.concat_states([([synth.layered_dag(rng, 60)], np.ones(1, np.uint8))]))
    out = captured.encode(small)
    torch.cuda.synchronize()
    emb, n = encode(captured, batch)
    assert n == 7 and torch.equal(emb, first)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
        captured.encode(small, out=out)
    for _ in range(2):
        emb, n = encode(captured, batch)
        assert n == 0 and torch.equal(emb, first)
        eager = captured.encode(small)
        torch.cuda.synchronize()
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
    later = captured.pack(state)
    emb, n = encode(captured, later)
    assert n == 0 and torch.equal(emb, first)
    del graph
    for b in (batch, small, later):
        b.free()
    for e in (owner, other, captured):
        e.close()
