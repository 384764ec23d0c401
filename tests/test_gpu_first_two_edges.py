"""The first two in-edges of a node count in either order when a batch is reduced to its distinct nodes; the
third and further ones keep their places. Same bits as the whole batch."""
import dataclasses

import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded ahead of the library)

import paper_2304_14698_amd as xrl
import synth

pytestmark = pytest.mark.gpu


def _in_edges_rotated(g, places):
    """g with every receiver's first `places` in-edges in another order (the first of them moved behind the last)."""
    order = np.argsort(g.dst, kind="stable")
    first = np.searchsorted(g.dst[order], np.arange(g.n_nodes))
    for n in np.flatnonzero(np.bincount(g.dst, minlength=g.n_nodes) >= places):
        order[first[n]:first[n] + places] = np.roll(order[first[n]:first[n] + places], -1)
    return dataclasses.replace(g, src=g.src[order], dst=g.dst[order], efeat=g.efeat[order])


def _run(model, w, graphs, min_us, monkeypatch):
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
    monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
    enc = xrl.Encoder(model, w)
    batch = enc.pack(synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))]))
    enc.encode(batch)
    emb = enc.encode(batch).cpu().numpy()
    nodes = [enc.batch_level(batch, r)[0] for r in range(model["rounds"] + 1)]
    batch.free()
    enc.close()
    return emb, nodes


@pytest.mark.parametrize("hidden,precision", [(64, "fp32"), (128, "bf16"), (256, "bf16")])
def test_first_two_in_edges_in_either_order(hidden, precision, monkeypatch):
    rng = np.random.Generator(np.random.PCG64(3))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, rounds=3)
    base = synth.resnet_dag(rng, 3)
    indeg = np.bincount(base.dst, minlength=base.n_nodes)
    assert (indeg == 2).any() and (indeg == 3).any()
    swapped, rotated = _in_edges_rotated(base, 2), _in_edges_rotated(base, 3)
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    one, two, three = ([base, base], [base, swapped], [base, swapped, rotated])
    nodes = {k: _run(model, w, g, "0", monkeypatch)[1] for k, g in (("one", one), ("two", two), ("three", three))}
    assert nodes["two"] == nodes["one"] and nodes["three"][0] > nodes["one"][0]
    assert np.array_equal(_run(model, w, three, "0", monkeypatch)[0], _run(model, w, three, "-1", monkeypatch)[0])


def _senders(rng, differ):
    """Receivers of two edges with the same attributes, from senders that differ in one thing only; behind each receiver a node.
    differ: their operator, their last dense attribute, their number of in-edges, or nothing but their senders' operators."""
    like = synth.resnet_dag(rng, 1)
    pairs, per = 12, 6                            # of a pair: two sources, two senders, the receiver, the node behind it
    n = pairs * per
    op = np.repeat(np.arange(pairs) % 12, per).astype(np.int32) * 2
    dense = np.zeros((n, like.dense.shape[1]), np.float32)
    src, dst = [], []
    for p in range(0, n, per):
        s, t, a, b, c, d = range(p, p + per)
        if differ == "operator":
            op[b] += 1
        if differ == "dense":
            dense[b, -1] = 1
        if differ == "senders":
            op[t] += 1
        edges = [(s, a), (t, b), (a, c), (b, c), (c, d)]
        if differ == "in-edges":
            edges.insert(2, (s, b))
        for x, y in edges:
            src.append(x)
            dst.append(y)
    src, dst = np.asarray(src, np.int32), np.asarray(dst, np.int32)
    return dataclasses.replace(like, op=op, dense=dense, layer=np.zeros(n, like.layer.dtype), block=np.zeros(n, like.block.dtype), src=src, dst=dst,
                               efeat=np.ones((len(src), like.efeat.shape[1]), np.float32))


@pytest.mark.parametrize("differ", ["operator", "dense", "in-edges", "senders"])
def test_the_senders_decide_between_edges_alike(differ, monkeypatch):
    """Edges with the same attributes are ordered by what their senders are, and keep their order where that says nothing: then a
    receiver whose two change places is another node than its copy."""
    rng = np.random.Generator(np.random.PCG64(4))
    model, _ = synth.make_config(1)
    model.update(hidden=128, precision="bf16", rounds=3)
    base = _senders(rng, differ)
    back = np.concatenate([np.flatnonzero(base.dst % 6 != 4), np.flatnonzero(base.dst % 6 == 4)[::-1]])   # (every receiver's two swapped)
    swapped = dataclasses.replace(base, src=base.src[back], dst=base.dst[back], efeat=base.efeat[back])
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    one, two = ([base, base], [base, swapped])
    (_, of_one), (emb, of_two) = _run(model, w, one, "0", monkeypatch), _run(model, w, two, "0", monkeypatch)
    if differ == "senders":
        assert of_two[:2] == of_one[:2] and of_two[2] == of_one[2] + 12 and of_two[3] == of_one[3] + 24, (of_one, of_two)
    else:
        assert of_two == of_one and max(of_one) <= base.n_nodes
    assert np.array_equal(emb, _run(model, w, two, "-1", monkeypatch)[0])
