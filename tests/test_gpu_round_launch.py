"""A message-passing round in one launch (forward only, bf16, small batches): the bits of the two launches it stands
for, with receivers of every in-degree up to the 32 edges of a pass, passes cut short by a receiver that does not
fit, batches around the nodes of a block, attributes wider than a slab, and a receiver of more than 32
in-edges, which keeps the two launches."""
import dataclasses

import numpy as np
import pytest

import paper_2304_14698_amd as xrl
import synth

pytestmark = pytest.mark.gpu


def _graph(rng, n, degrees, d_edge):
    g = synth.layered_dag(rng, n)
    n = g.n_nodes
    dst = np.repeat(np.arange(n), [min(degrees[i % len(degrees)], 40) for i in range(n)]).astype(np.int32)
    src = rng.integers(0, n, len(dst)).astype(np.int32)
    order = rng.permutation(len(dst))
    return dataclasses.replace(g, src=src[order], dst=dst[order], efeat=rng.standard_normal((len(dst), d_edge)).astype(np.float32))


@pytest.mark.parametrize("hidden,d_edge,rounds", [(64, 8, 2), (128, 8, 3), (128, 20, 2), (64, 4, 1)])
@pytest.mark.parametrize("sizes", [(1,), (15,), (16, 17), (28, 300), (50,) * 100, (4000, 3200), (13000,)])
def test_round_in_one_launch_equals_two(hidden, d_edge, rounds, sizes, monkeypatch):
    import torch  # noqa: F401  (its runtime is loaded first)
    rng = np.random.Generator(np.random.PCG64(41))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="bf16", rounds=rounds, d_edge=d_edge)
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    for degrees in ((0,), (1,), (0, 1, 2), (31, 1, 1), (32, 0, 0, 5), (17, 16, 3, 0), (33, 1, 0, 1)):
        graphs = [_graph(rng, n, degrees, d_edge) for n in sizes]
        state = synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))])
        got = []
        for blocks in ("0", "1000"):
            monkeypatch.setenv("XRL_ROUND_BLOCKS", blocks)
            enc = xrl.Encoder(model, w)
            batch = enc.pack(state)
            enc.set_timing(True)
            got.append(enc.encode(batch).cpu().numpy())
            small = max(batch.N, batch.E) < 32768
            assert (enc.read_timing("round")[1] > 0) == (blocks != "0" and 33 not in degrees and small)
            batch.free()
            enc.close()
        assert np.array_equal(got[0], got[1]), degrees


@pytest.mark.parametrize("hidden", [64, 128])
@pytest.mark.parametrize("degrees,one", [((1,), True), ((0, 2, 4, 2), True), ((4, 4, 5, 4), True), ((8, 0), True), ((6,), False), ((10, 0), False), ((30,), False), ("cluster", False)])
def test_dense_receivers_keep_two_launches(hidden, degrees, one, monkeypatch):
    """A block's in-edges go 32 at a time, one pass after the other: where its nodes have more than 72, in one block of
    the batch too, the edges have a launch of their own."""
    import torch  # noqa: F401
    monkeypatch.delenv("XRL_ROUND_BLOCKS", raising=False)
    rng = np.random.Generator(np.random.PCG64(43))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="bf16", rounds=2)
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1))
    degrees = [1] * 500 + [16] * 8 + [1] * 600 if degrees == "cluster" else degrees
    graphs = [_graph(rng, 1000, degrees, model["d_edge"])]
    batch = enc.pack(synth.concat_states([(graphs, np.ones(1, np.uint8))]))
    enc.set_timing(True)
    enc.encode(batch)
    assert (enc.read_timing("round")[1] > 0) == one
    batch.free()
    enc.close()
