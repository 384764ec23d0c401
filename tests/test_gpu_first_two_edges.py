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


@pytest.mark.parametrize("hidden,precision", [(64, "fp32"), (128, "bf16"), (256, "bf16")])
@pytest.mark.parametrize("alike", [False, True])
def test_first_two_in_edges_in_either_order(hidden, precision, alike, monkeypatch):
    """alike: all edges have the same attributes, so that the senders decide."""
    rng = np.random.Generator(np.random.PCG64(3))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, rounds=3)
    base = synth.resnet_dag(rng, 3)
    indeg = np.bincount(base.dst, minlength=base.n_nodes)
    assert (indeg == 2).any() and (indeg == 3).any()
    if alike:
        base = dataclasses.replace(base, efeat=np.ones_like(base.efeat))
    swapped, rotated = _in_edges_rotated(base, 2), _in_edges_rotated(base, 3)
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)

    def run(graphs, min_us):
        monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
        monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
        enc = xrl.Encoder(model, w)
        batch = enc.pack(synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))]))
        enc.encode(batch)
        emb = enc.encode(batch).cpu().numpy()
        nodes = [enc.batch_level(batch, r)[0] for r in range(4)]
        batch.free()
        enc.close()
        return emb, nodes

    one, two, three = ([base, base], [base, swapped], [base, swapped, rotated])
    nodes = {k: run(g, "0")[1] for k, g in (("one", one), ("two", two), ("three", three))}
    if alike:                                    # (senders alike in what is compared keep their order)
        assert nodes["two"][0] == nodes["one"][0] and all(x <= 2 * y for x, y in zip(nodes["two"], nodes["one"]))
    else:
        assert nodes["two"] == nodes["one"] and nodes["three"][0] > nodes["one"][0]
    assert np.array_equal(run(three, "0")[0], run(three, "-1")[0])
