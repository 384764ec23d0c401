"""The pool's gradient by windows of graphs (1, 4 and 16 consecutive ones): classes that lie in every graph, in runs with gaps, twice
in a graph, in one graph; runs that begin and end inside, at the end of and across a wave's 64 places. The same sums as row by
row in another order, in fp32: n terms of either order err by at most n * 2^-24 of the sum of their absolute values, and by about
the root of that; the largest class here has 700 terms: 2^-24 * 700 = 4.2e-5 of a sum that does not cancel, asserted at a quarter of it on the
whole gradient. In bf16 the sums are rounded to 2^-9 once per class either way."""
import dataclasses

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def states_of_repeated_graphs(rng):
    """Three base graphs over and over, by themselves and in runs; one that holds the first twice; a few of their own."""
    base = [synth.layered_dag(rng, n) for n in (11, 7, 5)]
    b, n = base[0], base[0].n_nodes
    two = lambda x: np.concatenate([x, x])
    twice = dataclasses.replace(b, op=two(b.op), dense=two(b.dense), layer=two(b.layer), block=two(b.block), efeat=two(b.efeat),
                                src=np.concatenate([b.src, b.src + n]), dst=np.concatenate([b.dst, b.dst + n]))
    graphs = [base[0]] * 333 + [base[int(i)] for i in rng.integers(0, 3, 200)] + [base[i % 17 == 0] for i in range(163)]
    graphs[40] = graphs[41] = graphs[350] = twice                # classes with two places in a graph
    graphs += [synth.layered_dag(rng, 6) for _ in range(9)]      # classes of one graph
    return synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))])


def gradients(model, w, state, up, window_nodes, monkeypatch):
    import torch

    import paper_2304_14698_amd as xrl
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", "0")
    monkeypatch.setenv("XRL_POOL_WINDOW_NODES", window_nodes)
    enc = xrl.Encoder(model, w)
    batch = enc.pack(state)
    enc.encode(batch, save_for_backward=True)
    assert enc.batch_level(batch, model["rounds"])[0] < len(state["node_op"]) // 4
    dw = torch.zeros(enc.n_weights, device="cuda")
    enc.encode_backward(batch, up, dw)
    batch.free()
    enc.close()
    return dw


def identity_readout(model, w):
    """Weights under which the readout MLP hands an upstream gradient through unchanged: identity matrices, biases that keep every unit on (the
    pool is a sum of states behind a ReLU)."""
    import paper_2304_14698_amd as xrl
    w, at, H = w.copy(), 0, model["hidden"]
    for name, shape in xrl.weight_layout(model):
        n = int(np.prod(shape))
        if name.startswith("readout.W"):
            w[at:at + n] = np.eye(shape[0], H, dtype=np.float32).ravel()
        elif name.startswith("readout.b"):
            w[at:at + n] = 1.0
        at += n
    return w


@pytest.mark.parametrize("readout", ["sum", "mean"])
@pytest.mark.parametrize("hidden,precision", [(64, "fp32"), (128, "fp32"), (256, "fp32"), (64, "bf16"), (128, "bf16"), (256, "bf16")])
def test_pool_gradient_by_windows(hidden, precision, readout, monkeypatch):
    """Windows are for rows of 256 columns: narrower ones take the class sums' order whatever the threshold, so the same bits."""
    import torch

    import paper_2304_14698_amd as xrl
    rng = np.random.Generator(np.random.PCG64(hidden))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, rounds=2, readout=readout)
    state = states_of_repeated_graphs(rng)
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    up = torch.randn(len(state["slot_mask"]), hidden, generator=torch.Generator().manual_seed(1)).cuda()
    got = [gradients(model, w, state, up, nodes, monkeypatch) for nodes in ("0", "1000000000")]
    assert got[1].any()
    if hidden < 256:
        assert torch.equal(*got)
    got = [x.double() for x in got]
    assert float((got[0] - got[1]).norm() / got[1].norm()) <= (1e-5 if precision == "fp32" else 2e-2)


@pytest.mark.parametrize("readout", ["sum", "mean"])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_sums_that_are_exact(precision, readout, monkeypatch):
    """Gradients of the pool that are whole numbers up to 8 (times a graph's node count for the mean, which divides by it): every sum of at most
    700 of them is exact in fp32 in any order, so both ways give the same bits throughout, a place too few or too many on either side shows."""
    import torch

    import paper_2304_14698_amd as xrl
    rng = np.random.Generator(np.random.PCG64(2))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision=precision, rounds=2, readout=readout)
    state = states_of_repeated_graphs(rng)
    w = identity_readout(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1))
    up = rng.integers(-8, 9, (len(state["slot_mask"]), 256)).astype(np.float32)
    if readout == "mean":
        up *= np.diff(state["graph_node_ptr"])[:, None].astype(np.float32)
    got = [gradients(model, w, state, torch.from_numpy(up).cuda(), nodes, monkeypatch) for nodes in ("0", "1000000000")]
    assert got[0].any() and torch.equal(*got)
