"""The recomputing backward pass through the fused MLPs, a tile of 32 rows per block: batches of one node, of 31, 33 and 65
nodes and their in-edges, receivers of up to 40 in-edges, attributes of less than a slab, one and several, at every hidden
width, whole chain and encoder alone against the oracle at the fp32 criterion of test_gpu_backward.py."""
import numpy as np
import pytest

import synth
from test_gpu_backward import run_backward_case, xrl  # noqa: F401
from test_gpu_forward import weights_for
from test_gpu_round_launch import _graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,d_edge", [(64, 8), (64, 20), (128, 4), (128, 20), (256, 8)])
@pytest.mark.parametrize("sizes,degrees", [((1,), (0,)), ((31,), (1,)), ((33, 65), (0, 1, 2)), ((40,), (32, 0, 0, 5)), ((50,), (40, 1, 0, 0))])
def test_mlp_backward_tiles(xrl, hidden, d_edge, sizes, degrees):  # noqa: F811
    rng = np.random.Generator(np.random.PCG64(61))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="fp32", rounds=2, d_edge=d_edge)
    graphs = [_graph(rng, n, degrees, d_edge) for n in sizes]
    run_backward_case(xrl, model, synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))]), weights_for(model))


@pytest.mark.parametrize("kind", ["edge", "node"])
@pytest.mark.parametrize("hidden,rows", [(64, 97_000), (64, 190_000), (128, 65_000), (128, 196_000), (256, 32_600), (256, 163_000)])
@pytest.mark.parametrize("d_edge", [4, 16, 20, 40])
def test_mlp_backward_of_many_rows(xrl, hidden, rows, kind, d_edge):  # noqa: F811
    """bf16, as many rows as nearly fill one pass of the chip, or several, by four tiles a block: every copy of a graph of some 300 nodes gets
    the bits that it gets alone, a tile a block."""
    import torch
    rng = np.random.Generator(np.random.PCG64(62))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="bf16", rounds=1, d_edge=d_edge)
    graph = _graph(rng, 301, (0, 1, 2, 3, 33, 1, 1), d_edge)
    copies = rows // (graph.n_edges if kind == "edge" else graph.n_nodes)
    enc = xrl.Encoder(model, weights_for(model))
    one, many = (enc.pack(synth.concat_states([([graph] * n, np.ones(n, np.uint8))])) for n in (1, copies))
    g = torch.Generator().manual_seed(1)
    h, agg, y, dy = (torch.randn(graph.n_nodes, hidden, generator=g).relu().bfloat16().cuda() for _ in range(4))
    dy -= 0.5
    kw = {} if kind == "edge" else dict(agg=agg, y=y)
    alone = enc.mlp_backward(one, kind, 0, h, dy, **kw)
    all_ = enc.mlp_backward(many, kind, 0, h.repeat(copies, 1), dy.repeat(copies, 1), **{k: v.repeat(copies, 1) for k, v in kw.items()})
    for k, v in all_.items():
        assert torch.equal(v.view(copies, -1, hidden), alone[k].expand(copies, -1, -1)), k
    one.free()
    many.free()
    enc.close()
