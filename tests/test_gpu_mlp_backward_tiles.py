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
