"""The fp32 edge and node MLPs at H = 128, whose products run on bf16 parts: tiles of one row and of 31, 32, 33, receivers
of up to 32 in-edges and beyond (pieces carried between tiles), attributes of less than a slab, one and two. Every
intermediate and output against the oracle at the fp32 criterion of test_gpu_forward.py; and the embeddings' error over
a state as a whole, which may not exceed what sums in fp32 show (2^-24 times the square root of the roundings a value
has met, about 100 in each of the 2 R + 2 layers of fp32 instructions: 4e-7 at R = 3)."""
import numpy as np
import pytest

import synth
from oracle import xrl_oracle as O
from test_gpu_forward import oracle_model, run_case, weights_for, xrl  # noqa: F401
from test_gpu_round_launch import _graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_edge", [4, 8, 20])
@pytest.mark.parametrize("sizes,degrees", [((1,), (0,)), ((31,), (1,)), ((33, 65), (0, 1, 2)), ((40,), (32, 0, 0, 5)), ((50,), (40, 1, 0, 0))])
def test_split_products(xrl, d_edge, sizes, degrees):  # noqa: F811
    rng = np.random.Generator(np.random.PCG64(51))
    model, _ = synth.make_config(1)
    model.update(hidden=128, precision="fp32", rounds=2, d_edge=d_edge)
    graphs = [_graph(rng, n, degrees, d_edge) for n in sizes]
    run_case(xrl, model, synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))]), weights_for(model))


def test_split_products_error(xrl):  # noqa: F811
    rng = np.random.Generator(np.random.PCG64(52))
    model, _ = synth.make_config(1)
    model.update(hidden=128, precision="fp32", rounds=3)
    graphs, mask = synth.make_state(rng, synth.resnet_dag(rng, 4), 8, by_block=True)
    state, w = synth.concat_states([(graphs, mask)]), weights_for(model)
    enc = xrl.Encoder(model, w)
    got = enc.encode(enc.pack(state)).cpu().numpy().astype(np.float64)
    ref = O.encode(oracle_model(model), w, state)
    assert np.linalg.norm(got - ref) <= 4e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("where", ["attribute", "first weights", "second weights", "overflow"])
def test_split_products_of_values_without_parts(xrl, where):  # noqa: F811
    """Finite values of 2^128 (1 - 2^-9) and above, which no bf16 part can hold, as an edge attribute (in some rows of
    a tile alone), in the weights of either layer, and a first layer that overflows. What is multiplied with them is
    small, or zero, so that every other value is of ordinary size."""
    rng = np.random.Generator(np.random.PCG64(53))
    model, _ = synth.make_config(1)
    model.update(hidden=128, precision="fp32", rounds=2)
    g = _graph(rng, 70, (2, 1, 0, 3), 8)
    state = synth.concat_states([([g], np.ones(1, np.uint8))])
    layout, w = xrl.weight_layout(model), weights_for(model).copy()
    at, o = {}, 0
    for name, shape in layout:
        at[name] = w[o:o + int(np.prod(shape))].reshape(shape)
        o += int(np.prod(shape))
    big = np.float32(3.4e38)
    feat = state["edge_feat"]
    feat[:, 0] = 0.0
    if where in ("attribute", "overflow"):
        feat[7::23, 0] = big
        at["embed.W0"][0] = 0.0
        for r in range(model["rounds"]):
            at[f"edge{r}.W0"][256] = 1e-37 * rng.standard_normal(128)
    if where == "overflow":                       # one hidden feature far beyond fp32, which switches the row's outputs off
        at["edge0.W0"][256, 5] = 3.0
        at["edge0.W1"][5] = -np.abs(at["edge0.W1"][5]) - 0.01
    if where == "first weights":                  # times an attribute of zero or 2e-38 (6.8)
        at["edge0.W0"][256, 9] = big
        feat[3::11, 0] = 2e-38
    if where == "second weights":                 # of a hidden feature that is always off
        at["node1.W0"][:, 77] = 0.0
        at["node1.b0"][77] = -1.0
        at["node1.W1"][77, 40] = -big
    run_case(xrl, model, state, w)
