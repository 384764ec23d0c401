"""The sender index, which the device makes for a backward pass: graphs whose counters lie in LDS and one too large
for that, senders of one to thousands of edges, quarters of a graph's edges that are not multiples of a wave,
small graphs. Through the backward pass (fp32, mask-stable weights) against the oracle."""
import dataclasses

import numpy as np
import pytest

import synth
from test_gpu_backward import run_stable_case, xrl  # noqa: F401

pytestmark = pytest.mark.gpu


def _with_hub(rng, g, n):
    """n more edges from node 0, to nodes that have few."""
    to = rng.choice(np.arange(1, g.n_nodes), n, replace=False).astype(np.int32)
    return dataclasses.replace(g, src=np.concatenate([g.src, np.zeros(n, np.int32)]), dst=np.concatenate([g.dst, to]),
                               efeat=np.concatenate([g.efeat, rng.standard_normal((n, g.efeat.shape[1])).astype(np.float32)]))


@pytest.mark.parametrize("nodes,hub", [([8193, 30], 3000), ([257, 30, 1, 64], 200)])
def test_sender_index(xrl, nodes, hub, monkeypatch):  # noqa: F811
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", "-1")
    rng = np.random.Generator(np.random.PCG64(21))
    model, _ = synth.make_config(1)
    model.update(hidden=64, precision="fp32", rounds=1)
    graphs = [synth.layered_dag(rng, n) for n in nodes]
    graphs[0] = _with_hub(rng, graphs[0], hub)
    state = synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))])
    run_stable_case(xrl, model, state, "fixed", max_nodes=max(g.n_nodes for g in graphs))
