"""Attention rounds at the edges of their kernels: receivers of no, one, two (requested together) and more in-edges,
node counts around a 32-row tile, a lone node; every width. Forward and backward against the oracle, at the
criteria of test_gpu_backward.py for attention rounds. In bf16 there are as many such graphs that a ReLU mask which
the forward's rounding turns over is a small share of a gradient."""
import dataclasses

import numpy as np
import pytest

import synth
from test_gpu_backward import run_backward_case, xrl  # noqa: F401
from test_gpu_forward import weights_for

pytestmark = pytest.mark.gpu


def _graph(rng, n, degrees):
    """n nodes; node i has degrees[i % len] in-edges from other nodes."""
    g = synth.layered_dag(rng, n)
    n = g.n_nodes
    dst = np.repeat(np.arange(n), [min(degrees[i % len(degrees)], n - 1) for i in range(n)]).astype(np.int32)
    src = ((dst + 1 + rng.integers(0, max(n - 1, 1), len(dst))) % n).astype(np.int32)
    order = rng.permutation(len(dst))
    feat = rng.standard_normal((len(dst), g.efeat.shape[1])).astype(np.float32)
    return dataclasses.replace(g, src=src[order], dst=dst[order], efeat=feat)


@pytest.mark.parametrize("hidden,precision", [(64, "fp32"), (128, "fp32"), (256, "fp32"), (64, "bf16"), (128, "bf16"), (256, "bf16")])
def test_attention_edge_cases(xrl, hidden, precision):  # noqa: F811
    rng = np.random.Generator(np.random.PCG64(31))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, round_kind="gat", rounds=2)
    kinds = ((27, (0, 1, 2, 3, 5)), (33, (1,)), (64, (2,)), (1, (0,)), (40, (0, 0, 40)))
    graphs = [_graph(rng, n, d) for _ in range(1 if precision == "fp32" else 40) for n, d in kinds]
    state = synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))])
    run_backward_case(xrl, model, state, weights_for(model), bf16_rel=0.3, bf16_cos=0.95)
