"""Weight-gradient products of several layers in one launch: widths of the edge attributes at the edge of
the tile's extra columns, both operand types at every hidden width, more products than one launch takes,
and so little room for gradients that every MLP is launched by itself. Criteria: those of
test_gpu_weight_gradient.py (the product against float64 on the same operands) and test_gpu_backward.py (the
backward pass against the oracle, fp32)."""
import numpy as np
import pytest

import synth
from test_gpu_backward import run_backward_case
from test_gpu_forward import weights_for
from test_gpu_weight_gradient import run, xrl  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,precision,d_edge,wide", [
    (64, "fp32", 8, False), (256, "fp32", 4, False),
    (128, "bf16", 28, False),                      # 28 attributes and the bias fill 29 of the 32 extra columns
    (64, "bf16", 32, False), (128, "fp32", 32, False), (256, "bf16", 28, True), (256, "bf16", 60, True),
    (128, "bf16", 132, False)])                    # ... from 32 on a product of their own; 132 + 1 need two tiles
def test_weight_gradient_edge_attribute_widths(xrl, hidden, precision, d_edge, wide, monkeypatch):  # noqa: F811
    if wide:
        monkeypatch.setenv("XRL_WGRAD_WIDE_MIN_ROWS", "0")
    model, state = synth.make_config(4, n_cand=2)
    model.update(hidden=hidden, precision=precision, d_edge=d_edge)
    rng = np.random.Generator(np.random.PCG64(9))
    state = dict(state, edge_feat=rng.standard_normal((len(state["edge_src"]), d_edge)).astype(np.float32))
    run(xrl, model, state, n_plain=65)


@pytest.mark.parametrize("room", ["0", None])
def test_backward_of_more_products_than_one_launch_takes(xrl, room, monkeypatch):  # noqa: F811
    if room is not None:
        monkeypatch.setenv("XRL_GRAD_ROOM", room)
    model, state = synth.make_config(1)
    model.update(rounds=7)                         # 30 products; a launch takes 24
    run_backward_case(xrl, model, state, weights_for(model))
