"""Attention rounds that aggregate and form the next round's product in one launch: the bits of the two kernels
that larger batches run, kept for the backward pass or not, for any number of rounds."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded ahead of the library)

import paper_2304_14698_amd as xrl
import synth
from test_gpu_attention_edges import _graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,precision", [(64, "fp32"), (64, "bf16"), (128, "bf16")])
@pytest.mark.parametrize("rounds", [1, 2, 3, 4])
def test_rounds_in_one_launch(hidden, precision, rounds):
    rng = np.random.Generator(np.random.PCG64(33))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, round_kind="gat", rounds=rounds)
    kinds = [(27, (0, 1, 2, 3, 5)), (33, (1,)), (64, (2,)), (1, (0,)), (40, (0, 0, 40)), (300, (3, 1))]
    few = [_graph(rng, n, d) for n, d in kinds]
    more = few + [synth.layered_dag(rng, 600) for _ in range(3)]
    long = synth.layered_dag(rng, 3400)
    some, many, big = (few + [long] * n for n in (6, 17, 20))
    # a launch has two blocks a compute unit, 512 of them, and a tile is 32 rows: `some` two tiles for some of the blocks, `many` three or
    # four for each (both tile buffers written and read again, the product passed from wave to wave), `big` more nodes than such a
    # launch takes; the last tile partly filled
    nodes = {k: sum(g.n_nodes for g in v) for k, v in dict(more=more, some=some, many=many, big=big).items()}
    assert nodes["more"] < 8192 and 16384 < nodes["some"] < 2 * 16384 and 3 * 16384 < nodes["many"] < 65536 < nodes["big"], nodes
    assert nodes["some"] % 32 and nodes["many"] % 32
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1))
    got = []
    for graphs in (few, more, big, some, many, few[3:4]):
        batch = enc.pack(synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))]))
        embs = [enc.encode(batch, save_for_backward=save).cpu().numpy() for save in (False, True, False)]
        assert all(np.array_equal(e, embs[0]) for e in embs)
        got.append(embs[0])
        batch.free()
    n = len(few)
    assert all(np.array_equal(e[:n], got[0]) for e in got[1:-1]) and np.array_equal(got[-1], got[0][3:4])
    assert all(np.array_equal(e[n:], np.broadcast_to(got[2][n], e[n:].shape)) for e in got[2:5])     # (copies of one graph)
    enc.close()
