"""Sums per class of a reduced batch's gradients: classes of a few rows up to several hundred, inside a group of sixteen
rows, across two and across many (copies of one graph are one class per node). Against the batch taken whole, at the
criteria of test_gpu_distinct.py: fp32, sums of thousands of products in another order; bf16, a class's gradient
rounded once where each of its nodes' was."""
import numpy as np
import pytest

import paper_2304_14698_amd as xrl
import synth
from test_gpu_distinct import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [2, 7, 8, 15, 16, 17, 33, 700])
@pytest.mark.parametrize("hidden,precision", [(64, "fp32"), (256, "fp32"), (64, "bf16"), (128, "bf16"), (256, "bf16")])
def test_classes_of_copies(copies, hidden, precision, monkeypatch):
    import torch
    rng = np.random.Generator(np.random.PCG64(11))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision=precision, rounds=2)
    a, b = synth.layered_dag(rng, 21), synth.layered_dag(rng, 30)
    state = synth.concat_states([([a] * copies + [b], np.ones(copies + 1, np.uint8))])
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    got = {}
    for min_us in ("-1", "0"):                      # whole, reduced
        monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
        monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
        if precision == "bf16":
            monkeypatch.setenv("XRL_PERSISTENT_MIN_ROWS", "0")
        enc = xrl.Encoder(model, w)
        batch = enc.pack(state)
        up = torch.tensor(np.random.default_rng(3).standard_normal((batch.G, hidden)), dtype=torch.float32, device="cuda")
        got[min_us] = _run(enc, batch, up, model["rounds"])
        assert (enc.batch_level(batch, 0)[0] < batch.N) == (min_us == "0")
        batch.free()
        enc.close()
    (fa, da), (fb, db) = got["-1"], got["0"]
    for k in fa:
        assert np.array_equal(fa[k], fb[k]), k
    assert np.linalg.norm(da - db) <= (1e-5 if precision == "fp32" else 2e-2) * np.linalg.norm(da)
