"""Class sums of one, two and four steps of sixteen rows a group: classes that end on a step's edge, begin in one step and end in
another, fill a group or several (the cases and criteria of test_gpu_class_sums.py)."""
import pytest

from test_gpu_class_sums import test_classes_of_copies as classes_of_copies

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [1, 2, 4])
@pytest.mark.parametrize("copies", [2, 16, 31, 33, 64, 300])
@pytest.mark.parametrize("hidden,precision", [(64, "fp32"), (128, "bf16"), (256, "bf16")])
def test_class_sum_steps(copies, hidden, precision, steps, monkeypatch):
    monkeypatch.setenv("XRL_SUM_STEPS", str(steps))
    classes_of_copies(copies, hidden, precision, monkeypatch)


def test_pool_gradient_by_column_slices(monkeypatch):
    """H = 256 and more graphs than an XCD's L2 holds rows of the pool's gradient for: gradients of the reduced batch
    against the whole one's (the bound of test_reduction_changes_nothing)."""
    import numpy as np
    import torch

    import paper_2304_14698_amd as xrl
    import synth
    rng = np.random.Generator(np.random.PCG64(21))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", rounds=2)
    base = [synth.layered_dag(rng, 11), synth.layered_dag(rng, 7)]
    graphs = [base[i % 3 == 0] for i in range(4099)]
    state = synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))])
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    up = torch.randn(len(graphs), 256, generator=torch.Generator().manual_seed(1)).cuda()
    got = []
    for min_us in ("-1", "0"):
        monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
        enc = xrl.Encoder(model, w)
        batch = enc.pack(state)
        emb = enc.encode(batch, save_for_backward=True)
        dw = torch.zeros(enc.n_weights, device="cuda")
        enc.encode_backward(batch, up, dw)
        got.append((emb, dw.double()))
        batch.free()
        enc.close()
    assert torch.equal(got[0][0], got[1][0])
    assert float((got[1][1] - got[0][1]).norm() / got[0][1].norm()) <= 2e-2
