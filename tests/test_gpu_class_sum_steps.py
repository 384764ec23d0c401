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


def test_column_slices_column_by_column(monkeypatch):
    """The same sums one column at a time: copies of one graph, whose upstream gradients are positive multiples of one row, so that
    no two terms of a column of the last node MLP's second bias gradient (the sum of the pool's gradient over the rows whose output is
    positive) have different signs. Rows rounded to bf16 one by one, or their sums: at most 2^-9 of each, so 2^-8 between the two."""
    import numpy as np
    import torch

    import paper_2304_14698_amd as xrl
    import synth
    rng = np.random.Generator(np.random.PCG64(22))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", rounds=2)
    graph = synth.layered_dag(rng, 18)
    state = synth.concat_states([([graph] * 4133, np.ones(4133, np.uint8))])
    layout = xrl.weight_layout(model)
    w = synth.init_weights(rng, layout, bias_range=0.1)
    g = torch.Generator().manual_seed(2)
    up = ((torch.rand(4133, 1, generator=g) + 0.5) * torch.randn(1, 256, generator=g)).cuda()
    got = []
    for min_us in ("-1", "0"):
        monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
        enc = xrl.Encoder(model, w)
        batch = enc.pack(state)
        enc.encode(batch, save_for_backward=True)
        assert (enc.batch_level(batch, 2)[0] < 32) == (min_us == "0")
        dw = torch.zeros(enc.n_weights, device="cuda")
        enc.encode_backward(batch, up, dw)
        got.append(dw.double().cpu().numpy())
        batch.free()
        enc.close()
    at = 0
    for name, shape in layout:
        if name == "node1.b1":
            break
        at += int(np.prod(shape))
    whole, reduced = (x[at:at + 256] for x in got)
    assert np.count_nonzero(whole) > 128
    assert np.all(np.abs(whole - reduced) <= (2.0 ** -8 + 1e-5) * np.abs(whole))
