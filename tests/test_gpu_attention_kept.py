"""Attention rounds: the node-update layer's backward from what the persistent forward kept against the one
that recomputes its first layer. Both start from the same stored states; they round the same
intermediate rows and differ in the order of the weight gradients' sums: bf16 rounding, 2e-2."""
import numpy as np
import pytest

import paper_2304_14698_amd as xrl
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,n_cand,layers", [(64, 3, 2), (128, 11, 2), (128, 1, 1), (256, 6, 2)])
def test_embed_backward_from_the_kept_forward(hidden, n_cand, layers, monkeypatch):
    import torch
    rng = np.random.Generator(np.random.PCG64(3))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="bf16", rounds=2, round_kind="gat", mlp_layers=layers)
    state = synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 3), n_cand, by_block=True)])
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    got = {}
    for rows in ("0", "1000000000"):                # kept, recomputed
        monkeypatch.setenv("XRL_PERSISTENT_MIN_ROWS", rows)
        enc = xrl.Encoder(model, w)
        batch = enc.pack(state)
        up = torch.tensor(np.random.default_rng(3).standard_normal((batch.G, hidden)), dtype=torch.float32, device="cuda")
        emb = enc.encode(batch, save_for_backward=True)
        dw = torch.zeros(enc.n_weights, dtype=torch.float32, device="cuda")
        enc.encode_backward(batch, up, dw)
        got[rows] = emb.cpu().numpy(), dw.cpu().numpy().astype(np.float64)
        batch.free()
        enc.close()
    (ea, da), (eb, db) = got.values()
    assert np.array_equal(ea, eb)
    n = dict((name, np.prod(shape)) for name, shape in xrl.weight_layout(model))
    o = 0
    for name, size in n.items():
        x, y = da[o:o + size], db[o:o + size]
        o += int(size)
        assert np.linalg.norm(x - y) <= 2e-2 * max(np.linalg.norm(y), 1e-3 * np.linalg.norm(db)), name
