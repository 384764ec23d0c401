"""A batch encoded once, forward only, in bf16 at H = 256: its levels are made on the device, one at a time, in
front of the round that runs on them. Embeddings have to be the bits of the whole batch's."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded ahead of the library)

import paper_2304_14698_amd as xrl
import synth
from test_gpu_distinct import _state

pytestmark = pytest.mark.gpu


def _embeddings(model, w, pack, min_us, monkeypatch):
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
    monkeypatch.setenv("XRL_PERSISTENT_MIN_ROWS", "0")
    enc = xrl.Encoder(model, w)
    enc.set_timing(True)
    got = []
    for _ in range(3):                       # (batches in turn: the levels' memory is used again)
        for state, edits in pack:
            batch = enc.pack_edits(state) if edits else enc.pack(state)
            got.append(enc.encode(batch).cpu().numpy())
            # (the memory made ready, then the level of the node-update layer and one a round)
            assert enc.read_timing("levels")[1] == (0 if min_us == "-1" else model["rounds"] + 2)
            batch.free()
    enc.close()
    return got


@pytest.mark.parametrize("readout,rounds", [("sum", 3), ("mean", 1)])
def test_levels_made_on_the_device(readout, rounds, monkeypatch):
    """Edge cases (see _edge_cases), several states, edits, and a state of one graph shape but for the order of edges:
    more nodes than a block of the level kernels takes, and fewer."""
    rng = np.random.Generator(np.random.PCG64(11))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="bf16", readout=readout, rounds=rounds)
    pack = [_state(kind, rng, model) for kind in ("edges", "resnet", "transformer", "edits")]
    w = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    whole = _embeddings(model, w, pack, "-1", monkeypatch)
    levels = _embeddings(model, w, pack, "0", monkeypatch)
    assert all(np.array_equal(a, b) for a, b in zip(whole, levels))


@pytest.mark.parametrize("save", [False, True])
def test_a_kept_batch_is_reduced_after_some_encodes(save):
    """Below the threshold of the first: the more an encode takes, the sooner; same bits before and after."""
    rng = np.random.Generator(np.random.PCG64(12))
    model, _ = synth.make_config(1)
    model.update(hidden=128, precision="bf16", rounds=5)
    state = synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 16), 90, by_block=True)])
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1))
    batch = enc.pack(state)
    us = 10 * 128 * (batch.N * 384 + batch.E * 392) / 7e8
    assert 30 < us < 300
    first, whole = enc.encode(batch, save_for_backward=save).cpu().numpy(), 1
    while enc.batch_level(batch, 0)[0] == batch.N and whole < 20:
        assert np.array_equal(enc.encode(batch, save_for_backward=save).cpu().numpy(), first)
        whole += 1
    assert whole == np.ceil(450 / (us * (3.0 if save else 0.8))) + 1
    assert np.array_equal(enc.encode(batch).cpu().numpy(), first)
    batch.free()
    enc.close()
