"""fp32 encodes of a reduced batch, forward only, read the states of the level below by index: the same bits as from a copy of each
class's state (the saving encode of the same batch) and as the whole batch, rows that are computed once more without parts
among them (H = 128: values next to the largest float and beyond)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 1e34, 1e36])
@pytest.mark.parametrize("hidden,rounds", [(64, 3), (128, 5), (256, 2)])
def test_states_of_the_level_below(hidden, rounds, scale, monkeypatch):
    import torch

    import paper_2304_14698_amd as xrl
    rng = np.random.Generator(np.random.PCG64(hidden))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="fp32", rounds=rounds)
    base = synth.transformer_dag(rng, 3)
    state = synth.concat_states([synth.make_state(rng, base, 40, by_block=True)])
    layout = xrl.weight_layout(model)
    w = synth.init_weights(rng, layout, bias_range=0.1)
    at = 0
    for name, shape in layout:
        n = int(np.prod(shape))
        if name == "embed.W1":
            w[at:at + n] *= np.float32(scale)
        at += n
    embs = []
    for min_us in ("-1", "0"):
        monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
        enc = xrl.Encoder(model, w)
        batch = enc.pack(state)
        embs += [enc.encode(batch, save_for_backward=save).clone() for save in (False, True, False)]
        assert (enc.batch_level(batch, rounds)[0] < len(state["node_op"]) // 2) == (min_us == "0")
        batch.free()
        enc.close()
    nan = torch.isnan(embs[0])
    for e in embs[1:]:
        assert torch.equal(torch.isnan(e), nan) and torch.equal(e[~nan], embs[0][~nan])


def test_levels_read_by_index_need_no_room_for_copies(monkeypatch):
    """The encode that reduces a batch to levels as large as the batch itself -- no two nodes alike, H = 256, one round -- takes the levels' own
    memory, 303 bytes a node, and no more workspace than the whole batch had (copies of the states would be 1 KB a node, of which the whole
    batch's plan has room for 440 bytes: 887 in all)."""
    import torch

    import paper_2304_14698_amd as xrl
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", "0")
    rng = np.random.Generator(np.random.PCG64(1))
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="fp32", rounds=1)
    graphs = [synth.layered_dag(rng, 50) for _ in range(1900)]
    state = synth.concat_states([(graphs, np.ones(len(graphs), np.uint8))])
    n = len(state["node_op"])
    enc = xrl.Encoder(model, synth.init_weights(rng, xrl.weight_layout(model)))
    batch = enc.pack(state)
    free, embs = [], []
    for _ in range(2):
        embs.append(enc.encode(batch))
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
        level = enc.batch_level(batch, 1)[0]
    assert level > 0.9 * n and torch.equal(*embs)
    assert free[0] - free[1] < 450 * n, (free, n)
    batch.free()
    enc.close()
