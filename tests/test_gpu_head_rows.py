"""Both heads at the edges of a policy block's sixteen slots: the last block full, of one slot and of fifteen, states of one slot (several
in a block), states that begin or end inside a block or fill it, states of 64 slots (a wave's softmax) and of 65 (the block's), several states
to a block of the value head, widths of 16-byte columns and of single ones. Against the float64
oracle: a dot of n fp32 terms errs by at most n * 2^-24 of the sum of their absolute values, here three layers of at most 512
terms, and by far less as it is summed in four chains: 2e-5 of the largest value. A state's results do not depend on the batch around it."""
import numpy as np
import pytest

import synth
from oracle import xrl_oracle as O
from test_gpu_forward import heads_only_state, oracle_model, weights_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,heads,n_states,n_cand", [
    (128, None, 127, 0), (64, None, 43, 4), (256, None, 1, 128), (128, (100, 35), 3, 42),
    (64, None, 1023, 0), (128, None, 93, 10), (128, (100, 35), 206, 4), (256, None, 6, 205),
    (128, None, 4, 15), (64, None, 2, 16), (256, None, 2, 63), (64, (100, 35), 2, 64), (256, None, 1040, 0),
    (64, (300, 140), 6, 60), (256, (512, 512), 14, 20), (128, (40, 200), 4, 70)])    # alone a slot a block, with the others sixteen
def test_heads_at_rows_per_block(hidden, heads, n_states, n_cand):
    import torch
    import paper_2304_14698_amd as xrl
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="fp32")
    if heads:
        model.update(head_hidden=heads)
    rng = np.random.Generator(np.random.PCG64(7 * n_states + n_cand))
    if n_cand == 0:                                             # n_states states of one slot
        state = heads_only_state(rng, model, 1, n_states - 1, fixed=True)
        state.update(n_states=n_states, state_graph_ptr=np.arange(n_states + 1, dtype=np.int32), slot_mask=np.ones(n_states, np.uint8))
    else:
        state = heads_only_state(rng, model, n_states, n_cand, fixed=n_states % 2 == 0 or n_states == 1)
    G, w, om = len(state["slot_mask"]), weights_for(model), oracle_model(model)
    emb = rng.standard_normal((G, hidden)).astype(np.float32)
    enc = xrl.Encoder(model, w)
    run = lambda st, e: {k: v.cpu().numpy() for k, v in enc.policy_value(enc.pack(st), torch.from_numpy(e).cuda()).items()}
    got = run(state, emb)
    ref = O.policy_value(om, w, emb.astype(np.float64), state)
    valid = state["slot_mask"].astype(bool)
    for k in ("logp", "entropy", "value"):
        a, r = (np.asarray(x[k], np.float64) for x in (got, ref))
        a, r = (a[valid], r[valid]) if k == "logp" else (a, r)
        assert np.abs(a - r).max() <= 2e-5 * max(1.0, np.abs(r).max()), k
    assert np.isneginf(got["logp"][~valid]).all()
    sgp = state["state_graph_ptr"]
    logit = np.asarray(ref["logit"], np.float64)
    for s in range(n_states):
        a, z = sgp[s], sgp[s + 1]
        best = np.where(valid[a:z], logit[a:z], -np.inf)
        assert best[got["action"][s]] >= best.max() - 4e-5 * max(1.0, np.abs(logit).max())
    s = n_states // 2
    a, z = sgp[s], sgp[s + 1]
    one = dict(state, n_states=1, state_graph_ptr=np.array([0, z - a], np.int32),
               graph_node_ptr=np.arange(z - a + 1, dtype=np.int32), graph_edge_ptr=np.zeros(z - a + 1, np.int32),
               node_op=state["node_op"][a:z], node_dense=state["node_dense"][a:z], graph_global=state["graph_global"][a:z],
               slot_mask=state["slot_mask"][a:z])
    alone = run(one, emb[a:z])
    assert np.array_equal(alone["logp"], got["logp"][a:z]) and alone["value"][0] == got["value"][s]
    assert alone["entropy"][0] == got["entropy"][s] and alone["action"][0] == got["action"][s]
