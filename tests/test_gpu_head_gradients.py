"""Heads backward at the row counts where its launches change shape: rows per block of the row-MLP
backward (1, 2, 4, 8), chunks of 64 rows and their remainders in the weight gradients, layers of
one chunk beside layers of many. Against the float64 oracle, every tensor by itself: 1e-5 of its norm
and, for sums that cancel (the last bias: the gradients of a softmax's logits sum to zero), the heads'
kappa of grad_checks times the norm of the sums of absolute terms."""
import numpy as np
import pytest

import grad_checks as GC
import synth
from oracle import xrl_oracle as O
from test_gpu_forward import heads_only_state, oracle_model, weights_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,n_states,n_cand", [(64, 1, 0), (64, 1, 62), (128, 1, 63), (64, 1, 64), (256, 2, 254), (128, 2, 255),
                                                    (64, 1, 1022), (128, 1, 1023), (64, 23, 88), (64, 1, 2048), (128, 70, 70)])
def test_head_gradients_at_row_counts(hidden, n_states, n_cand):
    import torch
    import paper_2304_14698_amd as xrl
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="fp32")
    rng = np.random.Generator(np.random.PCG64(100 + n_cand))
    state = heads_only_state(rng, model, n_states, n_cand, fixed=True)
    G, w, om = len(state["slot_mask"]), weights_for(model), oracle_model(model)
    emb = rng.standard_normal((G, hidden)).astype(np.float32)
    dlogp = (rng.standard_normal(G) * state["slot_mask"]).astype(np.float32)
    dvalue, dentropy = (rng.standard_normal(n_states).astype(np.float32) for _ in range(2))
    enc = xrl.Encoder(model, w)
    batch = enc.pack(state)
    t = lambda x: torch.from_numpy(x).cuda()
    dw = torch.zeros(enc.n_weights, dtype=torch.float32, device="cuda")
    demb = enc.policy_value_backward(batch, t(emb), t(dlogp), t(dvalue), t(dentropy), dw)
    bound = O.zero_grads(om)
    ref_demb, ref_dw = O.policy_value_backward(om, w, emb.astype(np.float64), state, dlogp, dvalue, dentropy, bound=bound)
    assert np.linalg.norm(demb.cpu().numpy() - ref_demb) <= 1e-5 * np.linalg.norm(ref_demb)
    got, bound = dw.cpu().numpy().astype(np.float64), O.flatten(om, bound)
    L = float(np.abs(O.policy_value(om, w, emb.astype(np.float64), state)["logit"]).max())
    for name, sl, _ in GC.tensors(om):
        err = np.linalg.norm(got[sl] - ref_dw[sl])
        if not name.startswith(("policy", "value")):
            assert err == 0, name
            continue
        tol = 1e-5 * np.linalg.norm(ref_dw[sl]) + (2e-6 + 1e-5 * max(1.0, L)) * np.linalg.norm(bound[sl])
        assert err <= tol, (name, err, tol)
