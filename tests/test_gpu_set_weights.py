"""New weights in a context that already has some (xrl_set_weights): the context then computes what a
context created with them computes, bit for bit, forward and backward, whatever is still queued with
the old ones; a vector with a value that is not finite is refused and leaves the old weights."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,precision,round_kind,layers", [(64, "fp32", "mlp", 2), (128, "bf16", "mlp", 1), (256, "bf16", "mlp", 2),
                                                                (64, "bf16", "gat", 2), (128, "fp32", "gat", 1)])
def test_new_weights(hidden, precision, round_kind, layers):
    import torch
    import paper_2304_14698_amd as xrl
    model, state = synth.make_config(2, n_cand=3)
    model.update(hidden=hidden, precision=precision, round_kind=round_kind, mlp_layers=layers, rounds=3)
    rng = np.random.Generator(np.random.PCG64(hidden))
    w = [synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1) for _ in range(3)]
    demb = torch.from_numpy(rng.standard_normal((4, hidden)).astype(np.float32)).cuda()

    def outputs(enc, batch):
        emb = enc.encode(batch, save_for_backward=True)
        pv = enc.policy_value(batch, emb)
        dw = torch.zeros(enc.n_weights, device="cuda")
        enc.encode_backward(batch, demb, dw)
        return [emb, pv["logit"], pv["value"], dw]

    want = []
    for x in w:
        enc = xrl.Encoder(model, x)
        want.append([t.cpu() for t in outputs(enc, enc.pack(state))])
        enc.close()
    assert not torch.equal(want[0][0], want[1][0])
    enc = xrl.Encoder(model, w[0])
    batch = enc.pack(state)
    got = [outputs(enc, batch)]
    for x in (w[1], w[2], w[1]):                 # back to back: nothing waits in between
        keep = x.copy()
        enc.set_weights(keep)
        keep[:] = np.nan                         # the caller's vector is free on return
        got.append(outputs(enc, batch))
    for at in (0, enc.n_weights // 2, enc.n_weights - 1):
        bad = w[2].copy()
        bad[at] = np.inf
        with pytest.raises(xrl.XrlError) as e:
            enc.set_weights(bad)
        assert e.value.code == xrl.ERR["VALUE"] and f"[{at}]" in str(e.value)
    got.append(outputs(enc, batch))
    for g, i in zip(got, (0, 1, 2, 1, 1)):
        for a, b in zip(g, want[i]):
            assert torch.equal(a.cpu(), b)
    enc.close()


def test_refused_while_the_stream_is_captured():
    """A captured copy would send whatever the staging buffer holds at each replay. The capture goes on, and
    new weights given afterwards are what its replays use."""
    import torch
    import paper_2304_14698_amd as xrl
    model, state = synth.make_config(2, n_cand=3)
    rng = np.random.Generator(np.random.PCG64(8))
    w = [synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1) for _ in range(2)]
    side = torch.cuda.Stream()
    enc = xrl.Encoder(model, w[0], stream=side)
    batch = enc.pack(state)
    first = enc.encode(batch)
    out = torch.empty_like(first)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
        enc.encode(batch, out=out)
        with pytest.raises(xrl.XrlError) as e:
            enc.set_weights(w[1])
        assert e.value.code == xrl.ERR["HIP"] and "captured" in str(e.value)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, first)
    enc.set_weights(w[1])
    second = enc.encode(batch)
    torch.cuda.synchronize()
    assert not torch.equal(second, first)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, second)
    batch.free()
    enc.close()
