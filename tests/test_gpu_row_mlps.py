"""The row-MLPs (readout, heads) where their launches and loops change: widths that are no multiples of sixteen, one tile, more
tiles than waves, as wide as they go; states that share a block of the value head, more states than there are slot counters; one
and several chunks of rows in the weight gradients; graphs
up to two or three a compute unit (readout in one launch, vector instructions) and beyond (sum and MLP apart, matrix instructions), wide and no
global attributes.
Against the float64 oracle with the heads' criterion of test_gpu_head_gradients.py and the forward's fp32 tolerance; a graph's
embedding and a state's outputs are the same bits whatever the batch around them."""
import numpy as np
import pytest

import grad_checks as GC
import synth
from oracle import xrl_oracle as O
from test_gpu_forward import check_emb, heads_only_state, oracle_model, weights_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,heads,n_states,n_cand", [
    (64, (16, 16), 2, 20), (128, (17, 3), 3, 42), (64, (129, 64), 2, 70), (256, (512, 512), 2, 30), (128, (1, 1), 1, 16),
    (64, (256, 64), 300, 1), (64, (40, 12), 4100, 0),
    (64, (128, 128), 2, 20), (256, (113, 128), 2, 30), (128, (512, 17), 2, 40), (64, (128, 130), 2, 15),
    (256, (17, 512), 2, 40), (128, (200, 300), 1, 254), (64, (129, 64), 9, 40), (256, (512, 512), 2, 150),
    (64, (256, 64), 1, 127), (128, (256, 64), 1, 128), (128, (100, 36), 3, 170), (64, (65, 66), 9, 255)])   # a chunk of rows, and more
def test_heads_of_any_width(hidden, heads, n_states, n_cand):
    import torch
    import paper_2304_14698_amd as xrl
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="fp32", head_hidden=heads)
    rng = np.random.Generator(np.random.PCG64(n_states + heads[0]))
    if n_cand == 0:                                             # n_states states of one slot
        state = heads_only_state(rng, model, 1, n_states - 1, fixed=True)
        state.update(n_states=n_states, state_graph_ptr=np.arange(n_states + 1, dtype=np.int32), slot_mask=np.ones(n_states, np.uint8))
    else:
        state = heads_only_state(rng, model, n_states, n_cand, fixed=True)
    G, w, om = len(state["slot_mask"]), weights_for(model), oracle_model(model)
    emb = rng.standard_normal((G, hidden)).astype(np.float32)
    dlogp = (rng.standard_normal(G) * state["slot_mask"]).astype(np.float32)
    dvalue, dentropy = (rng.standard_normal(n_states).astype(np.float32) for _ in range(2))
    enc = xrl.Encoder(model, w)
    batch = enc.pack(state)
    t = lambda x: torch.from_numpy(x).cuda()
    got = {k: v.cpu().numpy() for k, v in enc.policy_value(batch, t(emb)).items()}
    ref = O.policy_value(om, w, emb.astype(np.float64), state)
    valid = state["slot_mask"].astype(bool)
    L = max(1.0, float(np.abs(ref["logit"]).max()))
    for k in ("logp", "entropy", "value"):
        a, r = (np.asarray(x[k], np.float64) for x in (got, ref))
        a, r = (a[valid], r[valid]) if k == "logp" else (a, r)
        assert np.abs(a - r).max() <= 2e-5 * max(1.0, np.abs(r).max()), k
    dw = torch.zeros(enc.n_weights, dtype=torch.float32, device="cuda")
    demb = enc.policy_value_backward(batch, t(emb), t(dlogp), t(dvalue), t(dentropy), dw).cpu().numpy()
    bound = O.zero_grads(om)
    ref_demb, ref_dw = O.policy_value_backward(om, w, emb.astype(np.float64), state, dlogp, dvalue, dentropy, bound=bound)
    assert np.linalg.norm(demb - ref_demb) <= 1e-5 * np.linalg.norm(ref_demb)
    assert not demb[~valid].any()
    bound, dw = O.flatten(om, bound), dw.cpu().numpy().astype(np.float64)
    for name, sl, _ in GC.tensors(om):
        if name.startswith(("policy", "value")):
            tol = 1e-5 * np.linalg.norm(ref_dw[sl]) + (2e-6 + 1e-5 * L) * np.linalg.norm(bound[sl])
            assert np.linalg.norm(dw[sl] - ref_dw[sl]) <= tol, name


def some_graphs(state, a, z):
    """The state's graphs a .. z - 1, as one state."""
    n0, n1, e0, e1 = (int(state[k][g]) for k in ("graph_node_ptr", "graph_edge_ptr") for g in (a, z))
    out = {k: state[k][n0:n1] for k in ("node_op", "node_dense")}
    out.update({k: state[k][e0:e1] for k in ("edge_src", "edge_dst", "edge_feat")})
    out.update({k: state[k][a:z + 1] - state[k][a] for k in ("graph_node_ptr", "graph_edge_ptr")})
    if state.get("graph_global") is not None:
        out["graph_global"] = state["graph_global"][a:z]
    return dict(out, n_states=1, state_graph_ptr=np.array([0, z - a], np.int32), slot_mask=state["slot_mask"][a:z])


@pytest.mark.parametrize("readout", ["sum", "mean"])
@pytest.mark.parametrize("hidden,d_global,precision", [(64, 0, "fp32"), (128, 100, "fp32"), (256, 1, "fp32"), (128, 3, "bf16"),
                                                       (64, 1, "bf16"), (64, 256, "fp32"), (128, 256, "bf16"), (256, 256, "fp32")])
def test_readout_at_graph_counts(hidden, d_global, precision, readout):
    import torch
    import paper_2304_14698_amd as xrl
    model, state = synth.make_config(1, n_cand=790)
    model.update(hidden=hidden, precision=precision, rounds=1, d_global=d_global, readout=readout)
    rng = np.random.Generator(np.random.PCG64(hidden))
    state["graph_global"] = rng.standard_normal((791, d_global)).astype(np.float32) if d_global else None
    w, om = weights_for(model), oracle_model(model)
    enc = xrl.Encoder(model, w)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count

    def encoded(a, z):
        batch = enc.pack(some_graphs(state, a, z))
        out = enc.encode(batch).cpu().numpy()
        batch.free()
        return out
    # every graph's row from batches of few graphs, some of them against the oracle
    pieces = [(a, min(a + n_cu, 791)) for a in range(0, 791, n_cu)]
    alone = np.concatenate([encoded(*p) for p in pieces])
    assert np.array_equal(encoded(0, 7), alone[:7])
    for a in (0, 784):
        check_emb(alone[a:a + 7], O.encode(om, w, some_graphs(state, a, a + 7)), model, "emb")
    for n in (n_cu + 1, 2 * n_cu, 2 * n_cu + 1, 3 * n_cu, 3 * n_cu + 1, 3 * n_cu + 16, 791):
        n = min(n, 791)
        assert np.array_equal(encoded(0, n), alone[:n]), n


@pytest.mark.parametrize("hidden,heads", [(256, (256, 64)), (128, (512, 200))])
def test_heads_and_readout_under_capture(hidden, heads):
    """Both heads forward and back and the readout's backward pass in a captured graph (launches with more LDS than one may have by itself):
    every replay, with eager passes between, gives the eager bits."""
    import torch
    import paper_2304_14698_amd as xrl
    model, state = synth.make_config(1, n_cand=40)
    model.update(hidden=hidden, precision="fp32", rounds=1, head_hidden=heads)
    side = torch.cuda.Stream()
    enc = xrl.Encoder(model, weights_for(model), stream=side)
    batch = enc.pack(state)
    g = torch.Generator(device="cpu").manual_seed(3)
    G = len(state["slot_mask"])
    dl, ds = torch.randn(G, generator=g).cuda(), torch.randn(1, generator=g).cuda()

    def step(dw):
        emb = enc.encode(batch, save_for_backward=True)
        pv = enc.policy_value(batch, emb)
        demb = enc.policy_value_backward(batch, emb, dl, ds, ds, dw)
        enc.encode_backward(batch, demb, dw)
        return pv["logp"], pv["value"], demb
    with torch.cuda.stream(side):
        want_dw = torch.zeros(enc.n_weights, device="cuda")
        want = step(want_dw)
        torch.cuda.synchronize()
        dw = torch.zeros_like(want_dw)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
            dw.zero_()
            out = step(dw)
        for _ in range(3):
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(dw, want_dw) and all(torch.equal(a, b) for a, b in zip(out, want))
            eager = torch.zeros_like(want_dw)
            assert all(torch.equal(a, b) for a, b in zip(step(eager), want)) and torch.equal(eager, want_dw)
            torch.cuda.synchronize()
            dw.fill_(7.0)
    batch.free()
    enc.close()


@pytest.mark.parametrize("hidden", [64, 128, 256])
def test_upstream_gradient_of_any_alignment(hidden):
    """A caller's gradient of the embeddings may begin at any fp32 address: the same bits as from an aligned copy, over 17 rows (a tile and
    one row more)."""
    import torch
    import paper_2304_14698_amd as xrl
    model, state = synth.make_config(1, n_cand=16)
    model.update(hidden=hidden, precision="fp32", rounds=1)
    enc = xrl.Encoder(model, weights_for(model))
    batch = enc.pack(state)
    enc.encode(batch, save_for_backward=True)
    room = torch.randn(17 * hidden + 4, generator=torch.Generator().manual_seed(5)).cuda()
    up = room[:17 * hidden].clone()
    got = []
    for offset in range(4):
        at = room[offset:offset + 17 * hidden].view(17, hidden)
        at.copy_(up.view(17, hidden))
        assert at.data_ptr() % 16 == 4 * offset
        dw = torch.zeros(enc.n_weights, device="cuda")
        enc.encode_backward(batch, at, dw)
        got.append(dw)
    assert got[0].any() and all(torch.equal(got[0], g) for g in got[1:])
    batch.free()
    enc.close()


def test_models_of_other_sizes_in_other_threads():
    """Heads that need more and less LDS than a launch may have by itself, of the same kernels, called from two threads on streams of their own:
    every pass gives the bits of a pass alone."""
    import threading

    import torch
    import paper_2304_14698_amd as xrl
    work = []
    for heads in ((512, 512), (300, 100)):
        model, state = synth.make_config(1, n_cand=20)
        model.update(hidden=128, precision="fp32", rounds=1, head_hidden=heads)
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            enc = xrl.Encoder(model, weights_for(model), stream=stream)
            batch = enc.pack(state)
            emb = torch.randn(21, 128, generator=torch.Generator().manual_seed(1)).cuda()
            d = torch.randn(21, generator=torch.Generator().manual_seed(2)).cuda()
            dw = torch.zeros(enc.n_weights, device="cuda")
            torch.cuda.synchronize()

        def step(enc=enc, batch=batch, emb=emb, d=d, dw=dw):
            pv = enc.policy_value(batch, emb)
            return [pv["logp"], pv["value"], enc.policy_value_backward(batch, emb, d, d[:1], d[:1], dw)]
        with torch.cuda.stream(stream):
            want = [x.clone() for x in step()]
            torch.cuda.synchronize()
        work.append((enc, batch, stream, step, want))
    failed = []

    def run(stream, step, want):
        try:
            with torch.cuda.stream(stream):
                for _ in range(30):
                    got = step()
                    stream.synchronize()
                    assert all(torch.equal(a, b) for a, b in zip(got, want))
        except BaseException as e:
            failed.append(e)
    threads = [threading.Thread(target=run, args=w[2:]) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for w in work:
        w[1].free()
        w[0].close()
    assert not failed, failed


@pytest.mark.parametrize("hidden", [64, 256])
def test_slots_share_of_the_mean_gradient(hidden):
    """The embeddings' gradient where its last step -- the mean embedding's share, 64 slots a block -- has full blocks, a remainder, states that
    cross blocks, masked slots, and an output that begins at any fp32 address."""
    import torch
    import paper_2304_14698_amd as xrl
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="fp32")
    rng = np.random.Generator(np.random.PCG64(hidden))
    state = heads_only_state(rng, model, 13, 24)
    G, S, w, om = len(state["slot_mask"]), 13, weights_for(model), oracle_model(model)
    assert G > 64 and G % 64
    emb = rng.standard_normal((G, hidden)).astype(np.float32)
    dlogp = (rng.standard_normal(G) * state["slot_mask"]).astype(np.float32)
    dvalue, dentropy = (rng.standard_normal(S).astype(np.float32) for _ in range(2))
    ref, _ = O.policy_value_backward(om, w, emb.astype(np.float64), state, dlogp, dvalue, dentropy)
    enc = xrl.Encoder(model, w)
    batch = enc.pack(state)
    t = lambda x: torch.from_numpy(x).cuda()
    args, dw, got = [t(x) for x in (emb, dlogp, dvalue, dentropy)], torch.zeros(enc.n_weights, device="cuda"), []
    for offset in (0, 1, 2):
        room = torch.full((G * hidden + 4,), 7.0, device="cuda")
        at = room[offset:offset + G * hidden]
        enc._empty = lambda shape, dtype=None: at.view(shape)
        assert enc.policy_value_backward(batch, *args, dw).data_ptr() == at.data_ptr()
        got.append(at.view(G, hidden).cpu().numpy())
        assert (room[:offset] == 7.0).all() and (room[offset + G * hidden:] == 7.0).all()
    assert np.linalg.norm(got[0] - ref) <= 1e-5 * np.linalg.norm(ref)
    assert not got[0][state["slot_mask"] == 0].any()
    assert all(np.array_equal(got[0], g) for g in got[1:])
    batch.free()
    enc.close()
