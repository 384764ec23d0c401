"""Precision of the backward pass of batches reduced to distinct nodes (bf16): what a class receives is one
fp32 sum rounded once, as a node's gradient is in a batch that is not reduced, and the weight
gradients are no farther from float64 than those of the whole batch.

The float64 reference differentiates the stored forward (the node states and received sums the device
kept, whose values are the same bits in both forms; the hidden rows rounded to bf16 as the device
rounds them), so that the forward's own rounding, which is a hundred times larger than what is
compared here, is not part of the difference. The weights are mask-stable (grad_checks), so no
ReLU mask depends on rounding either."""
import numpy as np
import pytest
import torch

import paper_2304_14698_amd as xrl
import synth
import grad_checks as GC
from test_gpu_forward import oracle_model

pytestmark = pytest.mark.gpu


def _gradients(model, w, state, up, min_us, monkeypatch, stored=False):
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", min_us)
    enc = xrl.Encoder(model, w)
    batch = enc.pack(state)
    emb = enc.encode(batch, save_for_backward=True)
    reduced = enc.batch_level(batch, 0)[0] < batch.N
    dw = torch.zeros(enc.n_weights, dtype=torch.float32, device="cuda")
    enc.encode_backward(batch, torch.tensor(up, dtype=torch.float32, device="cuda"), dw)
    out = dw.cpu().numpy().astype(np.float64)
    acts = None
    if stored:
        R = model["rounds"]
        acts = dict(h=[enc.get_activation(batch, "h", r).cpu().double() for r in range(R + 1)],
                    agg=[None] + [enc.get_activation(batch, "agg", r).cpu().double() for r in range(1, R + 1)],
                    pool=enc.get_activation(batch, "pool").cpu().double(), emb=emb.cpu().double(), view=batch.host_view())
    batch.free()
    enc.close()
    return out, reduced, acts


@pytest.mark.parametrize("d_edge", [8, 20])         # from the kept forward; recomputing (attributes wider than a slab)
def test_a_class_receives_one_sum(d_edge, monkeypatch):
    """Chains u -> n -> v, four times the same, in which n's state receives 256 (its own node MLP), 1 (as a receiver) and
    -256 (as a sender): 257 does not fit the 8 significant bits of bf16, and the sum is 1."""
    model, _ = synth.make_config(1)
    H = 64
    model.update(hidden=H, precision="bf16", rounds=1, d_edge=d_edge, n_node_dense=0)
    t = {name: np.zeros(shape, np.float32) for name, shape in xrl.weight_layout(model)}
    eye = np.eye(H, dtype=np.float32)
    for name in ("embed", "edge0", "node0", "readout"):
        t[f"{name}.W1"][:] = eye
    t["embed.b0"][:] = 1
    t["node0.W0"][:H], t["node0.W0"][H:] = 256 * eye, eye
    t["edge0.W0"][:H], t["edge0.W0"][H:2 * H], t["edge0.b0"][:] = -256 * eye, eye, 1024
    t["readout.W0"][:H] = eye
    w = np.concatenate([x.ravel() for x in t.values()])
    G = 4
    state = dict(n_states=1, state_graph_ptr=np.array([0, G], np.int32), graph_node_ptr=np.arange(0, 3 * G + 1, 3, dtype=np.int32),
                 graph_edge_ptr=np.arange(0, 2 * G + 1, 2, dtype=np.int32), node_op=np.tile([0, 1, 2], G).astype(np.int32),
                 node_dense=np.zeros((3 * G, 0), np.float32), edge_src=np.tile([0, 1], G).astype(np.int32),
                 edge_dst=np.tile([1, 2], G).astype(np.int32), edge_feat=np.zeros((2 * G, d_edge), np.float32),
                 graph_global=np.zeros((G, model["d_global"]), np.float32), slot_mask=np.ones(G, np.uint8))
    got = {us: _gradients(model, w, state, np.ones((G, H)), us, monkeypatch)[:2] for us in ("-1", "0")}
    assert not got["-1"][1] and got["0"][1]
    at = sum(t[name].size for name in ("embed.W0", "embed.b0", "embed.W1"))
    for dw, _ in got.values():
        # u: 256 - 256; n: 256 + 1 - 256; v: 256 + 1, rounded to 256 as it is stored
        assert np.all(dw[at:at + H] == G * (0 + 1 + 256))
    assert np.array_equal(got["-1"][0], got["0"][0])


def _float64(model, w, acts, up):
    """dweights of the encoder in float64 from the stored forward (two-layer MLP rounds, sum readout)."""
    H, R, De, Tn = model["hidden"], model["rounds"], model["d_edge"], model["n_op_types"]
    low = lambda x: x.float().bfloat16().double()
    W, o = {}, 0
    for name, shape in xrl.weight_layout(model):
        n = int(np.prod(shape))
        W[name] = torch.from_numpy(w[o:o + n].reshape(shape)).double()
        o += n
    g = {k: torch.zeros_like(v) for k, v in W.items()}
    v = acts["view"]
    src, dst = (torch.from_numpy(v[k]).long() for k in ("in_src", "in_dst"))
    ef = torch.from_numpy(v["edge_feat"]).double()

    def back(name, x, z1, on, dy, rounded=True):
        W0, W1 = ((low(W[f"{name}.W{i}"]) for i in (0, 1)) if rounded else (W[f"{name}.W{i}"] for i in (0, 1)))
        dz2 = dy * on
        dz1 = (dz2 @ W1.T) * (z1 > 0)
        g[f"{name}.W1"] += z1.T @ dz2
        g[f"{name}.b1"] += dz2.sum(0)
        g[f"{name}.W0"] += x.T @ dz1
        g[f"{name}.b0"] += dz1.sum(0)
        return dz1 @ W0.T
    hidden = lambda name, x: torch.relu(x @ low(W[f"{name}.W0"]) + W[f"{name}.b0"])
    x = torch.cat([acts["pool"], torch.zeros(len(up), model["d_global"], dtype=torch.float64)], 1)
    z1 = torch.relu(x @ W["readout.W0"] + W["readout.b0"])
    dpool = back("readout", x, z1, acts["emb"] > 0, torch.from_numpy(up).double(), rounded=False)[:, :H]
    dh = dpool[torch.from_numpy(v["node_graph"]).long()]
    for r in range(R, 0, -1):
        h = acts["h"][r - 1]
        x = torch.cat([h, acts["agg"][r]], 1)
        dx = back(f"node{r - 1}", x, low(hidden(f"node{r - 1}", x)), acts["h"][r] > 0, dh)
        dh, dagg = dx[:, :H].clone(), dx[:, H:]
        x = torch.cat([h[src], h[dst], low(ef)], 1)
        z1 = low(hidden(f"edge{r - 1}", x))
        z2 = z1 @ low(W[f"edge{r - 1}.W1"]) + W[f"edge{r - 1}.b1"]
        dx = back(f"edge{r - 1}", x, z1, z2 > 0, dagg[dst])
        dh.index_add_(0, src, dx[:, :H])
        dh.index_add_(0, dst, dx[:, H:2 * H])
    sums = torch.zeros(len(dh), De, dtype=torch.float64).index_add_(0, dst, ef)
    x = torch.cat([sums, torch.nn.functional.one_hot(acts["op"], Tn).double(), acts["dense"]], 1)
    z1 = low(torch.relu(x @ W["embed.W0"] + W["embed.b0"]))
    back("embed", low(x), z1, acts["h"][0] > 0, dh)
    return torch.cat([y.ravel() for y in g.values()]).numpy()


def upstreams(rng, model, w, state):
    """Embedding gradients of given shapes, and the heads' own: of a value loss alone, of a policy loss alone, of both."""
    G, H, S = len(state["slot_mask"]), model["hidden"], state["n_states"]
    yield "of both signs", rng.standard_normal((G, H))
    yield "of one sign", np.abs(rng.standard_normal((G, H)))
    yield "nearly equal", 1 + 0.1 * rng.standard_normal((G, H))
    x = 1 + 0.1 * rng.standard_normal((G, H))
    yield "cancelling", x - x.mean(0)
    enc = xrl.Encoder(model, w)
    batch = enc.pack(state)
    emb = enc.encode(batch)
    t = lambda x: torch.tensor(np.asarray(x, np.float32), device="cuda")
    pv = enc.policy_value(batch, emb)
    ptr = state["state_graph_ptr"]
    taken = np.array([rng.integers(0, b - a) for a, b in zip(ptr[:-1], ptr[1:])])
    old = pv["logp"][torch.from_numpy(ptr[:-1] + taken).long().cuda()].clone()
    _, dlogp, dvalue, dent = enc.ppo_objective(batch, pv, t(taken).int(), old, t(rng.standard_normal(S)), t(rng.standard_normal(S)))
    for name, a, b in (("heads", 1, 1), ("value head", 0, 1), ("policy head", 1, 0)):
        dw = torch.zeros(enc.n_weights, device="cuda")
        yield name, enc.policy_value_backward(batch, emb, dlogp * a, dvalue * b, dent * a, dw).cpu().numpy()
    batch.free()
    enc.close()


@pytest.mark.parametrize("base,hidden,n_cand", [("resnet", 64, 60), ("resnet", 128, 150), ("transformer", 256, 50)])
def test_no_farther_from_float64_than_the_whole_batch(base, hidden, n_cand, monkeypatch):
    rng = np.random.Generator(np.random.PCG64(17))
    model, _ = synth.make_config(1)
    model.update(hidden=hidden, precision="bf16", rounds=3, readout="sum")
    dag = synth.resnet_dag(rng, 4) if base == "resnet" else synth.transformer_dag(rng, 2)
    state = synth.concat_states([synth.make_state(rng, dag, n_cand, by_block=True)])
    om = oracle_model(model)
    indeg = np.bincount(dag.dst).max()
    w = GC.stable_weights(om, "fixed", 3, max_indeg=int(indeg) + 4, max_nodes=int(np.diff(state["graph_node_ptr"]).max()))
    monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
    monkeypatch.setenv("XRL_PERSISTENT_MIN_ROWS", "0")    # both from the kept forward
    for name, up in upstreams(rng, model, w, state):
        up = up.astype(np.float32)
        whole, reduced0, acts = _gradients(model, w, state, up, "-1", monkeypatch, stored=True)
        part, reduced1, _ = _gradients(model, w, state, up, "0", monkeypatch)
        assert not reduced0 and reduced1
        acts.update(op=torch.from_numpy(state["node_op"]).long(), dense=torch.from_numpy(state["node_dense"]).double())
        ref = _float64(model, w, acts, up)
        o, err = 0, {}
        for tensor, shape in xrl.weight_layout(model):
            sl = slice(o, o + int(np.prod(shape)))
            o = sl.stop
            if not tensor.startswith(("policy", "value", "readout")):    # (heads and readout: the same kernels on both sides)
                err[tensor] = [np.linalg.norm(x[sl] - ref[sl]) / np.linalg.norm(ref[sl]) for x in (whole, part)]
        rms = np.sqrt(np.mean(np.square(list(err.values())), axis=0))
        ratio = {k: e[1] / e[0] for k, e in err.items()}
        k = max(ratio, key=ratio.get)
        print(f"{base} {hidden}, gradient {name}: relative error per tensor (rms), whole {rms[0]:.2e}, reduced {rms[1]:.2e}; "
              f"largest ratio {ratio[k]:.2f} ({k} {err[k][0]:.1e} / {err[k][1]:.1e})")
        # A class's gradient is rounded once where each of its nodes' was: with the heads' own gradients
        # (signs mixed over a state's candidates) half the error and less, in every tensor. Nodes with nearly
        # equal gradients have roundings that average out over a class: there the last round's
        # node MLP, which has the smallest error of all tensors, may have up to 2.5 times as much.
        assert rms[1] <= rms[0], name
        if name in ("heads", "value head", "of both signs", "cancelling"):
            assert ratio[k] <= 1, (name, k)
        else:
            assert ratio[k] <= 3, (name, k)
