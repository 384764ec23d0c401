"""Workloads of the state encoder: what a program that uses the library has it do.

An agent meets two kinds of work. Acting: at every rewriting step the environment hands over a new
state (the current graph and its candidates) in host memory; it is packed, uploaded, encoded and
scored by the heads, once. Updating: a minibatch of states goes through set_weights (the optimiser
has just stepped), the forward pass, the clipped objective and both backward passes; the minibatch
is either packed anew (minibatches drawn afresh in every epoch) or kept packed on the device over
the epochs. In between, a kept batch is re-evaluated under new weights (log-probabilities and
values recomputed before the epochs begin).

Graphs, candidates and states come from `synth`: DAGs shaped like the networks the agent rewrites,
candidates that are local rewrites of the current graph, and, along an episode of eight steps, each
state's current graph one of the candidates of the state before.
"""
import math

import numpy as np
import torch

import paper_2304_14698_amd as xrl
import synth

EPISODE = 8          # states of one episode before the next starts from the base graph again

# node count of one unit of each kind of base graph (blocks, modules), for sizing drawn cases
NODES_PER_BLOCK = {"transformer": 47, "resnet": 20, "inception": 113, "layered": 50}


def _case(name, step, base, blocks, n_states, cand, hidden, rounds, precision, round_kind="mlp", mlp_layers=2,
          features="default", readout="sum"):
    return dict(name=name, step=step, base=base, blocks=blocks, n_states=n_states, cand_min=cand[0], cand_max=cand[1],
                hidden=hidden, rounds=rounds, precision=precision, round_kind=round_kind, mlp_layers=mlp_layers,
                features=features, readout=readout)


def listed():
    return [
        # one step on a toy graph: nine graphs of about fifty nodes, all latency
        _case("act_tiny_fp32", "act", "layered", 1, 1, (8, 8), 64, 2, "fp32"),
        # one step on a residual network with few applicable rules: fifteen graphs of 338 nodes
        _case("act_resnet_bf16", "act", "resnet", 16, 1, (14, 14), 128, 5, "bf16"),
        # one step on a transformer encoder: 129 graphs of about 565 nodes, given whole ...
        _case("act_transformer_bf16", "act", "transformer", 12, 1, (128, 128), 128, 5, "bf16"),
        # ... and given as edits of the current graph, the form a rewrite engine has them in
        _case("act_edits_bf16", "act_edits", "transformer", 12, 1, (128, 128), 128, 5, "bf16"),
        # one step on a wide network with many candidates at the largest hidden width
        _case("act_inception_bf16_h256", "act", "inception", 11, 1, (256, 256), 256, 5, "bf16"),
        # one step with the layers exactly as the paper prints them: attention rounds, one learned
        # matrix per layer, 40 operator types, shapes over 4096 as edge attributes
        _case("act_attention_bf16", "act", "inception", 6, 1, (64, 64), 128, 5, "bf16", "gat", 1, "paper"),
        # a rollout step of 32 environments run side by side, one pack
        _case("rollout_resnet_bf16", "act", "resnet", 16, 32, (64, 64), 128, 5, "bf16"),
        # a kept state re-evaluated under new weights, in single precision
        _case("evaluate_transformer_fp32", "evaluate", "transformer", 12, 1, (128, 128), 128, 5, "fp32"),
        # update steps: a small one in single precision, minibatch packed anew
        _case("update_resnet_fp32", "update_fresh", "resnet", 8, 4, (10, 40), 64, 3, "fp32"),
        # ... a residual network's minibatch, kept over the epochs
        _case("update_resnet_bf16", "update", "resnet", 16, 16, (32, 96), 128, 5, "bf16"),
        # ... attention rounds, minibatch packed anew
        _case("update_attention_bf16", "update_fresh", "transformer", 12, 4, (32, 96), 128, 5, "bf16", "gat"),
        # ... and the largest: transformer-shaped states of up to 512 candidates, hidden width 256
        _case("update_transformer_bf16_h256", "update", "transformer", 20, 16, (64, 512), 256, 5, "bf16"),
    ]


def draw(rng):
    step = rng.choice(["act", "act", "act_edits", "evaluate", "update", "update_fresh"])
    base = rng.choice(["layered", "resnet", "transformer", "inception"])
    hidden = rng.choice([64, 128, 256])
    precision = rng.choice(["bf16", "bf16", "fp32"])
    gat = rng.random() < 0.2
    blocks = {"layered": 1, "resnet": rng.randint(4, 16), "transformer": rng.randint(3, 20),
              "inception": rng.randint(2, 11)}[base]
    cand = int(round(math.exp(rng.uniform(math.log(4), math.log(512)))))
    # nodes of the whole batch, up to what one step of that kind meets
    most = {"act": 700e3, "act_edits": 700e3, "evaluate": 700e3, "update": 2e6, "update_fresh": 1e6}[step]
    if precision == "fp32":
        most /= 8
    nodes = math.exp(rng.uniform(math.log(1e3), math.log(most)))
    per_graph = NODES_PER_BLOCK[base] * blocks
    cand = max(1, min(cand, int(most / per_graph) - 1))
    n_states = max(1, min(64, int(nodes / (per_graph * (cand + 1)))))
    return dict(step=step, base=base, blocks=blocks, n_states=n_states, cand_min=max(1, cand // 2), cand_max=cand,
                hidden=hidden, rounds=rng.randint(2, 5), precision=precision, round_kind="gat" if gat else "mlp",
                mlp_layers=1 if gat and rng.random() < 0.5 else 2, features=rng.choice(["default", "default", "paper"]),
                readout=rng.choice(["sum", "sum", "mean"]))


def _model(case):
    paper = case["features"] == "paper"
    return dict(n_op_types=40 if paper else synth.graphs.N_OP_TYPES, n_node_dense=0 if paper else synth.graphs.N_NODE_DENSE,
                d_edge=4 if paper else synth.graphs.D_EDGE, d_global=1, hidden=case["hidden"], rounds=case["rounds"],
                mlp_layers=case["mlp_layers"], head_hidden=(256, 64), readout=case["readout"],
                precision=case["precision"], round_kind=case["round_kind"])


def _base(rng, case):
    make = {"layered": lambda: synth.layered_dag(rng, 50), "resnet": lambda: synth.resnet_dag(rng, case["blocks"]),
            "transformer": lambda: synth.transformer_dag(rng, case["blocks"]),
            "inception": lambda: synth.inception_dag(rng, case["blocks"])}
    return make[case["base"]]()


def _paper_edges(feat):
    """Tensor shapes over 4096 in place of the first four generic attributes (powers of two)."""
    return (np.exp2(np.clip(np.round(6.0 + 3.0 * feat[:, :4]), 0, 12)) / 4096.0).astype(np.float32)


def _host_state(rng, case):
    """The arrays the packer takes, as the environment hands them over."""
    base, by_block = _base(rng, case), case["base"] != "layered"
    # candidates per state: spread over the range, in an order of the seed's (so their sum is the case's)
    counts = np.round(np.linspace(case["cand_max"], case["cand_min"], case["n_states"])).astype(int)
    counts = rng.permutation(counts)
    if case["step"] == "act_edits":
        bases = [synth.shuffle_edges(rng, base)]
        for i in range(1, case["n_states"]):
            bases.append(synth.local_rewrite(rng, bases[-1] if i % EPISODE else base, 2, 2, by_block=by_block))
        state = synth.make_edit_states(rng, bases, [int(c) for c in counts], by_block=by_block)[0]
    else:
        states, first = [], base
        for i, c in enumerate(counts):
            base = base if i % EPISODE else first
            graphs, mask = synth.make_state(rng, base, int(c), del_ins=None if by_block else (1, 4), by_block=by_block)
            states.append((graphs, mask))
            base = graphs[int(rng.integers(1, len(graphs)))]       # the episode goes on from one of the candidates
        state = synth.concat_states(states)
    if case["features"] == "paper":
        for key in ("edge_feat", "add_edge_feat"):
            if key in state:
                state[key] = _paper_edges(state[key])
        for key in ("node_dense", "add_node_dense"):
            if key in state:
                state[key] = np.zeros((len(state[key]), 0), np.float32)
    return state


def _slots(case, state):
    """[S + 1] slot range of each state."""
    if case["step"] == "act_edits":
        return np.asarray(state["state_cand_ptr"]) + np.arange(case["n_states"] + 1)
    return np.asarray(state["state_graph_ptr"])


def prepare(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    model, state = _model(case), _host_state(rng, case)
    weights = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    enc = xrl.Encoder(model, weights)
    s = dict(step=case["step"], enc=enc, state=state, weights=weights, fp32=case["precision"] == "fp32", batch=None)
    if case["step"] in ("evaluate", "update"):
        s["batch"] = enc.pack(state)
    if case["step"].startswith("update"):
        # the rollout's records: a valid slot taken in each state, its log-probability when sampled
        # (an untrained policy: near uniform), advantage and value target
        ptr, mask = _slots(case, state), state["slot_mask"]
        taken, old = [], []
        for a, b in zip(ptr[:-1], ptr[1:]):
            valid = np.flatnonzero(mask[a:b])
            taken.append(int(rng.choice(valid)))
            old.append(-math.log(len(valid)) + 0.1 * rng.standard_normal())
        n = len(taken)
        cuda = lambda x, t: torch.tensor(np.asarray(x), dtype=t, device="cuda")
        s["records"] = (cuda(taken, torch.int32), cuda(old, torch.float32), cuda(rng.standard_normal(n), torch.float32),
                        cuda(rng.standard_normal(n), torch.float32))
        s["dweights"] = torch.zeros(enc.n_weights, dtype=torch.float32, device="cuda")
    return s


def _scores(s, emb, pv):
    """What the heads give. (The greedy slot is a function of the logits; in bf16 a state of hundreds of
    near-identical candidates has near ties, so it is compared in single precision only.)"""
    out = dict(emb=emb, logit=pv["logit"], logp=pv["logp"], value=pv["value"], entropy=pv["entropy"])
    if s["fp32"]:
        out["action"] = pv["action"]
    return out


def run(s):
    enc, step = s["enc"], s["step"]
    if step in ("act", "act_edits"):
        batch = enc.pack_edits(s["state"]) if step == "act_edits" else enc.pack(s["state"])
        emb = enc.encode(batch)
        return _scores(s, emb, enc.policy_value(batch, emb))
    enc.set_weights(s["weights"])
    if step == "evaluate":
        emb = enc.encode(s["batch"])
        return _scores(s, emb, enc.policy_value(s["batch"], emb))
    batch = s["batch"] if s["batch"] is not None else enc.pack(s["state"])
    dw = s["dweights"].zero_()
    emb = enc.encode(batch, save_for_backward=True)
    pv = enc.policy_value(batch, emb)
    J, dlogp, dvalue, dentropy = enc.ppo_objective(batch, pv, *s["records"])
    demb = enc.policy_value_backward(batch, emb, dlogp, dvalue, dentropy, dw)
    enc.encode_backward(batch, demb, dw)
    return dict(_scores(s, emb, pv), J=J, dweights=dw)


def _distinct(state, rounds):
    """(nodes, edges) of the state's graphs that differ from every other within `rounds` hops
    upstream, counted by colour refinement: what any implementation has to compute at least."""
    gnp, gep = state["graph_node_ptr"], state["graph_edge_ptr"]
    off = np.repeat(gnp[:-1], np.diff(gep)).astype(np.int64)
    src, dst = state["edge_src"] + off, state["edge_dst"] + off
    N, u = len(state["node_op"]), np.uint64

    def mix(x):
        x = (x ^ (x >> u(31))) * u(0x9E3779B97F4A7C15)
        x = (x ^ (x >> u(29))) * u(0xBF58476D1CE4E5B9)
        return x ^ (x >> u(32))

    def rows(a):
        h = np.zeros(len(a), np.uint64)
        for i in range(a.shape[1]):
            h = mix(h + np.ascontiguousarray(a[:, i]).view(np.uint32).astype(np.uint64) + u(i + 1))
        return h

    def received(v):
        out = np.zeros(N, np.uint64)
        np.add.at(out, dst, v)
        return out

    efeat = rows(state["edge_feat"])
    colour = mix(rows(state["node_dense"]) + state["node_op"].astype(np.uint64) + received(mix(efeat)))
    for _ in range(rounds):
        colour = mix(colour * u(3) + received(mix(colour[src] * u(5) + efeat)))
    first = np.unique(colour, return_index=True)[1]
    return len(first), int(np.bincount(dst, minlength=N)[first].sum())


def work(case):
    """Bytes: the batch as it is given (host arrays where the pass packs them, else the packed ones),
    the weights, and the outputs. Flops: the products of the layers over the nodes and edges that
    are distinct (a candidate shares all but a neighbourhood of its rewrite with its state's
    current graph), three times as many when the pass also differentiates."""
    rng = np.random.Generator(np.random.PCG64(0))
    model, H, R = _model(case), case["hidden"], case["rounds"]
    n_cand = (case["cand_min"] + case["cand_max"]) / 2
    sample = dict(case, step="act", n_states=1, cand_min=int(min(n_cand, 64)), cand_max=int(min(n_cand, 64)))
    state = _host_state(rng, sample)
    graphs = len(state["slot_mask"])
    base_n, base_e = int(state["graph_node_ptr"][1]), int(state["graph_edge_ptr"][1])
    nodes, edges = _distinct(state, R)
    scale = n_cand / max(1, graphs - 1)                 # distinct items beyond the current graph's, per candidate
    S, G = case["n_states"], case["n_states"] * (n_cand + 1)
    Nd, Ed = S * (base_n + scale * (nodes - base_n)), S * (base_e + scale * (edges - base_e))
    Nd, Ed = max(Nd, 1.0), max(Ed, 1.0)
    N, E = len(state["node_op"]) / graphs * G, len(state["edge_src"]) / graphs * G
    De, Dd = model["d_edge"], model["n_node_dense"]
    dense = 1 if case["mlp_layers"] == 1 else 2         # learned matrices per layer
    flops = 2.0 * Nd * H * (De + Dd) + (2.0 * Nd * H * H if dense == 2 else 0.0)
    if case["round_kind"] == "gat":
        flops += R * 2.0 * Nd * H * H
    else:
        flops += R * 2.0 * H * (Nd * 2 * H + Ed * (2 * H + De) + (dense - 1) * H * (Nd + Ed))
    flops += 2.0 * G * (H * H * dense + H * 256 + 256 * 64)
    weights = 4.0 * xrl.weight_count(model)
    if case["step"] == "act_edits":                     # the current graphs in full, a few items per candidate
        given = S * (base_n * (4 + 4 * Dd) + base_e * (8 + 4 * De)) + G * 3 * (8 + 4 * Dd + 2 * (8 + 4 * De))
    else:
        given = N * (4 + 4 * Dd) + E * (8 + 4 * De)
    out = 4.0 * G * (H + 2) + 12.0 * S
    if case["step"].startswith("update"):
        return dict(bytes=given + 2 * weights + out, flops=3.0 * flops)
    return dict(bytes=given + weights + out, flops=flops)


def tolerance(case):
    """Measured on the listed and some forty drawn cases. Forward: the same states with every graph's
    edges in another order, i.e. other sums of the received messages: in fp32 up to 5e-6 (logp, a
    difference of logits; 1.3e-5 for one value), in bf16, where a sum on the edge of a rounding flips
    a stored activation, up to 2.6e-4 (3e-2 for one value); four times that, and twice more in bf16,
    where implementations differ by more than the order of those sums. Gradients: the upstream
    gradient divided by 3 and by 1.7 and the result multiplied back, which moves every bf16 rounding
    of the backward pass: 1e-4 to 6e-3 (1.3e-2 once; 0.9 for one value), the more the gradients of
    near-identical candidates cancel; in fp32 2e-6 (1.7e-4 for one value)."""
    if case["precision"] == "fp32":
        return {"rel": 2e-5, "max": 7e-4, "differ": 0.01}
    if case["step"].startswith("update"):
        return {"rel": 2e-2, "max": 0.9, "differ": 0.01}
    return {"rel": 2e-3, "max": 0.2, "differ": 0.01}
