"""Weight-gradient products of several layers in one launch: widths of the edge attributes at the edge of
the tile's extra columns, both operand types at every hidden width, more products than one launch takes,
and so little room for gradients that every MLP is launched by itself. Criteria: those of
test_gpu_weight_gradient.py (the product against float64 on the same operands) and test_gpu_backward.py (the
backward pass against the oracle, fp32)."""
import numpy as np
import pytest

import paper_2304_14698_amd as xrl_package
import synth
from test_gpu_backward import run_backward_case
from test_gpu_forward import weights_for
from test_gpu_weight_gradient import run, xrl  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,precision,d_edge,wide", [
    (64, "fp32", 8, False), (256, "fp32", 4, False),
    (128, "bf16", 28, False),                      # 28 attributes and the bias fill 29 of the 32 extra columns
    (64, "bf16", 32, False), (128, "fp32", 32, False), (256, "bf16", 28, True), (256, "bf16", 60, True),
    (128, "bf16", 132, False)])                    # ... from 32 on a product of their own; 132 + 1 need two tiles
def test_weight_gradient_edge_attribute_widths(xrl, hidden, precision, d_edge, wide, monkeypatch):  # noqa: F811
    if wide:
        monkeypatch.setenv("XRL_WGRAD_WIDE_MIN_ROWS", "0")
    model, state = synth.make_config(4, n_cand=2)
    model.update(hidden=hidden, precision=precision, d_edge=d_edge)
    rng = np.random.Generator(np.random.PCG64(9))
    state = dict(state, edge_feat=rng.standard_normal((len(state["edge_src"]), d_edge)).astype(np.float32))
    run(xrl, model, state, n_plain=65)


@pytest.mark.parametrize("room", ["0", None])
def test_backward_of_more_products_than_one_launch_takes(xrl, room, monkeypatch):  # noqa: F811
    if room is not None:
        monkeypatch.setenv("XRL_GRAD_ROOM", room)
    model, state = synth.make_config(1)
    model.update(rounds=7)                         # 30 products; a launch takes 24
    run_backward_case(xrl, model, state, weights_for(model))


@pytest.mark.parametrize("hidden,precision,rows", [(64, "fp32", 1 << 20), (128, "fp32", (1 << 20) + 37), (256, "fp32", 1 << 20),
                                                   (64, "bf16", 1 << 22), (128, "bf16", (1 << 22) - 5), (256, "bf16", 1 << 21)])
def test_weight_gradient_error_of_long_sums(xrl, hidden, precision, rows):  # noqa: F811
    """Slices of thousands of rows. Terms of random sign: a sum of k of them grows with the root of k, and L additions
    one after the other, each rounded to 2^-24 / sqrt(3) of the sum so far (root mean square, at most), leave
    2^-24 sqrt(L / 6) of the whole. Added one after the other: the steps (2 rows in fp32, 16 in bf16) between two
    foldings into the second sums, the foldings of a slice, an eighth of the slices, eight; a third of room on top."""
    import torch
    model, state = synth.make_config(1)
    model.update(hidden=hidden, precision=precision)
    enc = xrl.Encoder(model, weights_for(model))
    batch = enc.pack(state)
    gen = torch.Generator(device="cuda").manual_seed(5)
    dt = torch.float32 if precision == "fp32" else torch.bfloat16
    x = torch.relu(torch.randn(rows, hidden, generator=gen, device="cuda")).to(dt)
    dz = torch.randn(rows, hidden, generator=gen, device="cuda").to(dt)
    dW, db = torch.zeros(hidden, hidden, device="cuda"), torch.zeros(hidden, device="cuda")
    enc.weight_gradient(batch, "plain", x=x, dz=dz, dW=dW, db=db)
    torch.cuda.synchronize()
    ref, step = torch.zeros(hidden, hidden, dtype=torch.float64, device="cuda"), 1 << 17
    for i in range(0, rows, step):
        ref += x[i:i + step].double().t().contiguous() @ dz[i:i + step].double()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    wide = precision == "bf16" and hidden == 256
    slices = cus if wide else 2 * cus * 128 // max(hidden, 128)
    per_slice = rows / slices
    fold = {64: (128, 1024), 128: (128, 1024), 256: (192, per_slice)}[hidden][precision == "bf16"]
    L = fold / (2 if precision == "fp32" else 16) + per_slice / fold + slices / 8 + 8
    for got, want in ((dW, ref), (db, dz.double().sum(0))):
        err = float((got.double() - want).norm() / want.norm())
        print(f"{err:.2e} of {4 / 3 * 2 ** -24 * (L / 6) ** 0.5:.2e}")
        assert err <= 4 / 3 * 2 ** -24 * (L / 6) ** 0.5
    batch.free()
    enc.close()


def test_backward_of_a_larger_batch_leaves_a_graphs_workspace():
    """A captured backward pass keeps its addresses: a larger batch whose gradients' room would not fit beside what it
    cannot do without takes the room that is there. Its gradients are those of a context without graphs but for the
    order of the weight gradients' sums, whose slices follow the room."""
    import torch
    rng = np.random.Generator(np.random.PCG64(8))
    model, _ = synth.make_config(1)
    model.update(hidden=64, precision="fp32", rounds=5)
    w = weights_for(model)
    base = synth.resnet_dag(rng, 8)
    states = [synth.concat_states([synth.make_state(rng, base, n, by_block=True)]) for n in (60, 72)]
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        alone = xrl_package.Encoder(model, w, stream=side)
        enc = xrl_package.Encoder(model, w, stream=side)

        def step(e, b):
            emb = e.encode(b, save_for_backward=True)
            dw = torch.zeros(e.n_weights, device="cuda")
            e.encode_backward(b, torch.ones_like(emb), dw)
            return dw
        large = [e.pack(states[1]) for e in (alone, enc)]
        enc.encode(large[1], save_for_backward=True)          # (the forward's workspace has its size)
        small = enc.pack(states[0])
        want = step(enc, small)
        dw, up = torch.zeros_like(want), torch.ones(small.G, 64, device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
            dw.zero_()
            enc.encode_backward(small, up, dw)
        reference = step(alone, large[0])
        for _ in range(3):
            got = step(enc, large[1])
            torch.cuda.synchronize()
            assert float((got - reference).norm()) <= 1e-6 * float(reference.norm())
            step(enc, small)                                  # (what the graph's backward pass is of)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(dw, want)
        for x in large + [small, alone, enc]:
            x.free() if hasattr(x, "free") else x.close()


@pytest.mark.parametrize("form", ["kept", "reduced", "attention", "attention fp32"])
def test_little_room_launches_mlp_by_mlp(form, monkeypatch):
    """Room for the largest MLP's gradients alone: the others wait for the launch of those before, in the same place. Against all of
    them in one launch: what is multiplied is the same, in bits, so a tensor may differ by the order of its sums alone,
    2^-24 times the root of its additions (a few hundred: 1e-6) of the sum of its terms' sizes, here a few times the
    tensor. By form: dz2 written into the room by the gather of a whole batch, by the class sums of a reduced one; dz1
    read by dh = dz W^T after its product has been queued, and reductions alone in the queue, 26 jobs of them."""
    monkeypatch.setenv("XRL_PERSISTENT_MIN_ROWS", "0")
    monkeypatch.setenv("XRL_RESIDENT_MAX_GRAPHS", "0")
    monkeypatch.setenv("XRL_DISTINCT_MIN_US", "0" if form == "reduced" else "-1")
    import torch
    rng = np.random.Generator(np.random.PCG64(13))
    model, _ = synth.make_config(1)
    gat = form.startswith("attention")
    model.update(hidden=128, precision="fp32" if form.endswith("fp32") else "bf16", rounds=12 if gat else 5, round_kind="gat" if gat else "mlp")
    state = synth.concat_states([synth.make_state(rng, synth.resnet_dag(rng, 4), n, by_block=True) for n in (30, 9)])
    w, got = weights_for(model), []
    up = torch.randn(41, 128, generator=torch.Generator().manual_seed(2)).cuda()
    for room in ("0", None):
        monkeypatch.delenv("XRL_GRAD_ROOM", raising=False)
        if room is not None:
            monkeypatch.setenv("XRL_GRAD_ROOM", room)
        enc = xrl_package.Encoder(model, w)
        batch = enc.pack(state)
        enc.encode(batch, save_for_backward=True)
        assert (enc.batch_level(batch, 0)[0] < batch.N) == (form == "reduced")
        dw = torch.zeros(enc.n_weights, device="cuda")
        enc.encode_backward(batch, up, dw)                    # (workspaces)
        dw.zero_()
        enc.set_timing(True)
        enc.encode_backward(batch, up, dw)
        launches = enc.read_timing("wgrad")[1]
        assert launches >= 5 if room == "0" else launches <= 2
        got.append(dw.double().cpu().numpy())
        batch.free()
        enc.close()
    o = 0
    for name, shape in xrl_package.weight_layout(model):
        a, b = (x[o:o + int(np.prod(shape))] for x in got)
        o += int(np.prod(shape))
        assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b), name
