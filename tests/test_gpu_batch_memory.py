"""Packed batches take their host and device memory from pools: a block that changes hands while the
queue still holds work on its last owner must not disturb that work, whatever the sizes, contexts
and order of frees."""
import numpy as np
import pytest

import paper_2304_14698_amd as xrl
import synth

pytestmark = pytest.mark.gpu


def _setup(sizes):
    import torch
    model, _ = synth.make_config(1)
    rng = np.random.Generator(np.random.PCG64(11))
    weights = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)
    states = []
    for blocks, cand in sizes:
        graphs, mask = synth.make_state(rng, synth.resnet_dag(rng, blocks), cand, by_block=True)
        states.append(synth.concat_states([(graphs, mask)]))
    return torch, model, weights, states


@pytest.mark.parametrize("sizes", [[(2, 3)] * 6, [(2, 3), (8, 40), (2, 5), (8, 41), (16, 90), (2, 3)], [(16, 500), (16, 400)]])
def test_blocks_change_hands_behind_the_queue(sizes):
    torch, model, weights, states = _setup(sizes)
    enc = xrl.Encoder(model, weights)
    want = []
    for st in states:                               # one at a time, waited for
        b = enc.pack(st)
        want.append(enc.encode(b).cpu())
        b.free()
    for _ in range(3):                              # queued back to back, each batch freed at once
        got = []
        for st in states:
            b = enc.pack(st)
            got.append(enc.encode(b))
            b.free()
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert torch.equal(g.cpu(), w)


def test_batch_outlives_its_context_and_serves_another():
    torch, model, weights, states = _setup([(8, 40), (8, 40)])
    side = torch.cuda.Stream()
    a, b = xrl.Encoder(model, weights), xrl.Encoder(model, weights, stream=side)
    first, second = a.pack(states[0]), a.pack(states[1])
    on_a = a.encode(first)
    torch.cuda.synchronize()
    out = torch.empty_like(on_a)
    third = a.pack(states[0])
    torch.cuda.current_stream().wait_stream(side)
    on_b = b.encode(third, out=out)                 # another stream than the upload's, right behind it
    third.free()                                    # (in use on both streams: not recycled)
    again = a.encode(a.pack(states[1]))
    torch.cuda.synchronize()
    assert torch.equal(on_a.cpu(), on_b.cpu())
    a.close()
    late = b.encode(second)
    torch.cuda.synchronize()
    assert torch.equal(late.cpu(), again.cpu())
    first.free()
    second.free()


def test_forked_process_packs_views_and_frees():
    """A worker forked off a process with a context: pinned memory and the pool are not there in it."""
    import os
    import signal
    import time
    torch, model, weights, states = _setup([(8, 40), (4, 10), (2, 3)])
    enc = xrl.Encoder(model, weights)
    first, second = enc.pack(states[0]), xrl.Batch(model, states[1])       # uploaded; packed only
    want = [b.host_view() for b in (first, second)]
    third = enc.pack(states[2])
    want.append(third.host_view())
    emb = enc.encode(first).cpu()
    third.free()                                    # (its block is idle now)
    torch.cuda.synchronize()

    def same(batch, view):
        got = batch.host_view()
        return all(np.array_equal(got[k], view[k]) for k in view)

    pid = os.fork()
    if pid == 0:                                    # (no GPU call from here; nothing of pytest's runs either)
        ok = 0
        try:
            ok += same(first, want[0]) and same(second, want[1])
            mine = [xrl.Batch(model, s) for s in states]
            ok += all(same(b, w) for b, w in zip(mine, want))
            for b in mine + [first, second]:
                b.free()
            ok += same(xrl.Batch(model, states[2]), want[2])
        finally:
            os._exit(0 if ok == 3 else 1)
    for _ in range(600):
        done, status = os.waitpid(pid, os.WNOHANG)
        if done:
            break
        time.sleep(0.05)
    else:
        os.kill(pid, signal.SIGKILL)
        os.waitpid(pid, 0)
        status = -1
    assert status == 0
    assert torch.equal(enc.encode(first).cpu(), emb) and same(enc.pack(states[2]), want[2])
    first.free()
    second.free()
    enc.close()


def test_free_during_another_capture_leaves_no_error():
    """Freeing a batch whose context is on the default stream while a blocking stream is captured: asking for the
    default stream's state fails then, which is no error of the next call."""
    import ctypes as C
    torch, model, weights, states = _setup([(2, 3), (2, 4)])
    hip = xrl.load_library()                        # (its dependencies are looked up with it)
    stream, graph = C.c_void_p(), C.c_void_p()
    assert hip.hipStreamCreate(C.byref(stream)) == 0
    a, b = xrl.Encoder(model, weights), xrl.Encoder(model, weights, stream=torch.cuda.ExternalStream(stream.value))
    mine, other = a.pack(states[0]), b.pack(states[1])
    a.encode(mine)
    want = b.encode(other)
    out = torch.zeros_like(want)
    torch.cuda.synchronize()
    relaxed = 2
    assert hip.hipStreamBeginCapture(stream, relaxed) == 0
    try:
        mine.free()
        b.encode(other, out=out)
    finally:
        assert hip.hipStreamEndCapture(stream, C.byref(graph)) == 0
        assert hip.hipGraphDestroy(graph) == 0
    assert torch.equal(b.encode(other), want)
    other.free()
    a.close()
    b.close()
    assert hip.hipStreamDestroy(stream) == 0


@pytest.mark.parametrize("what", ["upload", "workspace"])
def test_idle_blocks_make_room(what):
    """With the device nearly full, memory that the pool keeps idle is given back before a call is refused."""
    import ctypes as C
    torch, _, _, _ = _setup([])
    model, _ = synth.make_config(1)
    model.update(hidden=256, precision="fp32", rounds=4, n_node_dense=900, n_op_types=32)
    rng = np.random.Generator(np.random.PCG64(2))
    weights = synth.init_weights(rng, xrl.weight_layout(model), bias_range=0.1)

    def state(n):                                   # n graphs of one node, 3.6 KB each
        return dict(n_states=1, state_graph_ptr=np.array([0, n], np.int32), graph_node_ptr=np.arange(n + 1, dtype=np.int32),
                    graph_edge_ptr=np.zeros(n + 1, np.int32), node_op=(np.arange(n) % 32).astype(np.int32),
                    node_dense=np.full((n, 900), 0.25, np.float32), edge_src=np.zeros(0, np.int32), edge_dst=np.zeros(0, np.int32),
                    edge_feat=np.zeros((0, model["d_edge"]), np.float32), graph_global=np.zeros((n, 1), np.float32),
                    slot_mask=np.ones(n, np.uint8))
    small, n, n_big = state(1000), 66000, 160000    # device blocks of 256 and 640 MiB; workspace of 0.9 GB
    hip = xrl.load_library()
    hip.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
    enc = xrl.Encoder(model, weights)
    first = enc.pack(small)
    want = enc.encode(first, save_for_backward=True).cpu()
    emb = torch.empty((n, 256), device="cuda")
    idle = [enc.pack(state(n)) for _ in range(3)]
    if what == "workspace":
        first = enc.pack(state(n))
    for b in idle:
        b.free()
    torch.cuda.synchronize()
    filler = []
    try:
        for _ in range(40):                         # (the free memory reported first is too little)
            left = torch.cuda.mem_get_info()[0] - (512 << 20)
            if left < 16 << 20:
                break
            p = C.c_void_p()
            assert hip.hipMalloc(C.byref(p), min(left, 16 << 30)) == 0
            filler.append(p)
        assert torch.cuda.mem_get_info()[0] < 530 << 20
        if what == "upload":
            big = enc.pack(state(n_big))
            big.free()
            assert torch.equal(enc.encode(first, save_for_backward=True).cpu(), want)
        else:
            enc.encode(first, save_for_backward=True, out=emb)
            torch.cuda.synchronize()
    finally:
        for p in filler:
            hip.hipFree(p)
    if what == "workspace":
        assert torch.equal(emb[:1000].cpu(), want)
    first.free()
    enc.close()


def test_another_contexts_batch_in_a_capture():
    """A batch that one context uploaded, encoded by another one under capture: the wait for its transfer is not
    captured and does not end the capture."""
    torch, model, weights, states = _setup([(4, 10)])
    side = torch.cuda.Stream()
    a, b = xrl.Encoder(model, weights, stream=torch.cuda.Stream()), xrl.Encoder(model, weights, stream=side)
    batch = a.pack(states[0])
    want = a.encode(batch)
    out = torch.empty_like(b.encode(batch))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        b.encode(batch, out=out)
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        eager = a.encode(batch)
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(eager, want)
    batch.free()
    a.close()
    b.close()
