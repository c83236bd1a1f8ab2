"""Calls of the matrix-core path's block kernel captured into a graph: every replay, with eager calls between them, gives what the
eager call gives, bit for bit."""
from dataclasses import replace

import numpy as np
import pytest

import synth
from gpu_util import gpu_engine
from test_gpu_prefill_buffers import _model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("env", [{}, {"LA_WGS": "37"}, {"LA_LDS_RING": "1"}])
def test_replayed_layers_and_head(monkeypatch, env):
    """(LA_LDS_RING: the earlier persistent kernel, whose barrier counts arrivals.)"""
    import torch
    from paper_2602_16760_amd import binding as B
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    shape, L, rows = synth.SHAPES["small_bf16"], 45, 31
    eng = gpu_engine(shape, L + rows, seed=3)
    stream = torch.cuda.Stream()
    try:
        for l in range(shape.n_layers):
            eng.fill_kv(l, *synth.kv_fill(shape, l, L, 4))
        B.la_kv_set_len(eng.kv, L)
        pos, vis = (B.to_device(a) for a in B.la_lookahead_layout(5, 4, 5, L, 5, rows))
        blocks = [torch.from_numpy(np.ascontiguousarray(synth.hidden_block(shape, rows, s), dtype=np.float32)).cuda() for s in range(3)]
        x = blocks[0].clone()

        def buffers():
            return x.clone(), torch.zeros(rows, dtype=torch.int32, device="cuda"), torch.zeros((rows, 2), device="cuda")

        def step(h, ids, top2):
            h.copy_(x)
            B.la_forward_layers(eng.model, 0, shape.n_layers, h, pos, vis, eng.kv)
            B.la_unembed_argmax(eng.model, h, ids, top2)

        want, eager, captured = [], buffers(), buffers()
        for b in blocks:
            x.copy_(b)
            step(*eager)
            want.append([t.clone() for t in eager])
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            step(*captured)
        for turn, between in enumerate((0, 1, 0, 3, 1, 2)):
            x.copy_(blocks[turn % 3])
            for t in captured:
                t.zero_()
            graph.replay()
            for got, w in zip(captured, want[turn % 3]):
                assert torch.equal(got, w), f"replay {turn}"
            for k in range(between):
                x.copy_(blocks[k])
                step(*eager)
                for got, w in zip(eager, want[k]):
                    assert torch.equal(got, w), f"eager call {k} behind replay {turn}"
        torch.cuda.synchronize()
        assert B.la_kv_get_len(eng.kv) == L  # (no error is pending either)
    finally:
        torch.cuda.synchronize()
        eng.close()


def test_replayed_short_prompt():
    """A prompt that goes through the block kernel."""
    import torch
    from paper_2602_16760_amd import binding as B
    n, sh = 50, replace(synth.SHAPES["small_bf16"], vocab=512)
    models = [_model(sh) for _ in range(2)]
    kvs = [B.la_kv_alloc(m, 320) for m in models]
    tok = torch.zeros(n, device="cuda", dtype=torch.int32)
    stream = torch.cuda.Stream()

    def rows(kv):
        out = [[torch.empty((n, sh.n_kv_heads, sh.head_dim), dtype=torch.bfloat16, device="cuda") for _ in "kv"] for _ in range(sh.n_layers)]
        for l, r in enumerate(out):
            B.la_kv_read(kv, l, 0, n, *r)
        return [x for r in out for x in r]

    try:
        B.la_prefill(models[0], kvs[0], tok[:40], 0)  # (a model's first block uploads its gains and waits)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.la_prefill(models[0], kvs[0], tok, 0)
        for turn in range(5):
            tok.copy_(torch.arange(n, device="cuda", dtype=torch.int32) * (7 + turn) % sh.vocab)
            graph.replay()
            got = rows(kvs[0])
            assert B.la_kv_get_len(kvs[0]) == n
            B.la_prefill(models[1], kvs[1], tok, 0)
            assert all(torch.equal(a, b) for a, b in zip(got, rows(kvs[1]))), f"replay {turn}"
            for k in range(turn % 3):
                B.la_prefill(models[0], kvs[0], tok[:31 + k], 0)  # (the model goes on being used between the replays)
            torch.cuda.synchronize()
    finally:
        torch.cuda.synchronize()
        for kv in kvs:
            B.la_free_kv(kv)
        for m in models:
            B.la_free_model(m)


@pytest.mark.parametrize("name", ["tiny_f32", "small_bf16"])
def test_the_legacy_stream_beside_a_capture(name):
    """While a blocking stream captures, the runtime does not tell whether the legacy stream does; a block on it runs as ever."""
    import ctypes as C
    import torch
    from paper_2602_16760_amd import binding as B
    hip = C.CDLL("libamdhip64.so")
    shape, rows, L = synth.SHAPES[name], 17, 40
    eng = gpu_engine(shape, 100, seed=3)
    blocking, graph = C.c_void_p(), C.c_void_p()
    try:
        for l in range(shape.n_layers):
            eng.fill_kv(l, *synth.kv_fill(shape, l, L, 4))
        B.la_kv_set_len(eng.kv, L)
        pos, vis = (B.to_device(a) for a in B.la_causal_layout(L, rows))
        x = torch.from_numpy(np.ascontiguousarray(synth.hidden_block(shape, rows, 3), dtype=np.float32)).cuda()
        want, got = x.clone(), [x.clone() for _ in range(3)]
        B.la_forward_layers(eng.model, 0, shape.n_layers, want, pos, vis, eng.kv)
        torch.cuda.synchronize()
        assert torch.cuda.current_stream().cuda_stream == 0
        assert hip.hipStreamCreate(C.byref(blocking)) == 0
        assert hip.hipStreamBeginCapture(blocking, 2) == 0  # (relaxed: the thread's other calls stay allowed)
        try:
            for h in got[:2]:
                B.la_forward_layers(eng.model, 0, shape.n_layers, h, pos, vis, eng.kv)
        finally:
            assert hip.hipStreamEndCapture(blocking, C.byref(graph)) == 0
        B.la_forward_layers(eng.model, 0, shape.n_layers, got[2], pos, vis, eng.kv)
        torch.cuda.synchronize()
        assert all(torch.equal(h, want) for h in got)
    finally:
        if graph:
            hip.hipGraphDestroy(graph)
        if blocking:
            hip.hipStreamDestroy(blocking)
        torch.cuda.synchronize()
        eng.close()


def test_recovery_does_not_wait_for_a_graph():
    """A reported error is cleared by the next launch; where that one is captured, by the next one outside the graph as well, which may
    never run."""
    import torch
    from paper_2602_16760_amd import binding as B
    shape, L0, rows, max_len = synth.SHAPES["tiny_f32"], 40, 17, 64
    eng = gpu_engine(shape, max_len, seed=3)
    stream, accept, forward = torch.cuda.Stream(), torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    try:
        prompt = B.to_device(np.zeros(L0 + 1, dtype=np.int32))
        state, emitted, ids = B.new_state(), torch.zeros(max_len, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        pos, vis = (B.to_device(a) for a in B.la_causal_layout(L0, rows))
        h = torch.zeros((rows, shape.d_model), device="cuda")
        B.la_jacobi_init(eng.kv, 1, prompt, 1, state)
        torch.cuda.synchronize()
        with torch.cuda.graph(accept, stream=stream):
            B.la_jacobi_accept(eng.kv, 1, ids, state, emitted, max_len)
        for _ in range(max_len - L0 - rows + 1):
            accept.replay()
        B.la_forward_layers(eng.model, 0, shape.n_layers, h, pos, vis, eng.kv)  # skipped: only the device knows the length
        torch.cuda.synchronize()
        with pytest.raises(B.LaError):
            B.la_kv_set_len(eng.kv, L0)
        B.la_kv_set_len(eng.kv, L0)
        torch.cuda.synchronize()
        with torch.cuda.graph(forward, stream=stream):
            B.la_forward_layers(eng.model, 0, shape.n_layers, h, pos, vis, eng.kv)
        B.la_forward_layers(eng.model, 0, shape.n_layers, h, pos, vis, eng.kv)
        B.la_jacobi_init(eng.kv, 1, prompt, 1, state)
        B.la_jacobi_accept(eng.kv, 1, ids, state, emitted, max_len)
        assert B.read_state(state).error == 0
        assert B.la_kv_get_len(eng.kv) == L0 + 1
        forward.replay()
        torch.cuda.synchronize()
        assert B.la_kv_get_len(eng.kv) == L0 + 1
    finally:
        torch.cuda.synchronize()
        eng.close()
