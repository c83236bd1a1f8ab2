"""The prompt pass's buffers: what a short prompt takes of the card, and first prompts that are captured into a graph."""
from dataclasses import replace

import pytest

import synth
from test_gpu_prefill_tiles import _layer, _normal

pytestmark = pytest.mark.gpu


def _model(sh):
    import torch
    from paper_2602_16760_amd import binding as B
    model = B.la_init_model(sh, _normal("embed", (sh.vocab, sh.d_model), 1.0, torch.bfloat16))
    for l in range(sh.n_layers):
        B.la_model_set_layer(model, l, _layer(sh, l, torch.bfloat16))
        torch.cuda.synchronize()
    return model


def test_prompts_below_128_tokens_take_no_whole_chunks_buffers():
    import torch
    from paper_2602_16760_amd import binding as B
    sh = replace(synth.SHAPES["mistral7b"], n_layers=2, vocab=512)
    model = _model(sh)
    kv = B.la_kv_alloc(model, 256)
    tok = torch.arange(256, device="cuda", dtype=torch.int32)

    def taken(n):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        B.la_prefill(model, kv, tok[:n], 0)
        torch.cuda.synchronize()
        return before - torch.cuda.mem_get_info()[0]

    try:
        taken(64)  # (block kernel; whatever the runtime sets up on a first launch)
        # 128 rows of every buffer, 1024 rows of the slices' products: 26.4 MB, and the driver's rounding
        assert taken(65) <= 32e6
        assert taken(127) == 0 and taken(100) == 0
        assert taken(128) >= 100e6 and taken(127) == 0 and taken(256) == 0
    finally:
        torch.cuda.synchronize()
        B.la_free_kv(kv)
        B.la_free_model(model)


@pytest.mark.parametrize("n", [100, 300])
def test_a_first_prompt_can_be_captured(n):
    """The model has only run a short prompt: the captured call is the one that needs the buffers.  Every replay, with eager
    work in between, against another model's eager call: the same kernels on the same rows, bit for bit."""
    import torch
    from paper_2602_16760_amd import binding as B
    sh = replace(synth.SHAPES["small_bf16"], vocab=512)
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
        B.la_prefill(models[0], kvs[0], tok[:40], 0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.la_prefill(models[0], kvs[0], tok, 0)
        for turn in range(3):
            tok.copy_(torch.arange(n, device="cuda", dtype=torch.int32) * (7 + turn) % sh.vocab)
            graph.replay()
            got = rows(kvs[0])
            assert B.la_kv_get_len(kvs[0]) == n
            B.la_prefill(models[1], kvs[1], tok, 0)
            assert all(torch.equal(a, b) for a, b in zip(got, rows(kvs[1]))), f"replay {turn}"
            B.la_prefill(models[0], kvs[0], tok[:50], 0)  # (the model goes on being used between the replays)
            torch.cuda.synchronize()
    finally:
        torch.cuda.synchronize()
        for kv in kvs:
            B.la_free_kv(kv)
        for m in models:
            B.la_free_model(m)
