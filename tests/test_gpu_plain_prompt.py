"""Prompts of small plain models go through a layer's launches whole: bit for bit what blocks of 64 rows leave in the cache, at lengths around a block, a
tile of 16 rows and a chunk of 1024, for the types and head widths that the launches take; one of them against the oracle's prefill."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_engine, launch_names, oracle_model, row_rel_err
from oracle import transformer as otf

pytestmark = pytest.mark.gpu
SHAPES = {
    "tiny": synth.SHAPES["tiny_f32"],
    "wide heads": synth.ModelShape("ph", 2, 320, 3, 1, 144, 200, 300, 1e-5, 1e4, "f32"),
    "bf16": synth.ModelShape("pb", 2, 100, 4, 2, 32, 70, 300, 1e-5, 1e4, "bf16"),
    "f16": synth.ModelShape("pq", 3, 68, 4, 4, 80, 33, 300, 1e-5, 1e4, "f16"),
}


@pytest.mark.parametrize("name", SHAPES)
@pytest.mark.parametrize("n,L0", [(1, 0), (63, 2), (64, 0), (65, 0), (80, 47), (129, 64), (1024, 1), (1025, 0), (1100, 600)])
def test_a_whole_prompt_is_its_blocks(name, n, L0):
    import torch
    from paper_2602_16760_amd import binding as B
    sh = SHAPES[name]
    td = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[sh.dtype]
    engines = [gpu_engine(sh, L0 + n, seed=2) for _ in range(2)]
    try:
        tok = torch.arange(n, device="cuda", dtype=torch.int32) * 37 % sh.vocab
        size, g = (L0, sh.n_kv_heads, sh.head_dim), torch.Generator(device="cuda").manual_seed(9)
        for l in range(sh.n_layers if L0 else 0):
            k, v = (torch.randn(size, generator=g, device="cuda").to(td) for _ in "kv")
            for e in engines:
                B.la_kv_fill(e.kv, l, 0, k, v)
        names = launch_names(lambda: B.la_prefill(engines[0].model, engines[0].kv, tok, L0))
        assert "plain_qkv" in names and "rope_table" not in names
        eng = engines[1]
        h = torch.zeros(64, sh.d_model, device="cuda")
        for s in range(0, n, 64):
            r = min(64, n - s)
            B.la_kv_set_len(eng.kv, L0 + s)
            B.la_embed(eng.model, tok[s:s + r].contiguous(), h[:r])
            pos, vis = (B.to_device(a) for a in B.la_causal_layout(L0 + s, r))
            B.la_forward_layers(eng.model, 0, sh.n_layers, h[:r], pos, vis, eng.kv)
        assert B.la_kv_get_len(engines[0].kv) == L0 + n
        for l in range(sh.n_layers):
            rows = [[torch.zeros(n, sh.n_kv_heads, sh.head_dim, dtype=td, device="cuda") for _ in "kv"] for _ in engines]
            for e, r in zip(engines, rows):
                B.la_kv_read(e.kv, l, L0, n, *r)
            for a, b in zip(*rows):
                assert torch.isfinite(a).all() and torch.equal(a, b), l
    finally:
        torch.cuda.synchronize()
        for e in engines:
            e.close()


def test_a_long_prompt_against_the_oracle():
    """1e-4 per row, the bar of the plain kernels' test."""
    import torch
    from paper_2602_16760_amd import binding as B
    sh = SHAPES["tiny"]
    eng, om = gpu_engine(sh, 200, seed=2), oracle_model(sh, seed=2)
    okv = otf.KVCache(sh, 200)
    try:
        tok = np.arange(200, dtype=np.int32) * 37 % sh.vocab
        B.la_prefill(eng.model, eng.kv, B.to_device(tok), 0)
        otf.prefill(om, okv, tok)
        for l in range(sh.n_layers):
            k, v = (torch.zeros(200, sh.n_kv_heads, sh.head_dim, device="cuda") for _ in "kv")
            B.la_kv_read(eng.kv, l, 0, 200, k, v)
            for got, want in ((k, okv.K[l]), (v, okv.V[l])):
                assert row_rel_err(got.cpu().numpy().reshape(200, -1), np.asarray(want)[:200].reshape(200, -1)).max() <= 1e-4
    finally:
        eng.close()


def test_a_first_prompt_can_be_captured():
    import torch
    from paper_2602_16760_amd import binding as B
    sh = SHAPES["tiny"]
    eng, ref = gpu_engine(sh, 300, seed=2), gpu_engine(sh, 300, seed=2)
    stream = torch.cuda.Stream()
    try:
        tok = torch.arange(300, device="cuda", dtype=torch.int32) % sh.vocab
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.la_prefill(eng.model, eng.kv, tok, 0)
        for turn in range(3):
            tok.copy_(torch.arange(300, device="cuda", dtype=torch.int32) * (turn + 3) % sh.vocab)
            B.la_prefill(ref.model, ref.kv, tok, 0)
            graph.replay()
            torch.cuda.synchronize()
            for l in range(sh.n_layers):
                rows = [[torch.zeros(300, sh.n_kv_heads, sh.head_dim, device="cuda") for _ in "kv"] for _ in "er"]
                for e, r in zip((eng, ref), rows):
                    B.la_kv_read(e.kv, l, 0, 300, *r)
                assert all(torch.equal(a, b) for a, b in zip(*rows))
    finally:
        torch.cuda.synchronize()
        eng.close()
        ref.close()


@pytest.mark.parametrize("name,n", [("tiny", 5), ("tiny", 100), ("small_bf16", 5), ("small_bf16", 100)])
def test_a_prompt_that_cannot_run_leaves_its_start_as_the_length(name, n):
    import torch
    from paper_2602_16760_amd import binding as B
    sh = SHAPES.get(name) or synth.SHAPES[name]
    eng = gpu_engine(sh, 300, seed=2)
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[sh.dtype]
    model = B.la_init_model(sh, torch.zeros(sh.vocab, sh.d_model, dtype=dt, device="cuda"))  # (no layer has weights)
    kv = B.la_kv_alloc(model, 300)
    try:
        tok = torch.zeros(n, dtype=torch.int32, device="cuda")
        B.la_kv_set_len(kv, 200)
        with pytest.raises(B.LaError, match="no weights"):
            B.la_prefill(model, kv, tok, 7)
        assert B.la_kv_get_len(kv) == 7
        B.la_prefill(eng.model, eng.kv, tok[:0], 9)
        assert B.la_kv_get_len(eng.kv) == 9
        B.la_prefill(eng.model, eng.kv, tok, 9)
        assert B.la_kv_get_len(eng.kv) == 9 + n
    finally:
        torch.cuda.synchronize()
        B.la_free_kv(kv)
        B.la_free_model(model)
        eng.close()
