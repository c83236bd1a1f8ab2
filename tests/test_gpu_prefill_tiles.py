"""The prompt pass at the sizes where its tiles, slices of the contraction, key blocks and chunks change,
against a float64 torch model of two layers of the 7B width (and of the 64-channel heads)."""
import math
import zlib
from dataclasses import replace

import pytest

import synth
from gpu_util import launch_names

pytestmark = pytest.mark.gpu
# (shape, dtype, [(tokens, start)]).  Every kernel that the pass picks from for these shapes between 65 and 2200 tokens, and every number of slices of O
# and of down with each, runs at one of these sizes or of test_prefill_rows.py's: test_prefill_plan.py asserts it, without a GPU.
SIZES = [
    ("mistral7b", "bf16", [(65, 0), (81, 20), (97, 3), (113, 0), (128, 1), (130, 37), (180, 3), (257, 0), (300, 31), (513, 0), (600, 0), (700, 5),
                           (1023, 0), (1100, 32), (1300, 0), (1600, 0), (1601, 0), (2049, 3), (2200, 3)]),
    ("mistral7b", "f16", [(193, 33), (1025, 0)]),
    ("nemo12b", "bf16", [(81, 0), (105, 0), (191, 5), (257, 0), (400, 64), (1024, 0), (1055, 0), (2049, 0)]),
    ("mistral7b/32 kv heads", "bf16", [(65, 0), (128, 9)]),  # (12288 columns of QKV: more than one round of the few-row product)
    ("small64_bf16", "bf16", [(65, 7), (90, 33), (128, 0), (191, 0), (440, 0), (820, 33), (879, 0), (2049, 100)]),
]
# max |got - want| over max |want| of a layer's cache rows: the bars of the prompt-pass parity tests (one storage
# rounding of the rows on top of the hidden-state error of one layer)
TOL = {"bf16": 2e-2, "f16": 2e-3}


def _normal(name, size, std, dtype):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(zlib.crc32(name.encode()))
    return torch.randn(size, generator=g, device="cuda").mul_(std).to(dtype)


def _layer(sh, l, dtype):
    import torch
    d, F, q, kv = sh.d_model, sh.d_ffn, sh.q_dim, sh.kv_dim
    size = {"wq": (d, q), "wk": (d, kv), "wv": (d, kv), "wo": (q, d), "wgate": (d, F), "wup": (d, F), "wdown": (F, d)}
    w = {k: _normal(f"{l}/{k}", s, 0.02, dtype) for k, s in size.items()}
    for k in ("g_attn", "g_mlp"):
        w[k] = 1.0 + 0.1 * _normal(f"{l}/{k}", (d,), 1.0, torch.float32)
    return w


def _reference(sh, embed, tok, L0, old, dtype):
    """K, V rows L0 .. of every layer in float64, all layers' weights made again."""
    import torch
    dev, f8 = "cuda", torch.float64
    n, half, g = len(tok), sh.head_dim // 2, sh.n_q_heads // sh.n_kv_heads
    pos = torch.arange(L0, L0 + n, device=dev, dtype=f8)
    ang = pos[:, None, None] * torch.pow(torch.tensor(sh.rope_theta, dtype=f8, device=dev), -torch.arange(half, device=dev, dtype=f8) / half)
    norm = lambda x, gain: x * torch.rsqrt(x.square().mean(1, keepdim=True) + sh.rms_eps) * gain.double()

    def rope(y):
        a, b = y[..., :half], y[..., half:]
        return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)

    see = torch.ones((n, L0 + n), dtype=torch.bool, device=dev).tril(L0)
    x, out = embed[tok.long()].double(), []
    for l in range(sh.n_layers):
        w = _layer(sh, l, dtype)
        h = norm(x, w["g_attn"])
        q = rope((h @ w["wq"].double()).view(n, sh.n_q_heads, sh.head_dim))
        k = rope((h @ w["wk"].double()).view(n, sh.n_kv_heads, sh.head_dim))
        v = (h @ w["wv"].double()).view(n, sh.n_kv_heads, sh.head_dim)
        out.append((k, v))
        if l + 1 == sh.n_layers:
            break
        ka, va = torch.cat([old[l][0].double(), k]), torch.cat([old[l][1].double(), v])
        o = torch.empty_like(q)
        for i in range(sh.n_q_heads):
            s = q[:, i] @ ka[:, i // g].t() / math.sqrt(sh.head_dim)
            o[:, i] = torch.softmax(s.masked_fill(~see, -math.inf), 1) @ va[:, i // g]
        x = x + o.reshape(n, -1) @ w["wo"].double()
        h = norm(x, w["g_mlp"])
        x = x + (torch.nn.functional.silu(h @ w["wgate"].double()) * (h @ w["wup"].double())) @ w["wdown"].double()
    return out


def shape_of(name, dtype):
    name, _, wide = name.partition("/")
    return replace(synth.SHAPES[name], n_layers=2, dtype=dtype, vocab=512, **({"n_kv_heads": 32} if wide else {}))


@pytest.mark.parametrize("name,dtype,cases", SIZES)
def test_prompt_pass_sizes(name, dtype, cases):
    import torch
    from paper_2602_16760_amd import binding as B
    sh = shape_of(name, dtype)
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    embed = _normal("embed", (sh.vocab, sh.d_model), 1.0, td)
    model = B.la_init_model(sh, embed)
    try:
        for l in range(sh.n_layers):
            B.la_model_set_layer(model, l, _layer(sh, l, td))
            torch.cuda.synchronize()
        for n, L0 in cases:
            print(f"{name} {dtype}: {n} tokens at {L0}", flush=True)
            kv = B.la_kv_alloc(model, L0 + n)
            try:
                old = [tuple(_normal(f"{l}/{c}", (L0, sh.n_kv_heads, sh.head_dim), 1.0, td) for c in "kv") for l in range(sh.n_layers)]
                if L0:
                    for l in range(sh.n_layers):
                        B.la_kv_fill(kv, l, 0, *old[l])
                tok = torch.randint(0, sh.vocab, (n,), device="cuda", dtype=torch.int32, generator=torch.Generator(device="cuda").manual_seed(n))
                B.la_prefill(model, kv, tok, L0)
                assert B.la_kv_get_len(kv) == L0 + n
                for l, want in enumerate(_reference(sh, embed, tok, L0, old, td)):
                    got = [torch.empty((n, sh.n_kv_heads, sh.head_dim), dtype=td, device="cuda") for _ in "kv"]
                    B.la_kv_read(kv, l, L0, n, *got)
                    for c, a, b in zip("KV", got, want):
                        e = ((a.double() - b).abs().max() / b.abs().max()).item()
                        assert e <= TOL[dtype], f"{n} tokens at {L0}, layer {l} {c}: {e:.3e}"
            finally:
                torch.cuda.synchronize()
                B.la_free_kv(kv)
    finally:
        torch.cuda.synchronize()
        B.la_free_model(model)


@pytest.mark.parametrize("name,dtype,piece", [("mistral7b", "bf16", 64), ("mistral7b", "bf16", 61), ("mistral7b", "f16", 50), ("small64_bf16", "bf16", 45)])
def test_prompt_pass_agrees_with_the_block_kernel(name, dtype, piece):
    """One call of 300 tokens (the large-M pass) against pieces that go through the block kernel, at starts inside and on the
    edges of key blocks.  The two add in another order: a stored element moves by one step of its type where the sums fall
    on either side of a rounding, at most 2^-7 (bf16) or 2^-10 (f16) of the largest one, and the second layer's inputs by what
    such steps do to the first one's output; as much again is allowed for that."""
    import torch
    from paper_2602_16760_amd import binding as B
    sh = shape_of(name, dtype)
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    bar = 2.0 ** (-6 if dtype == "bf16" else -9)
    embed = _normal("embed", (sh.vocab, sh.d_model), 1.0, td)
    model = B.la_init_model(sh, embed)
    kvs = [B.la_kv_alloc(model, 300) for _ in range(2)]
    try:
        for l in range(sh.n_layers):
            B.la_model_set_layer(model, l, _layer(sh, l, td))
            torch.cuda.synchronize()
        tok = torch.arange(300, device="cuda", dtype=torch.int32) * 7 % sh.vocab

        def pieces():
            for s in range(0, 300, piece):
                B.la_prefill(model, kvs[1], tok[s:s + piece].contiguous(), s)

        assert "layer_stack" not in launch_names(lambda: B.la_prefill(model, kvs[0], tok, 0))
        assert not any(n.startswith("pf_") for n in launch_names(pieces))
        for l in range(sh.n_layers):
            rows = [[torch.empty((300, sh.n_kv_heads, sh.head_dim), dtype=td, device="cuda") for _ in "kv"] for _ in kvs]
            for kv, r in zip(kvs, rows):
                B.la_kv_read(kv, l, 0, 300, *r)
            for c, a, b in zip("KV", *rows):
                e = ((a.double() - b.double()).abs().max() / b.double().abs().max()).item()
                print(f"{name} {dtype} pieces of {piece}, layer {l} {c}: {e:.2e}", flush=True)
                assert e <= bar
    finally:
        torch.cuda.synchronize()
        for kv in kvs:
            B.la_free_kv(kv)
        B.la_free_model(model)


def test_a_token_that_is_not_finite_stays_out_of_the_key_blocks_before_it():
    """Rows whose 32-key block ends before the token: bit for bit what they are without it (a masked key's probability is
    zero, and zero times a value that is not finite would not be)."""
    import torch
    from paper_2602_16760_amd import binding as B
    sh = replace(synth.SHAPES["mistral7b"], n_layers=2, vocab=512)
    embed = _normal("embed", (sh.vocab, sh.d_model), 1.0, torch.bfloat16)
    embed[511] = float("nan")
    model = B.la_init_model(sh, embed)
    try:
        for l in range(sh.n_layers):
            B.la_model_set_layer(model, l, _layer(sh, l, torch.bfloat16))
            torch.cuda.synchronize()
        for n, at in ((100, 32), (200, 100), (300, 255)):
            got = []
            for bad in (False, True):
                tok = torch.arange(n, device="cuda", dtype=torch.int32) * 7 % 511
                if bad:
                    tok[at] = 511
                kv = B.la_kv_alloc(model, n)
                try:
                    B.la_prefill(model, kv, tok, 0)
                    rows = [[torch.empty((at // 32 * 32, sh.n_kv_heads, sh.head_dim), dtype=torch.bfloat16, device="cuda") for _ in "kv"]
                            for _ in range(sh.n_layers)]
                    for l in range(sh.n_layers):
                        B.la_kv_read(kv, l, 0, at // 32 * 32, *rows[l])
                    got.append(rows)
                finally:
                    torch.cuda.synchronize()
                    B.la_free_kv(kv)
            for a, b in zip(got[0], got[1]):
                assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), f"{n} tokens, token {at}"
    finally:
        torch.cuda.synchronize()
        B.la_free_model(model)
