"""The work that programs built on this library have it do, as cases to be timed.

A case is one of four calls or call sequences, each through the public binding:

  step        one decode step of a layer range: la_embed, la_forward_layers, la_unembed_argmax
  unembed     the head alone: la_unembed_argmax
  prompt      the prompt pass (la_prefill) and the cache rows it leaves (la_kv_read), as a program
              that keeps prompt caches has them
  controller  a generation's integer side: la_state_init on a prompt, then a number of accept calls
              (la_ngram_accept or la_jacobi_accept) in a closed loop whose arg-max ids come from a
              successor table, so that candidates are confirmed and cache rows relocated

Model shapes are the repository's own (synth.SHAPES).  Weights are N(0, 0.02), norm gains U(0.5, 1.5),
committed cache rows N(0, 1), all drawn on the GPU from the seed.
"""
from __future__ import annotations

import math
import zlib
from dataclasses import replace

import torch

import synth
from paper_2602_16760_amd import binding as B

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def listed():
    def step(name, shape, layers, L, W, N, G, rows, dtype="bf16"):
        return {"name": name, "kind": "step", "shape": shape, "dtype": dtype, "layers": layers, "L": L,
                "W": W, "N": N, "G": G, "rows": rows}

    def prompt(name, shape, layers, n, L0, dtype="bf16"):
        return {"name": name, "kind": "prompt", "shape": shape, "dtype": dtype, "layers": layers, "n": n, "L0": L0}

    return [
        # the tiny fp32 decoder on one device: every call is launch latency
        step("tiny_f32_block17", "tiny_f32", 2, 47, 4, 3, 4, 17, "f32"),
        # a small model with ragged tile counts: the smallest blocks of the matrix-core path
        step("small_bf16_block31", "small_bf16", 3, 301, 5, 4, 5, 31),
        # sequential decoding of the 7B-shaped cloud share (30 layers behind a 2-layer split)
        step("7b_one_row", "mistral7b", 30, 512, 0, 1, 0, 1),
        # the verification step itself: 31 rows padded to 32
        step("7b_block32", "mistral7b", 30, 512, 5, 4, 5, 32),
        # a wider block against a longer context (24 layers behind an 8-layer split)
        step("7b_block43_ctx2048", "mistral7b", 24, 2048, 7, 4, 7, 43),
        # the 12B-shaped cloud share with its large vocabulary
        step("12b_block32_ctx4096", "nemo12b", 38, 4096, 5, 4, 5, 32),
        # the two local head layers in half-precision storage, the fullest block a call takes
        step("7b_f16_head_block64", "mistral7b", 2, 1000, 10, 4, 11, 64, "f16"),
        # the head of the 12B shape alone: a block's arg-max over 131072 entries
        {"name": "12b_unembed_32", "kind": "unembed", "shape": "nemo12b", "dtype": "bf16", "rows": 32},
        # a short chat turn, an ordinary prompt, a long document that continues a conversation
        prompt("7b_prompt_77", "mistral7b", 8, 77, 0),
        prompt("7b_prompt_1023", "mistral7b", 8, 1023, 0),
        prompt("7b_prompt_3000_at_1000", "mistral7b", 4, 3000, 1000),
        # pool seeding from a 2048-token prompt and sixteen accepts
        {"name": "controller_2048", "kind": "controller", "shape": "mistral7b", "dtype": "bf16", "mode": "lookahead",
         "P": 2048, "W": 7, "N": 4, "G": 7, "rows": 43, "steps": 16},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _lookahead(rng):
    """W, N, G and block rows of one lookahead block, sequential decoding among them."""
    if rng.random() < 0.2:
        return 0, 1, 0, 1
    N = rng.randint(2, 7)
    most = 63 // (N - 1)  # W + G
    W = rng.randint(1, max(1, min(15, most - 1)))
    G = rng.randint(0, max(0, min(15, most - W)))
    used = 1 + (W + G) * (N - 1)
    return W, N, G, min(64, used + rng.choice([0, 0, 1, 3]))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "unembed", "prompt", "prompt", "controller"])
    # the two large shapes are what the library is for; the small ones are what tests and trials run
    shape = rng.choice(["mistral7b", "mistral7b", "nemo12b", "small_bf16", "small64_bf16", "tiny_f32"])
    most = {"mistral7b": 30, "nemo12b": 24, "small_bf16": 3, "small64_bf16": 2, "tiny_f32": 2}[shape]
    dtype = "f32" if shape == "tiny_f32" else rng.choice(["bf16", "bf16", "f16"])
    W, N, G, rows = _lookahead(rng)
    if kind == "step":
        return {"kind": kind, "shape": shape, "dtype": dtype, "layers": rng.randint(1, most),
                "L": _log_int(rng, 1, 4096) - 1, "W": W, "N": N, "G": G, "rows": rows}
    if kind == "unembed":
        return {"kind": kind, "shape": shape, "dtype": dtype, "rows": rng.randint(1, 64)}
    if kind == "prompt":
        n = _log_int(rng, 1, 4000)
        cost = 24000 if shape == "mistral7b" else 12000  # n x layers
        return {"kind": kind, "shape": shape, "dtype": dtype, "layers": max(1, min(most, 8, cost // (2 * n))), "n": n,
                "L0": rng.choice([0, 0, _log_int(rng, 1, 2000)])}
    mode = rng.choice(["lookahead", "lookahead", "jacobi"])
    if mode == "jacobi":
        rows = rng.randint(1, 32)
        W, N, G = 0, 1, 0
    return {"kind": kind, "shape": shape, "dtype": dtype, "mode": mode, "P": _log_int(rng, 4, 4096), "W": W, "N": N, "G": G,
            "rows": rows, "steps": rng.randint(1, 32)}


# ---- inputs -------------------------------------------------------------------------------------
def _shape(case):
    sh = synth.SHAPES[case["shape"]]
    return replace(sh, n_layers=case.get("layers", 2 if case["kind"] == "controller" else 1), dtype=case["dtype"])


def _gen(seed, name):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 0x9E3779B1 + zlib.crc32(name.encode())) % (1 << 62))
    return g


def _normal(seed, name, size, std, dtype):
    x = torch.randn(size, generator=_gen(seed, name), device="cuda", dtype=torch.float32)
    return x.mul_(std).to(dtype) if std != 1.0 else x.to(dtype)


def _gain(seed, name, n):
    return torch.rand(n, generator=_gen(seed, name), device="cuda").add_(0.5)


def _ints(seed, name, n, high):
    return torch.randint(0, high, (n,), generator=_gen(seed, name), device="cuda", dtype=torch.int32)


def _layer(sh, seed, l):
    d, F, q, kv, t = sh.d_model, sh.d_ffn, sh.q_dim, sh.kv_dim, DTYPES[sh.dtype]
    sizes = {"wq": (d, q), "wk": (d, kv), "wv": (d, kv), "wo": (q, d), "wgate": (d, F), "wup": (d, F), "wdown": (F, d)}
    w = {k: _normal(seed, f"L{l}/{k}", s, 0.02, t) for k, s in sizes.items()}
    w["g_attn"], w["g_mlp"] = _gain(seed, f"L{l}/g_attn", d), _gain(seed, f"L{l}/g_mlp", d)
    return w


def _embed(sh, seed):
    return _normal(seed, "embed", (sh.vocab, sh.d_model), 0.02, DTYPES[sh.dtype])


def _unembed(sh, seed):
    return _normal(seed, "unembed", (sh.d_model, sh.vocab), 0.02, DTYPES[sh.dtype])


def _kv_rows(sh, seed, l, n):
    size = (n, sh.n_kv_heads, sh.head_dim)
    return _normal(seed, f"L{l}/k", size, 1.0, DTYPES[sh.dtype]), _normal(seed, f"L{l}/v", size, 1.0, DTYPES[sh.dtype])


def _unembed_hidden(case, sh, seed, unembed):
    """Rows as a trained model leaves them: each leans towards the entry it is about to choose."""
    h = _normal(seed, "hidden", (case["rows"], sh.d_model), 1.0, torch.float32)
    target = _ints(seed, "target", case["rows"], sh.vocab).long()
    u = unembed[:, target].float().t()
    lean = 6.0 + 8.0 * torch.rand((case["rows"], 1), generator=_gen(seed, "lean"), device="cuda")
    return (h + lean * u * (math.sqrt(sh.d_model) * 0.02 / u.square().sum(1, keepdim=True))
            * math.sqrt(4096 / sh.d_model)).contiguous()


def _text(case, sh, seed):
    """A code-like prompt and, for each token, what follows it: the token that followed it last in the prompt, and a
    random one for tokens the prompt does not hold."""
    prompt = torch.from_numpy(synth.markov_prompt(sh.vocab, case["P"], 0.30, int(seed) % (1 << 31)).astype("int64")).cuda()
    follow = _ints(seed, "follow", sh.vocab, sh.vocab)
    last = torch.full((sh.vocab,), -1, dtype=torch.int64, device="cuda")
    last.scatter_reduce_(0, prompt[:-1], torch.arange(case["P"] - 1, device="cuda"), "amax")
    seen = last >= 0
    follow[seen] = prompt[last[seen] + 1].int()
    return prompt.int(), follow


class State:
    """The handles and buffers one program keeps; frees the library's handles with itself."""

    def __init__(self, case):
        self.case, self.model, self.kv, self.pool = case, None, None, None

    def __del__(self):
        for handle, free in ((self.pool, B.la_free_pool), (self.kv, B.la_free_kv), (self.model, B.la_free_model)):
            if handle is not None:
                free(handle)


def prepare(case, seed):
    sh, kind = _shape(case), case["kind"]
    s = State(case)
    s.sh = sh
    embed = _embed(sh, seed) if kind in ("step", "prompt") else None
    unembed = _unembed(sh, seed) if kind in ("step", "unembed") else None
    g_final = _gain(seed, "g_final", sh.d_model) if unembed is not None else None
    s.model = B.la_init_model(sh, embed, g_final, unembed)
    if kind in ("step", "prompt"):
        for l in range(sh.n_layers):
            w = _layer(sh, seed, l)
            B.la_model_set_layer(s.model, l, w)
            torch.cuda.synchronize()
            del w
    if kind == "unembed":
        s.hidden = _unembed_hidden(case, sh, seed, unembed)
    rows = case.get("rows", 1)
    s.ids = torch.zeros(rows, dtype=torch.int32, device="cuda")
    s.top2 = torch.zeros((rows, 2), dtype=torch.float32, device="cuda")
    if kind == "step":
        L = case["L"]
        s.kv = B.la_kv_alloc(s.model, L + rows + 32)
        if L:
            for l in range(sh.n_layers):
                B.la_kv_fill(s.kv, l, 0, *_kv_rows(sh, seed, l, L))
                torch.cuda.synchronize()
        B.la_kv_set_len(s.kv, L)
        pos, vis = B.la_lookahead_layout(case["W"], case["N"], case["G"], L, case["G"], rows)
        s.pos, s.vis = B.to_device(pos), B.to_device(vis)
        s.tok = _ints(seed, "tok", rows, sh.vocab)
        s.hidden = torch.zeros((rows, sh.d_model), dtype=torch.float32, device="cuda")
    elif kind == "prompt":
        n, L0 = case["n"], case["L0"]
        s.kv = B.la_kv_alloc(s.model, L0 + n + 64)
        if L0:
            for l in range(sh.n_layers):
                B.la_kv_fill(s.kv, l, 0, *_kv_rows(sh, seed, l, L0))
                torch.cuda.synchronize()
        s.tok = _ints(seed, "tok", n, sh.vocab)
        size = (n, sh.n_kv_heads, sh.head_dim)
        s.rows = [[torch.zeros(size, dtype=DTYPES[sh.dtype], device="cuda") for _ in "kv"] for _ in range(sh.n_layers)]
    elif kind == "controller":
        P = case["P"]
        # what a generation of this length and one more block can reach
        s.total = case["steps"] * max(case["N"], rows if case["mode"] == "jacobi" else 1)
        s.kv = B.la_kv_alloc(s.model, P + s.total + 128)
        s.prompt, s.follow = _text(case, sh, seed)
        s.state = B.new_state()
        s.tok = B.state_field(s.state, "tok")[:rows]
        s.emitted = torch.zeros(s.total, dtype=torch.int32, device="cuda")
        if case["mode"] == "lookahead":
            s.pool = B.la_pool_alloc(sh.vocab, case["N"], case["G"])
        s.block = [_kv_rows(sh, seed, l, s.total + 64) for l in range(sh.n_layers)]
        s.rows = [[torch.zeros_like(x) for x in kv] for kv in s.block]
    torch.cuda.synchronize()
    return s


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "step":
        B.la_embed(s.model, s.tok, s.hidden)
        B.la_forward_layers(s.model, 0, s.sh.n_layers, s.hidden, s.pos, s.vis, s.kv)
        B.la_unembed_argmax(s.model, s.hidden, s.ids, s.top2)
        # the ids of random weights are near-ties that rounding decides: the two largest logits stand for them
        return {"hidden": s.hidden, "top2": s.top2}
    if kind == "unembed":
        B.la_unembed_argmax(s.model, s.hidden, s.ids, s.top2)
        return {"ids": s.ids, "top2": s.top2}
    if kind == "prompt":
        B.la_prefill(s.model, s.kv, s.tok, case["L0"])
        for l, (k, v) in enumerate(s.rows):
            B.la_kv_read(s.kv, l, case["L0"], case["n"], k, v)
        return s.rows
    # controller
    W, N, G, rows, P = case["W"], case["N"], case["G"], case["rows"], case["P"]
    for l, (k, v) in enumerate(s.block):  # (the rows that the layers would have written)
        B.la_kv_fill(s.kv, l, P - 1, k, v)
    if case["mode"] == "lookahead":
        B.la_state_init(s.pool, s.kv, W, N, G, s.prompt, rows, True, s.state)
    else:
        B.la_jacobi_init(s.kv, rows, s.prompt, rows, s.state)
    for _ in range(case["steps"]):
        torch.index_select(s.follow, 0, s.tok, out=s.ids)
        if case["mode"] == "lookahead":
            B.la_ngram_accept(s.pool, s.kv, W, N, G, s.ids, s.state, s.emitted, s.total)
        else:
            B.la_jacobi_accept(s.kv, rows, s.ids, s.state, s.emitted, s.total)
    for l, (k, v) in enumerate(s.rows):
        B.la_kv_read(s.kv, l, P - 1, k.shape[0], k, v)
    return {"state": s.state, "emitted": s.emitted, "cache": s.rows}


# ---- what a pass cannot do without ----------------------------------------------------------------
def work(case):
    sh, kind = _shape(case), case["kind"]
    e = 4 if sh.dtype == "f32" else 2
    d, F, q, kv = sh.d_model, sh.d_ffn, sh.q_dim, sh.kv_dim
    mats = d * (q + 2 * kv) + q * d + 3 * d * F  # weights of one layer
    head = d * sh.vocab
    rows = case.get("rows", 1)
    if kind == "step":
        L, n = case["L"], sh.n_layers
        return {"bytes": n * (mats * e + (L + rows) * 2 * kv * e + 2 * d * 4) + head * e + rows * d * (e + 4) + rows * 8,
                "flops": 2 * rows * (n * (mats + 2 * q * (L + rows)) + head)}
    if kind == "unembed":
        return {"bytes": head * e + rows * d * 4 + rows * 12, "flops": 2 * rows * head}
    if kind == "prompt":
        # the cache is what the pass leaves: of the last layer it needs K and V only
        n, L0, nl = case["n"], case["L0"], sh.n_layers
        last = d * 2 * kv
        keys = n * L0 + n * (n + 1) // 2
        return {"bytes": ((nl - 1) * mats + last) * e + nl * (L0 + 2 * n) * 2 * kv * e + n * d * e,
                "flops": 2 * n * ((nl - 1) * mats + last) + (nl - 1) * 4 * q * keys}
    slots = sh.vocab * max(1, case["G"])
    cache = 4 * sh.n_layers * 2 * (case["steps"] * max(case["N"], rows if case["mode"] == "jacobi" else 1) + 64) * kv * e
    return {"bytes": slots * 4 + case["P"] * case["N"] * 4 + case["steps"] * 2 * rows * 8 + cache, "flops": 0}


def tolerance(case):
    if case["kind"] == "controller":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["kind"] == "unembed":
        return {"rel": 2e-4, "differ": 0.0}
    return {"rel": 4e-3 if case["dtype"] == "f16" else 2e-2}


# ---- 64 bits ----------------------------------------------------------------------------------------
def _visible(W, N, G, rows):
    """Block row -> the block rows it attends to, and its distance from row 0's position."""
    at, seen = [0] * rows, [{i} for i in range(rows)]
    for r in range(N - 1):
        for c in range(W):
            i = 1 + r * W + c
            at[i] = 1 + c + r
            seen[i] = {0} | {1 + x for x in range(c + 1)} | {1 + y * W + c for y in range(1, r + 1)}
    for k in range(G):
        for j in range(N - 1):
            i = 1 + (W + k) * (N - 1) + j
            at[i] = 1 + j
            seen[i] = {0} | {i - x for x in range(j + 1)}
    mask = torch.zeros((rows, rows), dtype=torch.bool)
    for i, cols in enumerate(seen):
        mask[i, list(cols)] = True
    return torch.tensor(at).cuda(), mask.cuda()


def _norm64(x, g, eps):
    return x * torch.rsqrt(x.square().mean(1, keepdim=True) + eps) * g.double()


def _rope64(x, pos, theta):
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * torch.pow(torch.tensor(float(theta), dtype=torch.float64, device="cuda"),
                                            -torch.arange(half, device="cuda", dtype=torch.float64) / half)
    c, s = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _layers64(sh, seed, x, pos, L, mask):
    """All layers; mask [rows, rows] over the block's own rows.  Returns x and the block's (K, V) of every layer."""
    rows, group, kv_out = x.shape[0], sh.n_q_heads // sh.n_kv_heads, []
    see = torch.cat([torch.ones((rows, L), dtype=torch.bool, device="cuda"), mask], 1)
    for l in range(sh.n_layers):
        w = _layer(sh, seed, l)
        h = _norm64(x, w["g_attn"], sh.rms_eps)
        q = _rope64((h @ w["wq"].double()).view(rows, sh.n_q_heads, sh.head_dim), pos, sh.rope_theta)
        k = _rope64((h @ w["wk"].double()).view(rows, sh.n_kv_heads, sh.head_dim), pos, sh.rope_theta)
        v = (h @ w["wv"].double()).view(rows, sh.n_kv_heads, sh.head_dim)
        kv_out.append((k, v))
        k0, v0 = _kv_rows(sh, seed, l, L)
        ka, va = torch.cat([k0.double(), k]), torch.cat([v0.double(), v])
        o = torch.empty_like(q)
        for hq in range(sh.n_q_heads):
            sc = q[:, hq] @ ka[:, hq // group].t() / math.sqrt(sh.head_dim)
            o[:, hq] = torch.softmax(sc.masked_fill(~see, -math.inf), 1) @ va[:, hq // group]
        x = x + o.reshape(rows, -1) @ w["wo"].double()
        h = _norm64(x, w["g_mlp"], sh.rms_eps)
        x = x + (torch.nn.functional.silu(h @ w["wgate"].double()) * (h @ w["wup"].double())) @ w["wdown"].double()
        del w
    return x, kv_out


def _head64(sh, seed, x, unembed):
    h = _norm64(x, _gain(seed, "g_final", sh.d_model), sh.rms_eps)
    parts = [h @ unembed[:, c:c + 16384].double() for c in range(0, sh.vocab, 16384)]
    top = torch.topk(torch.cat(parts, 1), 2, 1)
    return top.values, top.indices[:, 0].int()


def exact(case, seed):
    sh, kind = _shape(case), case["kind"]
    if kind == "controller":
        return None
    if kind == "unembed":
        u = _unembed(sh, seed)
        top, ids = _head64(sh, seed, _unembed_hidden(case, sh, seed, u).double(), u)
        return {"ids": ids, "top2": top}
    n = case["rows"] if kind == "step" else case["n"]
    x = _embed(sh, seed)[_ints(seed, "tok", n, sh.vocab).long()].double()
    if kind == "step":
        at, mask = _visible(case["W"], case["N"], case["G"], n)
        x, _ = _layers64(sh, seed, x, case["L"] + at, case["L"], mask)
        return {"hidden": x, "top2": _head64(sh, seed, x, _unembed(sh, seed))[0]}
    mask = torch.ones((n, n), dtype=torch.bool, device="cuda").tril()
    pos = case["L0"] + torch.arange(n, device="cuda")
    return [list(kv) for kv in _layers64(sh, seed, x, pos, case["L0"], mask)[1]]
