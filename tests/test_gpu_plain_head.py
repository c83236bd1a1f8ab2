"""The plain kernels' first layer of a call (it makes the rotation table that the others read), their unembedding and arg-max, and keys behind the
length, at the edges of their tiles and turns."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_engine, prefill_both
from oracle import lookahead as ola
from oracle import transformer as otf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("d,heads,dh", [(256, 4, 64), (320, 3, 48)])  # two slices of a wave, six
def test_any_layer_can_be_the_first_of_a_call(rows, d, heads, dh):
    from paper_2602_16760_amd import binding as B
    shape = synth.ModelShape(f"first{d}", 3, d, heads, 1, dh, 200, 64, 1e-5, 1e4, "f32")
    eng = gpu_engine(shape, 100 + rows, seed=7)
    try:
        prefill_both(shape, eng, otf.KVCache(shape, 100 + rows), 100)
        pos, vis = ola.causal_block(100, rows)
        x = synth.hidden_block(shape, rows, 5)
        want = eng.forward(x, pos, vis)
        pos, vis = (B.to_device(np.asarray(a, dtype=t)) for a, t in ((pos, np.int32), (vis, np.uint64)))
        h = B.to_device(np.asarray(x, dtype=np.float32))
        for l in range(3):
            B.la_forward_layers(eng.model, l, l + 1, h, pos, vis, eng.kv)
        assert np.array_equal(h.cpu().numpy(), want)
    finally:
        eng.close()


def test_keys_behind_the_length_may_hold_anything():
    import torch
    from paper_2602_16760_amd import binding as B
    shape, got = synth.SHAPES["tiny_f32"], {}
    for L in (1, 47, 64, 130):
        for bad in (0.0, float("nan")):
            eng = gpu_engine(shape, 700, seed=4)
            try:
                prefill_both(shape, eng, otf.KVCache(shape, 700), L)
                rest = torch.full((700 - L, shape.n_kv_heads, shape.head_dim), bad, device="cuda")
                for l in range(shape.n_layers):
                    B.la_kv_fill(eng.kv, l, L, rest, rest)
                got[bad == 0.0] = eng.forward(synth.hidden_block(shape, 9, 2), *ola.causal_block(L, 9))
            finally:
                eng.close()
        assert np.isfinite(got[True]).all() and np.array_equal(got[True], got[False])


# columns around a tile of 16, a turn of 2048 and the last that a rule takes before the general product does (two rounds of 256 workgroups for contractions
# of at most 256, one for others, 2^24 weights)
@pytest.mark.parametrize("d,V", [(256, 1), (256, 15), (256, 17), (60, 257), (256, 2047), (257, 2049), (256, 4112), (257, 4096), (257, 4097), (256, 8192), (256, 8193), (4096, 4096)])
def test_unembedding_and_arg_max(d, V):
    """Logits are sums of d products of order 0.02, 1 and 1: bound d eps times the largest partial sum, 2^-24 * 16 d; ids where the margin is clear of
    it, and ties to the lowest index."""
    import torch
    from paper_2602_16760_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(d * 10007 + V)
    u = torch.randn(d, V, generator=g, device="cuda") * 0.02
    if V > 2:
        u[:, V - 1] = u[:, V // 2]  # a tie
    gain = torch.rand(d, generator=g, device="cuda") + 0.5
    shape = synth.ModelShape("head", 1, d, 1, 1, 16, 16, V, 1e-5, 1e4, "f32")
    model = B.la_init_model(shape, None, gain, u)
    try:
        for rows in (1, 16, 17, 33, 64):
            h = torch.randn(rows, d, generator=g, device="cuda")
            if V > 2:
                h[0] = u[:, V // 2] * 50.0  # row 0 chooses the tied column
            ids, top2 = torch.zeros(rows, dtype=torch.int32, device="cuda"), torch.zeros(rows, 2, device="cuda")
            B.la_unembed_argmax(model, h, ids, top2)
            x = h.double()
            logits = (x * torch.rsqrt(x.square().mean(1, keepdim=True) + 1e-5) * gain.double()) @ u.double()
            top = torch.topk(logits, min(2, V), 1).values
            bar = 2.0 ** -24 * 16 * d
            assert (top2[:, :top.shape[1]].double() - top).abs().max() <= bar
            if V == 1:
                assert torch.isneginf(top2[:, 1]).all() and (ids == 0).all()
                continue
            clear = top[:, 0] - top[:, 1] > 2 * bar
            assert torch.equal(ids.long()[clear], logits.argmax(1)[clear])
            if V > 2:
                assert ids[0] == V // 2 and top2[0, 0] == top2[0, 1]
    finally:
        torch.cuda.synchronize()
        B.la_free_model(model)


@pytest.mark.parametrize("d,V", [(60, 8192), (255, 8192), (256, 8192), (257, 4096), (1000, 4096), (1002, 4096), (4096, 4096)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [0, 1])
def test_the_small_product_and_the_general_one_sum_alike(d, V, dtype, shift, monkeypatch):
    """The last size of either rule, and one column of zeros more: the same bits, since that column wins nowhere.  Hidden states on any word."""
    import torch
    from paper_2602_16760_amd import binding as B
    monkeypatch.setenv("LA_FORCE_GENERIC", "1")
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(d + V)
    u = (torch.randn(d, V, generator=g, device="cuda") * 0.02).to(t)
    gain = torch.rand(d, generator=g, device="cuda") + 0.5
    hidden = [torch.randn(rows * d + shift, generator=g, device="cuda")[shift:].view(rows, d) for rows in (1, 17, 64)]
    got = []
    for columns in (V, V + 1):
        shape = synth.ModelShape("head", 1, d, 1, 1, 16, 16, columns, 1e-5, 1e4, dtype)
        model = B.la_init_model(shape, None, gain, torch.cat([u, torch.zeros(d, columns - V, dtype=t, device="cuda")], 1).contiguous())
        try:
            for h in hidden:
                ids, top2 = torch.zeros(len(h), dtype=torch.int32, device="cuda"), torch.zeros(len(h), 2, device="cuda")
                B.la_unembed_argmax(model, h, ids, top2)
                got.append((ids, top2))
        finally:
            torch.cuda.synchronize()
            B.la_free_model(model)
    for (a, x), (b, y) in zip(got[:3], got[3:]):
        assert (x > 0).all() and torch.equal(a, b) and torch.equal(x, y)
