"""The launches of small plain layers (fp32 arithmetic, five a layer) at their edges: contractions around 256 and 768 (two and six
slices of a wave, and several turns), widths that are no multiple of 8 or 16, heads of 16 to 256 channels, contexts around 64 and
512 keys; and what a row does not see need not be finite.  Against the oracle at the bars of the plain kernels' test: 1e-4 per row
in fp32, for 16-bit storage plus the rounding of the block's own K, V rows to the cache type."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_engine, oracle_model, prefill_both, row_rel_err
from oracle import lookahead as ola
from oracle import transformer as otf

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2, "f16": 2e-3}


@pytest.mark.parametrize("dims,dtype,rows,L", [
    # layers, d, q heads, kv heads, head_dim, F, vocab
    ((2, 256, 4, 2, 64, 768, 100), "f32", 16, 48),
    ((2, 257, 3, 1, 16, 769, 100), "f32", 17, 47),
    ((1, 255, 4, 4, 48, 13, 100), "f32", 33, 511),
    ((1, 772, 2, 1, 96, 1601, 100), "f32", 64, 449),
    ((2, 60, 8, 2, 128, 100, 100), "f32", 1, 512),
    ((1, 44, 2, 2, 256, 24, 100), "f32", 49, 1100),
    ((1, 100, 4, 2, 32, 70, 200), "bf16", 48, 0),
    ((1, 68, 4, 4, 80, 33, 50), "f16", 5, 600),
    ((1, 1536, 6, 2, 128, 4096, 50), "f32", 17, 100),   # larger layers: this attention beside the general products
])
def test_small_plain_layers(dims, dtype, rows, L):
    from paper_2602_16760_amd import binding as B
    nl, d, hq, hkv, dh, F, V = dims
    shape = synth.ModelShape(f"plain{d}", nl, d, hq, hkv, dh, F, V, 1e-5, 1e4, dtype)
    om = oracle_model(shape, seed=3)
    okv = otf.KVCache(shape, L + rows)
    eng = gpu_engine(shape, L + rows, seed=3)
    try:
        if L:
            prefill_both(shape, eng, okv, L)
        pos, vis = ola.causal_block(L, rows)
        x = synth.hidden_block(shape, rows, 1)
        want = otf.forward_block(om, okv, x, pos, vis)
        B.la_profile_enable(True)
        got = eng.forward(x, pos, vis)
        ran = B.la_profile_read()
        B.la_profile_enable(False)
        assert "plain_attention" in ran and ("plain_qkv" in ran) == (d < 1536)
        assert row_rel_err(got, want).max() <= TOL[dtype]
        again = eng.forward(x, pos, vis)
        assert np.array_equal(got, again)
    finally:
        eng.close()


def test_rows_that_are_not_seen_may_hold_anything():
    """One row of the block is infinite: the rows that do not see it give what they give without it."""
    shape = synth.SHAPES["tiny_f32"]
    eng = gpu_engine(shape, 128, seed=4)
    try:
        x = synth.hidden_block(shape, 6, 2)
        pos, vis = ola.causal_block(0, 6)
        vis = [int(v) for v in vis]
        vis[3] &= ~(1 << 2)  # rows 3 and 4 see neither row 2 nor a row that does
        vis[4] &= ~(1 << 2)
        want = eng.forward(x, pos, vis)
        bad = x.copy()
        bad[2] = np.inf
        got = eng.forward(bad, pos, vis)
        keep = [0, 1, 3, 4]
        assert np.isfinite(want[keep]).all()
        assert np.array_equal(got[keep], want[keep])
    finally:
        eng.close()


def test_lengths_that_replayed_accepts_reach():
    """A captured forward and accept, replayed until the cache holds more pieces of 64 keys than it did when it was captured, and
    behind that an eager forward, whose host knows nothing of the replays: a captured launch sums as one that knows the length, bit
    for bit, and so does the eager one (test_sums_depend_on_the_length_alone; held to the plain kernels' bar here)."""
    import torch
    from paper_2602_16760_amd import binding as B
    shape, L0, rows = synth.SHAPES["tiny_f32"], 40, 16
    eng = gpu_engine(shape, 400, seed=5)
    okv = otf.KVCache(shape, 400)
    stream = torch.cuda.Stream()
    try:
        prefill_both(shape, eng, okv, 300)
        x = torch.from_numpy(np.ascontiguousarray(synth.hidden_block(shape, rows, 3), dtype=np.float32)).cuda()
        pos, vis = (B.to_device(a) for a in B.la_causal_layout(L0, rows))
        state, emitted, h = B.new_state(), torch.zeros(300, dtype=torch.int32, device="cuda"), x.clone()
        B.la_jacobi_init(eng.kv, 1, B.to_device(np.zeros(L0 + 1, dtype=np.int32)), 1, state)
        ids = torch.zeros(1, dtype=torch.int32, device="cuda")

        def forward():
            h.copy_(x)
            B.la_forward_layers(eng.model, 0, shape.n_layers, h, pos, vis, eng.kv)

        forward()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            forward()
            B.la_jacobi_accept(eng.kv, 1, ids, state, emitted, 300)
        for n in (1, 30, 60, 150):
            for _ in range(n):
                graph.replay()
            got = h.clone()
            forward()  # (at the length behind the last accept)
            stale = h.clone()
            L = int(B.la_kv_get_len(eng.kv))
            forward()
            assert row_rel_err(stale.cpu().numpy(), h.cpu().numpy()).max() <= TOL["f32"]
            B.la_kv_set_len(eng.kv, L - 1)
            forward()
            assert torch.equal(got, h), L
            B.la_kv_set_len(eng.kv, L)
            torch.cuda.synchronize()
        assert L == L0 + 241
    finally:
        torch.cuda.synchronize()
        eng.close()


@pytest.mark.parametrize("dims,dtype", [
    ((2, 256, 4, 2, 64, 688, 100), "f32"),
    ((1, 1536, 6, 2, 128, 4096, 50), "bf16"),  # (this attention beside the general products)
])
def test_sums_depend_on_the_length_alone(dims, dtype):
    """What the host knows of the length decides how many waves a workgroup of the attention has, not what a row becomes: the same
    bits behind replayed accepts, which the host knows nothing of, and once it has asked for the length."""
    import torch
    from paper_2602_16760_amd import binding as B
    nl, d, hq, hkv, dh, F, V = dims
    shape, L0, rows = synth.ModelShape(f"bound{d}", nl, d, hq, hkv, dh, F, V, 1e-5, 1e4, dtype), 40, 16
    eng = gpu_engine(shape, 700, seed=5)
    try:
        for l in range(nl):
            eng.fill_kv(l, *synth.kv_fill(shape, l, 640, 4))
        x = torch.from_numpy(np.ascontiguousarray(synth.hidden_block(shape, rows, 3), dtype=np.float32)).cuda()
        pos, vis = (B.to_device(a) for a in B.la_causal_layout(L0, rows))
        state, emitted = B.new_state(), torch.zeros(700, dtype=torch.int32, device="cuda")
        B.la_jacobi_init(eng.kv, 1, B.to_device(np.zeros(L0 + 1, dtype=np.int32)), 1, state)
        ids = torch.zeros(1, dtype=torch.int32, device="cuda")

        def forward():
            h = x.clone()
            B.la_profile_enable(True)
            B.la_forward_layers(eng.model, 0, nl, h, pos, vis, eng.kv)
            torch.cuda.synchronize()
            B.la_profile_enable(False)
            assert "plain_attention" in B.la_profile_read()
            return h

        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            B.la_jacobi_accept(eng.kv, 1, ids, state, emitted, 700)
        for n in (60, 100, 250, 180):  # 2, 4, 8 pieces of 64 keys and a part, 10 and a part
            for _ in range(n):
                graph.replay()
            torch.cuda.synchronize()
            behind = forward()
            L = int(B.la_kv_get_len(eng.kv))
            assert torch.equal(behind, forward()), L
        assert L == L0 + 590
    finally:
        torch.cuda.synchronize()
        eng.close()


@pytest.mark.parametrize("dims,dtype,small", [
    # layers, d, q heads, kv heads, head_dim, F, vocab
    ((1, 512, 8, 4, 48, 2048, 50), "bf16", True),     # 256 workgroups for gate and up
    ((1, 264, 4, 2, 48, 2056, 50), "f16", False),     # 257
    ((1, 768, 12, 6, 80, 2064, 50), "bf16", False),   # 258
    ((1, 256, 4, 2, 48, 4096, 50), "bf16", True),     # 512, of the kernel with two slices
    ((1, 256, 4, 2, 48, 4100, 50), "f32", False),     # 513
    ((1, 272, 172, 43, 16, 64, 50), "f32", False),    # 258 for QKV
    ((1, 1536, 8, 8, 64, 2048, 50), "f32", True),     # 12.6 M weights
    ((1, 1792, 20, 10, 64, 2048, 50), "f32", False),  # 17.9 M
])
def test_layers_of_one_round_take_the_small_products(dims, dtype, small):
    """Both sides of the rule's lines, for either size of element; against the oracle at the bars above."""
    from paper_2602_16760_amd import binding as B
    nl, d, hq, hkv, dh, F, V = dims
    shape, L, rows = synth.ModelShape(f"round{d}", nl, d, hq, hkv, dh, F, V, 1e-5, 1e4, dtype), 47, 17
    om, okv = oracle_model(shape, seed=3), otf.KVCache(shape, L + rows)
    eng = gpu_engine(shape, L + rows, seed=3)
    try:
        prefill_both(shape, eng, okv, L)
        pos, vis = ola.causal_block(L, rows)
        x = synth.hidden_block(shape, rows, 1)
        want = otf.forward_block(om, okv, x, pos, vis)
        B.la_profile_enable(True)
        got = eng.forward(x, pos, vis)
        ran = B.la_profile_read()
        B.la_profile_enable(False)
        assert ("plain_qkv" in ran) == small and ("gemm_qkv" in ran) != small
        assert row_rel_err(got, want).max() <= TOL[dtype]
    finally:
        eng.close()


@pytest.mark.parametrize("dims,dtype,attention", [
    ((1, 256, 4, 2, 64, 688, 50), "f32", "plain_attention"),
    ((1, 512, 16, 4, 48, 2064, 50), "bf16", "plain_attention"),  # general products
    ((1, 512, 16, 4, 128, 6000, 50), "f32", "attention"),        # 32 workgroups a row
    ((1, 512, 17, 17, 64, 6000, 50), "f32", "attention"),
])
def test_a_row_does_not_depend_on_the_block_it_is_in(dims, dtype, attention):
    """The first rows of a causal block, in blocks of every height: the same bits, from the same kernels."""
    from paper_2602_16760_amd import binding as B
    nl, d, hq, hkv, dh, F, V = dims
    shape, L, most = synth.ModelShape(f"rows{d}", nl, d, hq, hkv, dh, F, V, 1e-5, 1e4, dtype), 300, 64
    eng = gpu_engine(shape, L + most, seed=3)
    try:
        eng.fill_kv(0, *synth.kv_fill(shape, 0, L, 4))
        B.la_kv_set_len(eng.kv, L)
        pos, vis = ola.causal_block(L, most)
        x, last = synth.hidden_block(shape, most, 1), None
        for rows in (most, 49, 33, 32, 17, 16, 1):
            B.la_profile_enable(True)
            got = eng.forward(x[:rows], pos[:rows], vis[:rows])
            ran = B.la_profile_read()
            B.la_profile_enable(False)
            assert last is None or np.array_equal(got, last[:rows]), rows
            assert attention in ran
            last = got
    finally:
        eng.close()


@pytest.mark.parametrize("dims,dtype", [((1, 256, 4, 2, 64, 688, 50), "f32"), ((1, 256, 4, 2, 48, 688, 50), "bf16"), ((1, 256, 2, 1, 144, 688, 50), "f16")])
def test_a_captured_block_waits_for_the_length_and_an_eager_one_does_not(dims, dtype):
    """The attention has a kernel for either: the same bits at lengths around one piece of 64 keys, all waves' first pieces, and second ones."""
    import torch
    from paper_2602_16760_amd import binding as B
    nl, d, hq, hkv, dh, F, V = dims
    shape, rows, most = synth.ModelShape(f"early{dh}", nl, d, hq, hkv, dh, F, V, 1e-5, 1e4, dtype), 17, 1100
    eng = gpu_engine(shape, most, seed=3)
    try:
        eng.fill_kv(0, *synth.kv_fill(shape, 0, most, 4))
        B.la_kv_set_len(eng.kv, 0)
        pos, vis = (B.to_device(a) for a in B.la_causal_layout(0, rows))
        x = torch.from_numpy(np.ascontiguousarray(synth.hidden_block(shape, rows, 1), dtype=np.float32)).cuda()
        h, stream, graph = x.clone(), torch.cuda.Stream(), torch.cuda.CUDAGraph()
        B.la_forward_layers(eng.model, 0, 1, h, pos, vis, eng.kv)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            h.copy_(x)
            B.la_forward_layers(eng.model, 0, 1, h, pos, vis, eng.kv)
        for L in (0, 46, 47, 48, 111, 112, 495, 496, 511, 512, 1000, 1083):
            B.la_kv_set_len(eng.kv, L)
            eager = x.clone()
            B.la_forward_layers(eng.model, 0, 1, eager, pos, vis, eng.kv)
            graph.replay()
            assert torch.isfinite(eager).all() and torch.equal(h, eager), L
    finally:
        torch.cuda.synchronize()
        eng.close()
