"""A block that the cache has no room for, which only the device knows (replayed accepts have moved the length): it is skipped as a
whole, the caller's hidden states stay as they are, and the next call says so."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,dtype,first", [
    ((2, 256, 4, 2, 64, 688, 100), "f32", "plain_qkv"),       # five launches a layer
    ((2, 256, 4, 2, 64, 688, 100), "f16", "plain_qkv"),
    ((2, 256, 4, 2, 24, 688, 100), "f32", "gemm_qkv"),        # heads of 24 channels: the general kernels
    ((2, 512, 8, 4, 64, 1024, 112), "bf16", "layer_stack"),   # the matrix-core path
])
@pytest.mark.parametrize("rows", [17, 64])
def test_hidden_states_of_a_skipped_block_stay(dims, dtype, first, rows):
    import torch
    from paper_2602_16760_amd import binding as B
    nl, d, hq, hkv, dh, F, V = dims
    if first != "layer_stack" and dtype != "f32":
        dh, hq, hkv = 48, 4, 2  # (heads that the matrix-core path does not take)
    shape = synth.ModelShape("skip", nl, d, hq, hkv, dh, F, V, 1e-5, 1e4, dtype)
    L0, max_len = 40, 160
    eng = gpu_engine(shape, max_len, seed=6)
    stream = torch.cuda.Stream()
    try:
        x = torch.from_numpy(np.ascontiguousarray(synth.hidden_block(shape, rows, 3), dtype=np.float32)).cuda()
        pos, vis = (B.to_device(a) for a in B.la_causal_layout(L0, rows))
        state, emitted = B.new_state(), torch.zeros(max_len, dtype=torch.int32, device="cuda")
        B.la_jacobi_init(eng.kv, 1, B.to_device(np.zeros(L0 + 1, dtype=np.int32)), 1, state)
        ids = torch.zeros(1, dtype=torch.int32, device="cuda")

        def forward():
            h = x.clone()
            B.la_forward_layers(eng.model, 0, nl, h, pos, vis, eng.kv)
            torch.cuda.synchronize()
            return h

        B.la_profile_enable(True)
        assert not torch.equal(forward(), x)  # (there is room: the scratch buffers hold a block's values)
        assert first in B.la_profile_read()
        B.la_profile_enable(False)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.la_jacobi_accept(eng.kv, 1, ids, state, emitted, max_len)
        for _ in range(max_len - rows - L0):
            graph.replay()
        assert not torch.equal(forward(), x)  # the last length that has room
        graph.replay()
        assert torch.equal(forward(), x)
        with pytest.raises(B.LaError) as e:
            forward()
        assert e.value.code == -3
        B.la_kv_set_len(eng.kv, L0)
        assert not torch.equal(forward(), x)
    finally:
        torch.cuda.synchronize()
        eng.close()
