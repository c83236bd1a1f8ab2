"""Cache rows of an accepted candidate (moved by the accept's launch, 1024 elements of a row at a time): rows of less than a turn's
elements, of a turn, of several and a remainder, plain and key-blocked caches.  The bytes that were there, whole."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,dh,dtype", [
    (5, 5, 10, "f32"),       # 50 elements a row
    (8, 8, 128, "bf16"),     # 1024
    (20, 20, 64, "f16"),     # 1280
    (29, 29, 40, "f32"),     # 1160
    (17, 17, 128, "bf16"),   # 2176
])
def test_accepted_rows_move_whole(hq, hkv, dh, dtype):
    import torch
    from paper_2602_16760_amd import binding as B
    W, N, G, Bp, period = 2, 5, 3, 24, 7
    shape = synth.ModelShape(f"rows{hkv * dh}", 2, 64, hq, hkv, dh, 64, 64, 1e-5, 1e4, dtype)
    prompt = (np.arange(60) % period).astype(np.int32)
    L0 = len(prompt) - 1
    eng = gpu_engine(shape, 128, head=False)
    pool = B.la_pool_alloc(shape.vocab, N, G)
    try:
        t = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
        rows = [[torch.randn((128, hkv, dh), device="cuda").to(t) for _ in "kv"] for _ in range(2)]
        for l, (k, v) in enumerate(rows):
            B.la_kv_fill(eng.kv, l, 0, k, v)
        state = B.new_state()
        B.la_state_init(pool, eng.kv, W, N, G, B.to_device(prompt), Bp, True, state)
        ids = np.zeros(Bp, dtype=np.int32)
        follow = [(int(prompt[-1]) + 1 + j) % period for j in range(N)]  # the text goes on: candidate 0 is its next tokens
        ids[0] = follow[0]
        first = 1 + W * (N - 1)
        ids[first:first + N - 1] = follow[1:]
        emitted = torch.zeros(16, dtype=torch.int32, device="cuda")
        B.la_ngram_accept(pool, eng.kv, W, N, G, B.to_device(ids), state, emitted, 16)
        torch.cuda.synchronize()
        assert emitted.cpu().numpy()[:N].tolist() == follow
        for l, (k, v) in enumerate(rows):
            want = [x.clone() for x in (k, v)]
            for x in want:
                x[L0 + 1:L0 + N] = x[L0 + first:L0 + first + N - 1].clone()
            got = [torch.zeros_like(x) for x in want]
            B.la_kv_read(eng.kv, l, 0, 128, *got)
            torch.cuda.synchronize()
            for g, x in zip(got, want):
                assert torch.equal(g, x)
    finally:
        torch.cuda.synchronize()
        B.la_free_pool(pool)
        eng.close()
