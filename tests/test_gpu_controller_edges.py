"""The controller where its wave-wide steps can go wrong: window columns that share a key, full and empty keys, keys seeded
from more than one stretch of the prompt, the widest pools, prompts shorter than an n-gram.  Every state word against the
oracle's controller, whole numbers throughout."""
import numpy as np
import pytest

import synth
from gpu_util import assert_state_equal, gpu_engine
from oracle import lookahead as ola

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,N,G,Bp,V,P", [
    (5, 4, 5, 32, 3, 600),      # three keys: columns share keys in every step, all keys full
    (7, 4, 7, 43, 1, 300),      # one token throughout: one tuple, seen 297 times
    (7, 4, 7, 64, 40, 1500),    # keys spread over several stretches of 256 positions
    (31, 2, 32, 64, 12, 257),   # 32 slots per key: two columns at a time
    (1, 2, 62, 64, 90, 2000),   # 62 slots: one column at a time
    (10, 7, 0, 64, 5, 50),      # no pool
    (0, 3, 4, 16, 6, 70),       # no window
    (9, 8, 0, 64, 5, 4),        # prompt shorter than an n-gram
    (3, 4, 2, 16, 2, 5),
    (2, 2, 3, 8, 4, 1),
])
def test_controller_edges(W, N, G, Bp, V, P):
    import torch
    from paper_2602_16760_amd import binding as B
    eng = gpu_engine(synth.SHAPES["small64_bf16"], P + 400, head=False)
    rng = np.random.default_rng(W * 1000 + N * 100 + G)
    prompt = rng.integers(0, V, size=P).astype(np.int32)
    pool = B.la_pool_alloc(eng.shape.vocab, N, G)
    try:
        state = B.new_state()
        total = 60
        emitted = torch.zeros(total, dtype=torch.int32, device="cuda")
        B.la_state_init(pool, eng.kv, W, N, G, B.to_device(prompt), Bp, True, state)
        ost = ola.LookaheadState(prompt, W, N, G, Bp)
        torch.cuda.synchronize()
        assert_state_equal(B.read_state(state), ost, W, N, G, Bp)
        step = 0
        while len(ost.emitted) < total:
            ids = rng.integers(0, V, size=Bp).astype(np.int32)
            if step % 2 and ost.cands:  # confirm one of the candidates
                k = int(rng.integers(0, len(ost.cands)))
                ids[0] = ost.cands[k][0]
                for j in range(1, N - 1):
                    ids[ola.v_row(W, N, G, k, j)] = ost.cands[k][j]
            B.la_ngram_accept(pool, eng.kv, W, N, G, B.to_device(ids), state, emitted, total)
            ost.step(ids, total - len(ost.emitted))
            torch.cuda.synchronize()
            st = B.read_state(state)
            assert_state_equal(st, ost, W, N, G, Bp)
            assert list(emitted.cpu().numpy()[:st.n_emitted]) == ost.emitted
            step += 1
    finally:
        torch.cuda.synchronize()
        B.la_free_pool(pool)
        eng.close()
