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
    (31, 2, 32, 64, 12, 257),   # 32 slots per key: two keys at a time
    (1, 2, 62, 64, 90, 2000),   # 62 slots: one key at a time
    (31, 2, 32, 64, 2, 100),    # all columns on one or two keys of many slots
    (15, 2, 15, 31, 40, 900),   # full keys, some shared: the oldest slot is looked for
    (8, 5, 7, 61, 3, 200),      # most words of tuples at hand
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


def test_generations_on_two_streams_share_a_pool_without_slots():
    """G = 0: nothing is kept in the pool, so generations on different streams may share one.  It is made while the default
    stream is busy: what the accept kernels count with has to be ready on their own streams all the same."""
    import torch
    from paper_2602_16760_amd import binding as B
    W, N, G, Bp, V, steps = 10, 7, 0, 64, 5, 24
    engs = [gpu_engine(synth.SHAPES["small64_bf16"], 200, head=False) for _ in range(2)]
    rng = np.random.default_rng(3)
    prompts = [rng.integers(0, V, size=50).astype(np.int32) for _ in engs]
    ids = [rng.integers(0, V, size=(steps, Bp)).astype(np.int32) for _ in engs]
    dev = [(B.to_device(p), B.to_device(i)) for p, i in zip(prompts, ids)]
    states, emitted = [B.new_state() for _ in engs], [torch.zeros(steps, dtype=torch.int32, device="cuda") for _ in engs]
    streams = [torch.cuda.Stream() for _ in engs]
    torch.cuda.synchronize()
    torch.cuda._sleep(50_000_000)
    pool = B.la_pool_alloc(engs[0].shape.vocab, N, G)
    try:
        for k, s in enumerate(streams):
            B.la_state_init(pool, engs[k].kv, W, N, G, dev[k][0], Bp, True, states[k], stream=s)
        for i in range(steps):
            for k, s in enumerate(streams):
                B.la_ngram_accept(pool, engs[k].kv, W, N, G, dev[k][1][i], states[k], emitted[k], steps, stream=s)
        torch.cuda.synchronize()
        for k in range(2):
            ost = ola.LookaheadState(prompts[k], W, N, G, Bp)
            for i in range(steps):
                ost.step(ids[k][i], steps - len(ost.emitted))
            assert_state_equal(B.read_state(states[k]), ost, W, N, G, Bp)
            assert B.read_state(states[k]).reserved == 0
            assert list(emitted[k].cpu().numpy()) == ost.emitted
    finally:
        torch.cuda.synchronize()
        B.la_free_pool(pool)
        for e in engs:
            e.close()
