"""The plain kernels at the edges of their tiles: contractions and widths that are no multiple of 16 or 4, one to four row
tiles, small and large heads, hidden states that are not 16-byte aligned; against the oracle at the fp32 bar (1e-4 per row,
which the 16-bit storage types meet too: their weights and cache rows are given, the arithmetic is float) plus the rounding of
the block's own K, V rows to the cache type."""
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
    ((2, 250, 5, 5, 10, 101, 333), "f32", 1, 0),
    ((2, 252, 6, 2, 66, 172, 1000), "f32", 17, 300),
    ((1, 130, 4, 1, 256, 90, 777), "f32", 64, 513),
    ((2, 36, 2, 1, 2, 15, 17), "f32", 33, 5),
    ((1, 100, 8, 4, 24, 1030, 16500), "f32", 32, 70),
    ((1, 100, 4, 2, 40, 70, 200), "bf16", 48, 40),
    ((1, 68, 4, 4, 20, 33, 50), "f16", 49, 260),
])
def test_plain_kernels_at_odd_shapes(dims, dtype, rows, L):
    import torch
    from paper_2602_16760_amd import binding as B
    nl, d, hq, hkv, dh, F, V = dims
    shape = synth.ModelShape(f"odd{d}", nl, d, hq, hkv, dh, F, V, 1e-5, 1e4, dtype)
    om = oracle_model(shape, seed=3)
    okv = otf.KVCache(shape, L + rows)
    eng = gpu_engine(shape, L + rows, seed=3)
    try:
        if L:
            prefill_both(shape, eng, okv, L)
        pos, vis = ola.causal_block(L, rows)
        x = synth.hidden_block(shape, rows, 1)
        want = otf.forward_block(om, okv, x, pos, vis)
        p, m = B.to_device(np.asarray(pos, dtype=np.int32)), B.to_device(np.asarray(vis, dtype=np.uint64))
        for shift in (0, 1):  # (one float: the rows are not 16-byte aligned)
            buf = torch.zeros(rows * d + 1, dtype=torch.float32, device="cuda")
            h = buf[shift:shift + rows * d].view(rows, d)
            h.copy_(torch.from_numpy(x))
            B.la_forward_layers(eng.model, 0, nl, h, p, m, eng.kv)
            torch.cuda.synchronize()
            assert row_rel_err(h.cpu().numpy(), want).max() <= TOL[dtype]
            ids = torch.empty(rows, dtype=torch.int32, device="cuda")
            top2 = torch.empty((rows, 2), dtype=torch.float32, device="cuda")
            B.la_unembed_argmax(eng.model, h, ids, top2)
            lg = otf.logits_of(om, h.cpu().numpy().astype(np.float64))
            t1, t2 = otf.top2_margin(lg)
            safe = (t1 - t2) > 1e-4 * np.abs(t1)
            assert np.array_equal(ids.cpu().numpy()[safe], otf.argmax_ids(lg)[safe])
            assert np.abs(top2.cpu().numpy()[:, 0] - t1).max() <= 1e-4 * np.abs(lg).max()
    finally:
        eng.close()
