"""The grid barrier where workgroups are not on the XCD that they are expected on (LA_FAR_FROM: the last one says so, the upper half, all
of them): every word of the launch is stored for the whole device, and the results are the same bits."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_engine
from oracle import lookahead as ola

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["small_bf16", "small64_bf16", "small_f16"])
@pytest.mark.parametrize("wgs", [256, 37, 5])
def test_far_workgroups(monkeypatch, name, wgs):
    shape, L, most = synth.SHAPES[name].with_layers(2), 70, 64
    monkeypatch.setenv("LA_WGS", str(wgs))

    def run():
        eng = gpu_engine(shape, L + most, seed=3)
        try:
            for l in range(shape.n_layers):
                eng.fill_kv(l, *synth.kv_fill(shape, l, L, 4))
            from paper_2602_16760_amd import binding as B
            B.la_kv_set_len(eng.kv, L)
            out = []
            for rows in (1, 17, 48, most, 31, 32):
                pos, vis = ola.causal_block(L, rows)
                h = eng.forward(synth.hidden_block(shape, rows, 1), pos, vis)
                ids, top2 = eng.unembed_argmax(h)
                out += [h, ids, top2]
            assert B.la_kv_get_len(eng.kv) == L
            return out
        finally:
            eng.close()

    want = run()
    for first in (wgs - 1, wgs // 2, 0):
        monkeypatch.setenv("LA_FAR_FROM", str(first))
        for got, w in zip(run(), want):
            assert np.array_equal(got, w), first
