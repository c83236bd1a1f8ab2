"""The embedding gather: every channel of every row, at widths around the 1024 channels a workgroup takes, ids outside
the vocabulary clamped."""
from dataclasses import replace

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("d", [32, 800, 1024, 1056, 4096])
def test_embed_rows_are_the_table_rows(dtype, d):
    import torch
    from paper_2602_16760_amd import binding as B
    td = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    sh = replace(synth.SHAPES["tiny_f32"], dtype=dtype, d_model=d, vocab=97, n_layers=1)
    table = torch.randn((sh.vocab, d), generator=torch.Generator(device="cuda").manual_seed(d), device="cuda").to(td)
    model = B.la_init_model(sh, table)
    try:
        for rows in (1, 17, 64):
            ids = np.arange(rows) * 31 % sh.vocab
            sent = ids.copy()
            sent[0], sent[-1] = -3, sh.vocab + 5 if rows > 1 else -3
            ids[0], ids[-1] = 0, sh.vocab - 1 if rows > 1 else 0
            out = torch.full((rows + 1, d), 7.5, device="cuda")
            B.la_embed(model, B.to_device(sent.astype(np.int32)), out[:rows])
            assert torch.equal(out[:rows], table[torch.as_tensor(ids, device="cuda")].float())
            assert (out[rows] == 7.5).all()
    finally:
        torch.cuda.synchronize()
        B.la_free_model(model)
