"""Cache rows in and out: every row range against 32-row blocks, both head sizes, aligned and unaligned buffers; bytes are
the same, rows outside the range stay as they were."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["small_bf16", "small64_f16", "tiny_f32"])
@pytest.mark.parametrize("row0,n", [(0, 1), (0, 32), (31, 2), (5, 27), (32, 64), (33, 95), (63, 1), (1, 126)])
@pytest.mark.parametrize("shift", [0, 1])
def test_cache_rows_come_back_as_written(name, row0, n, shift):
    import torch
    from paper_2602_16760_amd import binding as B
    shape = synth.SHAPES[name].with_layers(2)
    dt = torch.int32 if shape.dtype == "f32" else torch.int16
    model = B.la_init_model(shape)
    kv = B.la_kv_alloc(model, 128)
    size = (shape.n_kv_heads, shape.head_dim)

    def buf(rows):  # (shift: one element off the allocation's alignment)
        flat = torch.zeros(rows * size[0] * size[1] + 1, dtype=dt, device="cuda")
        return flat[shift:shift + rows * size[0] * size[1]].view(rows, *size)

    def rand(rows, seed):
        b = buf(rows)
        b.copy_(torch.from_numpy(np.random.default_rng(seed).integers(-30000, 30000, size=(rows, *size))).to(dt))
        return b

    try:
        want = [rand(128, 1), rand(128, 2)]
        B.la_kv_fill(kv, 1, 0, want[0], want[1])
        new = [rand(n, 3), rand(n, 4)]
        B.la_kv_fill(kv, 1, row0, new[0], new[1])
        got, part, other = [buf(128), buf(128)], [buf(n), buf(n)], [buf(128), buf(128)]
        B.la_kv_read(kv, 1, 0, 128, *got)
        B.la_kv_read(kv, 1, row0, n, *part)
        B.la_kv_read(kv, 0, 0, 128, *other)
        torch.cuda.synchronize()
        for i in range(2):
            want[i][row0:row0 + n] = new[i]
            assert torch.equal(got[i], want[i]) and torch.equal(part[i], new[i]) and not other[i].any()
    finally:
        torch.cuda.synchronize()
        B.la_free_kv(kv)
        B.la_free_model(model)
