"""Expansion to fp16 and to one byte per index where the kernel's split can go wrong: one and several segments per row (few rows are split
until there are 2048 waves: from one unit to a whole row per wave), a last unit of 128, 256 or 384 columns, fewer rows than a workgroup has waves, outputs aligned to one element only.  Bit-exact against the oracle."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("M,N", [(1, 128), (3, 384), (5, 512), (2, 4096), (7, 4224), (3, 8448), (2, 28672), (300, 3712), (700, 2176), (2049, 4224)])
def test_expansion_at_the_edges(M, N, bits):
    import torch
    import paper_2306_07629_amd as sq
    print(f"expand M={M} N={N} bits={bits}", flush=True)
    L = gen.make_layer(M, N, bits, frac=0.0, skew=None, seed=M + N + bits)
    D = sq.DeviceLayer(L)
    for off in (0, 1):
        w = torch.full((M * N + 9,), 0x5A5A, dtype=torch.int16, device="cuda")
        i = torch.full((M * N + 9,), 0xA5, dtype=torch.uint8, device="cuda")
        sq.sqllm_dequantize(M, N, bits, D.qidx, D.lut, w[off:])
        sq.sqllm_unpack_indices(M, N, bits, D.qidx, i[off:])
        torch.cuda.synchronize()
        w, i = w.cpu().numpy(), i.cpu().numpy()
        assert np.array_equal(w[off:off + M * N].view(np.uint16).reshape(M, N), oracle.dequant(M, N, bits, L.qidx, L.lut))
        assert np.array_equal(i[off:off + M * N].reshape(M, N), oracle.unpack(M, N, bits, L.qidx))
        assert (w[:off] == 0x5A5A).all() and (w[off + M * N:] == 0x5A5A).all()
        assert (i[:off] == 0xA5).all() and (i[off + M * N:] == 0xA5).all()
