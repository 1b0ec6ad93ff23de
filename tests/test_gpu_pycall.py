"""Single-layer calls from Python take the native path, on the stream they are given and on the current one."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", ["given", "current"])                   # what the first call of the process says about its stream
def test_native_path_and_its_streams(first):
    import torch
    import paper_2306_07629_amd as sq
    from paper_2306_07629_amd import binding
    L = gen.make_layer(40, 1024, 3, frac=0.0045, skew=(0.1, 0.5), seed=11)
    ref, absdot = oracle.layer_matvec(L)
    D = sq.DeviceLayer(L)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    binding._matvec = binding._matvec_first
    for stream in (side, None) if first == "given" else (None, side):
        D.y.zero_()
        torch.cuda.synchronize()
        D.matvec(stream)
        (side if stream is not None else torch.cuda.current_stream()).synchronize()
        y = D.y.cpu().numpy().view(np.float16).astype(np.float64)
        assert (np.abs(y - ref) <= 2e-3 * absdot + 2.0 ** -25).all()
        from paper_2306_07629_amd import _pycall
        assert binding._matvec is _pycall.matvec
    with torch.cuda.stream(side):                                         # the current stream is asked for at every call
        D.y.zero_()
        D.matvec()
    side.synchronize()
    assert (np.abs(D.y.cpu().numpy().view(np.float16).astype(np.float64) - ref) <= 2e-3 * absdot + 2.0 ** -25).all()
