"""Quantised rows into and from buffers of any alignment: the same codes and
scales as from aligned ones (the ends of a lane group, rows with and without
16-byte loads)."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,size", [(1, 2), (2, 1)])
@pytest.mark.parametrize("d", [1, 3, 4, 27, 64, 65, 128, 130, 300])
def test_quantize_any_alignment(prec, size, d):
    import torch
    import paper_1309_5478_amd as knn
    h = knn.Handle(0)
    n, dq = 77, (d + 127) // 128 * 128
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    x = torch.randn((n * d + 8,), generator=g, device="cuda")
    x[5] = float("inf")
    got = []
    for src in (0, 1, 4):                       # the same rows, 4 bytes and 16 bytes on
        y = torch.empty_like(x)
        y[src:src + n * d] = x[:n * d]
        for off in (0, 1 if size == 1 else 2, 4):
            out = torch.full((n * dq * size + 16,), 7, dtype=torch.uint8, device="cuda")
            scale = torch.zeros(n, device="cuda")
            st = h.lib.knn_quantize(h.h, ctypes.c_void_p(y.data_ptr() + 4 * src), n, d, prec,
                                    ctypes.c_void_p(out.data_ptr() + off), ctypes.c_void_p(scale.data_ptr()), None)
            torch.cuda.synchronize()
            assert st == 0
            assert (out[:off] == 7).all() and (out[off + n * dq * size:] == 7).all()
            got.append((out[off:off + n * dq * size].clone(), scale))
    for o, s in got[1:]:
        assert torch.equal(o, got[0][0]) and torch.equal(s, got[0][1])
