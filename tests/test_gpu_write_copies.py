"""vd_write into arrays that begin at any element (the copies of one value per
cell go 16 bytes at a time where the array begins on such a border): the same
values at every place, and nothing written beside them."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

FLAT = ("nbr_off", "facet_off", "vert_off", "vol", "centroid", "flags")


@pytest.mark.parametrize("n", [1, 2, 3, 15, 17, 1001, 70_001, 1_100_003])
def test_any_place(n):
    import torch
    import paper_2605_06408_amd as vd
    x = torch.rand((n, 3), generator=torch.Generator().manual_seed(n)).cuda()
    ctx = vd.Context(0)
    d = ctx.build(x, None, [0.0, 0, 0, 1, 1, 1])
    for fields, shift in [(FLAT, s) for s in (0, 1, 2, 3)] + [(("vol",), 0), (("flags",), 5), (("centroid", "nbr_off"), 0)]:
        bufs, rows = {}, []
        for k in vd.OUTPUT_FIELDS:
            if k not in fields:
                rows.append(None)
                continue
            t = getattr(d, k)
            e, at = t.element_size(), 64 + shift * t.element_size()
            buf = torch.full((at + t.numel() * e + 64,), 0xA5, dtype=torch.uint8, device="cuda")
            assert buf.data_ptr() % 64 == 0
            bufs[k] = (buf, at, t.numel() * e)
            rows.append(buf.data_ptr() + at)
        out = vd.Outputs(*rows)
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert ctx.lib.vd_write(ctx.handle, ctypes.byref(out), stream) == 0
        for k, (buf, at, size) in bufs.items():
            assert torch.equal(buf[at:at + size], getattr(d, k).contiguous().view(-1).view(torch.uint8)), (k, shift)
            assert bool((buf[:at] == 0xA5).all()) and bool((buf[at + size:] == 0xA5).all()), (k, shift)
