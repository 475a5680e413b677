"""The feature gather at the row widths where its chunks can go wrong: shorter than a chunk, one byte around a chunk's end,
one chunk per row, rows of more chunks than a workgroup takes, the longest row; unaligned addresses; empty tables."""
import numpy as np
import pytest

from oracle import gsso

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 255, 1433 * 2 + 1, 16384, 16385, 65537, 1 << 20])
@pytest.mark.parametrize("offset", [0, 1])
def test_gather_widths(width, offset):
    import torch
    from paper_2406_17918_amd import gss
    rs = np.random.default_rng(width)
    n, m = (37, 53) if width > 4096 else (1009, 3001)
    host = rs.integers(0, 256, size=(n, width)).astype(np.uint8)
    flat = torch.zeros(n * width + offset, dtype=torch.uint8, device="cuda")
    flat[offset:] = torch.from_numpy(host).reshape(-1).cuda()
    ids = rs.integers(-2, n + 2, size=m).astype(np.int32)
    # the output sits between bytes that must stay as they are
    guard = torch.full((m * width + 128,), 7, dtype=torch.uint8, device="cuda")
    out = guard[64 - offset:64 - offset + m * width].view(m, width)
    gss.gather_rows(flat[offset:].view(n, width), torch.from_numpy(ids).cuda(), out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), gsso.gather_rows(host, ids))
    assert bool((guard[:64 - offset] == 7).all()) and bool((guard[64 - offset + m * width:] == 7).all())


@pytest.mark.parametrize("width", [1, 6, 100])
def test_gather_from_an_empty_table(width):
    import torch
    from paper_2406_17918_amd import gss
    out = torch.full((5, width), 3, dtype=torch.uint8, device="cuda")
    gss.gather_rows(torch.zeros((0, width), dtype=torch.uint8, device="cuda"), torch.arange(-2, 3, dtype=torch.int32, device="cuda"), out)
    assert int(out.sum()) == 0
