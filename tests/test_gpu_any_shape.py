"""fp32 blocks and bf16 blocks whose extents are no multiples of 8, at the sizes where the
any-shape kernel can go wrong: one element around its tiles (32, 64), its stages (32, 64, 128
contracted elements) and the tile rule (128 tiles of 64 x 64), blocks smaller than a tile or a
stage, and views that start at an odd element.  Operands are small integers, so every product and
sum is exact in fp32 and the results must equal the fp64 oracle bit for bit."""
import numpy as np
import pytest
import torch

import paper_2105_14500_amd as tess
from paper_2105_14500_amd import binding as B
from oracle import tess_oracle as orc
from gpu_util import f64, share_desc, tdtype

pytestmark = pytest.mark.gpu


def _panels(q, rows, cols, dtype, gen):
    """q integer panels on the device as views of one matrix whose rows are one element longer and
    which starts at an odd element."""
    host = torch.randint(-2, 3, (q, rows, cols), generator=gen).to(tdtype(dtype))
    room = torch.full((q * rows * (cols + 1) + 1,), float("nan"), dtype=tdtype(dtype), device="cuda:0")
    views = room[1:].view(q, rows, cols + 1)[:, :, :cols]
    views.copy_(host)
    return [f64(h) for h in host], list(views)


SIZES = [(1, 1, 1), (31, 33, 65), (32, 32, 64), (33, 64, 63), (65, 127, 129), (3, 200, 7), (300, 1, 5),
         (63, 65, 257), (45, 127, 33), (45, 129, 33), (127, 45, 129), (705, 33, 769), (704, 257, 768), (769, 700, 65),
         # 64 x 64 tiles of eight wavefronts (fp32 outputs of 192 to 512 tiles), one call each
         (833, 131, 1025), (961, 1025, 66), (70, 961, 897), (1023, 33, 769)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,kb,n", SIZES)
def test_products_are_bit_exact_at_tile_edges(dtype, m, kb, n):
    if dtype == "bf16" and (m % 8 == 0 or kb % 8 == 0 or n % 8 == 0):
        m, kb, n = m + (m % 8 == 0), kb + (kb % 8 == 0), n + (n % 8 == 0)
    q = 2
    gen = torch.Generator().manual_seed(m * 7 + kb * 3 + n)
    desc = share_desc(q, 1, m, kb, n, dtype, "f32")
    assert tess.plan(desc, B.OP_FWD) == (0, 0, 1) and tess.workspace_bytes(desc, B.OP_FWD) == 0
    xs, xd = _panels(q, m, kb, dtype, gen)
    ws, wd = _panels(q, kb, n, dtype, gen)
    dys, dyd = _panels(q, m, n, dtype, gen)
    out = lambda r, c: torch.full((r, c + 3), 9.0, dtype=torch.float32, device="cuda:0")  # noqa: E731
    y, dx, dw = out(m, n), out(m, kb), out(kb, n)
    db = torch.full((n,), 5.0, dtype=torch.float32, device="cuda:0")
    tess.linear_fwd(desc, xd, wd, None, B.ACT_NONE, y[:, :n])
    tess.linear_bwd_dx(desc, dyd, wd, dx[:, :kb])
    tess.linear_bwd_dw_bias(desc, xd, dyd, dw[:, :n], db, accumulate=True)
    assert np.array_equal(f64(y[:, :n]), orc.fwd_panels(xs, ws))
    assert np.array_equal(f64(dx[:, :kb]), orc.bwd_dx_panels(dys, ws))
    assert np.array_equal(f64(dw[:, :n]), orc.bwd_dw_panels(xs, dys) + 9.0)
    assert np.array_equal(f64(db), sum(d.sum(0) for d in dys) + 5.0)
    for t, c in ((y, n), (dx, kb), (dw, n)):      # nothing was written beside the block
        assert (t[:, c:] == 9.0).all()


@pytest.mark.parametrize("dtype,m,kb,n", [("f32", 70, 100, 90), ("bf16", 71, 101, 91), ("f32", 800, 100, 700)])
def test_an_infinity_stays_in_its_row(dtype, m, kb, n):
    """The last stage of a panel reads contracted elements that the stage before had: they count once."""
    q = 2
    x = torch.ones((q, m, kb), dtype=tdtype(dtype))
    w = torch.ones((q, kb, n), dtype=tdtype(dtype))
    x[0, 5, kb - 60] = float("inf")
    w[1, kb - 50, 7] = float("-inf")
    desc = share_desc(q, 1, m, kb, n, dtype, "f32")
    y = torch.empty((m, n), dtype=torch.float32, device="cuda:0")
    tess.linear_fwd(desc, list(x.cuda()), list(w.cuda()), None, B.ACT_NONE, y)
    want = torch.full((m, n), float(q * kb))
    want[5, :] = float("inf")
    want[:, 7] = float("-inf")
    want[5, 7] = float("nan")
    assert torch.equal(torch.nan_to_num(y.cpu(), nan=1e30), torch.nan_to_num(want, nan=1e30))
