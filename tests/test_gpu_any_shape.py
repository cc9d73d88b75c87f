"""fp32 blocks and bf16 blocks whose extents are no multiples of 8, at the sizes where the
any-shape kernel can go wrong: one element around its tiles (32, 64), its stages (32, 64, 128
contracted elements) and the tile rule (bf16: 128 tiles of 64 x 64; fp32: 192 and 512), blocks
smaller than a tile or a stage, and views that start at an odd element.  Operands are small integers, so every product and
sum is exact in fp32 and the results must equal the fp64 oracle bit for bit."""
import numpy as np
import pytest
import torch

import paper_2105_14500_amd as tess
from paper_2105_14500_amd import binding as B
from oracle import tess_oracle as orc
from gpu_util import ACT, ORC_ACT, f64, rel_err, share_desc, tdtype

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
         (833, 131, 1025), (961, 1025, 66), (70, 961, 897), (1023, 33, 769),
         # 64 x 64 tiles of four wavefronts (fp32 outputs of more than 512), one call each: panels shorter
         # than a stage, of several and of a last one that reaches back
         (1500, 31, 1501), (1501, 1500, 40), (77, 1500, 1501), (1537, 97, 1473)]


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


# 32 x 32 tiles; 64 x 64 with eight wavefronts (fp32, 256 tiles), with four (576), and in bf16 (169)
WIDE = [("f32", 1000, 100, 1000), ("f32", 1500, 100, 1500), ("bf16", 801, 101, 801)]


@pytest.mark.parametrize("dtype,m,kb,n", [("f32", 70, 100, 90), ("bf16", 71, 101, 91), ("bf16", 71, 131, 91), ("f32", 800, 100, 700)] + WIDE)
def test_an_infinity_stays_in_its_row(dtype, m, kb, n):
    """The last stage of a panel reads contracted elements that the stage before had: they count once.
    Infinities 20 and 60 elements before the end lie in that overlap for every stage depth that there is."""
    q = 2
    x = torch.ones((q, m, kb), dtype=tdtype(dtype))
    w = torch.ones((q, kb, n), dtype=tdtype(dtype))
    want = torch.full((m, n), float(q * kb))
    rows, cols = [(0, 5, kb - 60), (1, 9, kb - 20), (0, m - 1, kb - 1)], [(1, kb - 50, 7), (0, kb - 15, 11), (1, 3, n - 1)]
    for t, r, k in rows:
        x[t, r, k] = float("inf")
        want[r, :] = float("inf")
    for t, k, c in cols:
        w[t, k, c] = float("-inf")
        want[:, c] = float("-inf")
    for _, r, _ in rows:
        for _, _, c in cols:
            want[r, c] = float("nan")
    desc = share_desc(q, 1, m, kb, n, dtype, "f32")
    y = torch.empty((m, n), dtype=torch.float32, device="cuda:0")
    tess.linear_fwd(desc, list(x.cuda()), list(w.cuda()), None, B.ACT_NONE, y)
    assert torch.equal(torch.nan_to_num(y.cpu(), nan=1e30), torch.nan_to_num(want, nan=1e30))


@pytest.mark.parametrize("dtype,rows,k,cols", [("f32", 70, 100, 90), ("bf16", 71, 101, 91)] + WIDE)
@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("act", ["none", "gelu_erf", "gelu_tanh"])
def test_epilogues(dtype, rows, k, cols, out, act):
    """Bias, pre-activation copy and activation of the forward and the activation's derivative in dX, on
    every kernel variant."""
    q = 2
    gen = torch.Generator().manual_seed(rows + k)
    # bf16 outputs: half an ulp (2^-9) and the tails of the GELU, in which the value itself is tiny;
    # fp32 outputs: sums of some 200 terms in fp32
    tol = 4e-3 if out == "bf16" else 5e-6
    odt = tdtype(out)
    draw = lambda r, c, s: (torch.randn(q, r, c, generator=gen) * s).to(tdtype(dtype))  # noqa: E731
    room = lambda r, c, dt: torch.full((r, c + 3), 9.0, dtype=dt, device="cuda:0")  # noqa: E731
    x, w, bias = draw(rows, k, 1.0), draw(k, cols, 0.1), torch.randn(cols, generator=gen).to(tdtype(dtype))
    y, z = room(rows, cols, odt), room(rows, cols, odt)
    desc = share_desc(q, 1, rows, k, cols, dtype, out)
    tess.linear_fwd(desc, list(x.cuda()), list(w.cuda()), bias.cuda(), ACT[act], y[:, :cols], preact_out=z[:, :cols])
    want_y, want_z = orc.fwd_panels([f64(a) for a in x], [f64(a) for a in w], bias=f64(bias), act=ORC_ACT[act], want_z=True)
    assert rel_err(y[:, :cols], want_y) <= tol and rel_err(z[:, :cols], want_z) <= tol
    # dX [rows, cols] through the activation of the layer below
    dy, w2, zin = draw(rows, k, 1.0), draw(cols, k, 0.1), torch.randn(rows, cols, generator=gen).to(tdtype(dtype))
    dz = room(rows, cols, odt)
    desc = share_desc(q, 1, rows, cols, k, dtype, out)
    tess.linear_bwd_dx_act(desc, list(dy.cuda()), list(w2.cuda()), zin.cuda(), ACT[act], dz[:, :cols])
    want = orc.bwd_dx_panels([f64(a) for a in dy], [f64(a) for a in w2])
    if act != "none":
        zt = torch.from_numpy(f64(zin)).requires_grad_()
        torch.nn.functional.gelu(zt, approximate="tanh" if act == "gelu_tanh" else "none").sum().backward()
        want = want * zt.grad.numpy()
    assert rel_err(dz[:, :cols], want) <= tol
    for t in (y, z, dz):
        assert (t[:, cols:] == 9.0).all()
