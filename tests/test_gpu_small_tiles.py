"""The 64 x 64 and 64 x 32 tiles of small outputs: remainders of the tiles, ragged panels, odd and
even numbers of stages, K parts, every epilogue, on the plans of the cost model (which are 64 x 32 for
nearly all of these shapes) and on each tile forced.  Products of small integers are exact in fp32 and
must equal the fp64 oracle bit for bit."""
import contextlib

import numpy as np
import pytest
import torch

import paper_2105_14500_amd as tess
from paper_2105_14500_amd import binding as B
from oracle import tess_oracle as orc
from gpu_util import ACT, ORC_ACT, f64, rel_err, share_desc, workspace

pytestmark = pytest.mark.gpu

SMALL = {(64, 64), (64, 32)}


def _panels(q, rows, cols, gen):
    """q integer panels with eight NaN columns beside them and eight NaN rows below."""
    host = torch.randint(-2, 3, (q, rows, cols), generator=gen).to(torch.bfloat16)
    room = torch.full((q, rows + 8, cols + 8), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    room[:, :rows, :cols] = host.cuda()
    return [f64(h) for h in host], [room[t, :rows, :cols] for t in range(q)]


# (q, m, kb, n): m needs no multiple of 8 for the forward call
SHAPES = [(1, 64, 64, 64), (1, 8, 8, 8), (3, 72, 64, 40), (2, 64, 192, 96), (1, 128, 320, 64), (3, 200, 264, 136),
          (2, 512, 448, 520), (8, 64, 512, 256), (8, 256, 256, 256), (4, 64, 1024, 1032)]


# (tile, K parts, (q, m, kb, n)): whole panels, then ragged ones in every call; with five stages or six
# in the ring: fewer stages than that, one more, and many
FORCED = [(tile, splits, shape) for tile in sorted(SMALL) for splits in (1, 3)
          for shape in [(2, 192, 256, 320), (1, 192, 192, 192), (4, 448, 64, 128), (3, 136, 200, 264), (1, 136, 392, 152), (8, 72, 8, 104)]
          if splits <= shape[0] * min(-(-k // 64) for k in shape[1:])]


@contextlib.contextmanager
def _forced(tile, splits):
    try:
        B.set_plan_override(tile=tile, k_splits=splits)
        yield
    finally:
        B.set_plan_override(0, 0)


@pytest.mark.parametrize("q,m,kb,n", SHAPES)
def test_products_are_bit_exact(q, m, kb, n):
    assert all(B.plan(share_desc(q, 1, m, kb, n, "bf16", "f32"), op)[:2] in SMALL for op in (B.OP_FWD, B.OP_BWD_DX, B.OP_BWD_DW))
    _check_products(q, m, kb, n)


@pytest.mark.parametrize("tile,splits,shape", FORCED)
def test_products_are_bit_exact_on_every_tile(tile, splits, shape):
    with _forced(tile, splits):
        assert all(B.plan(share_desc(shape[0], 1, *shape[1:], "bf16", "f32"), op) == (*tile, splits)
                   for op in (B.OP_FWD, B.OP_BWD_DX, B.OP_BWD_DW))
        _check_products(*shape)


def _check_products(q, m, kb, n):
    gen = torch.Generator().manual_seed(q + m + kb + n)
    desc = share_desc(q, 1, m, kb, n, "bf16", "f32")
    xs, xd = _panels(q, m, kb, gen)
    ws, wd = _panels(q, kb, n, gen)
    dys, dyd = _panels(q, m, n, gen)
    out = lambda r, c: torch.full((r, c), float("nan"), dtype=torch.float32, device="cuda:0")  # noqa: E731
    y, dx, dw = out(m, n), out(m, kb), out(kb, n)
    db = torch.full((n,), float("nan"), device="cuda:0")
    tess.linear_fwd(desc, xd, wd, None, B.ACT_NONE, y, workspace=workspace(desc, B.OP_FWD))
    tess.linear_bwd_dx(desc, dyd, wd, dx, workspace=workspace(desc, B.OP_BWD_DX))
    tess.linear_bwd_dw_bias(desc, xd, dyd, dw, db, workspace=workspace(desc, B.OP_BWD_DW))
    want_dw, want_db = orc.bwd_dw_panels(xs, dys), sum(d.sum(0) for d in dys)
    assert np.array_equal(f64(y), orc.fwd_panels(xs, ws))
    assert np.array_equal(f64(dx), orc.bwd_dx_panels(dys, ws))
    assert np.array_equal(f64(dw), want_dw) and np.array_equal(f64(db), want_db)
    tess.linear_bwd_dw_bias(desc, xd, dyd, dw, db, accumulate=True, workspace=workspace(desc, B.OP_BWD_DW))
    assert np.array_equal(f64(dw), 2 * want_dw) and np.array_equal(f64(db), 2 * want_db)


@pytest.mark.parametrize("m", [1, 17, 63, 65])
def test_forward_of_any_number_of_rows(m):
    q, kb, n = 2, 136, 72
    gen = torch.Generator().manual_seed(m)
    desc = share_desc(q, 1, m, kb, n, "bf16", "f32")
    assert B.plan(desc, B.OP_FWD)[:2] in SMALL
    xs, xd = _panels(q, m, kb, gen)
    ws, wd = _panels(q, kb, n, gen)
    y = torch.full((m + 2, n), 7.0, device="cuda:0")
    tess.linear_fwd(desc, xd, wd, None, B.ACT_NONE, y[:m], workspace=workspace(desc, B.OP_FWD))
    assert np.array_equal(f64(y[:m]), orc.fwd_panels(xs, ws)) and torch.all(y[m:] == 7.0)


# whole and split contractions, bf16 and fp32 outputs, rows that take vector stores and (out_ld odd) ones that do not
@pytest.mark.parametrize("q,m,kb,n", [(2, 136, 128, 200), (8, 256, 256, 256)])
@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("act", ["none", "gelu_erf", "gelu_tanh"])
@pytest.mark.parametrize("pad", [0, 1])
def test_epilogues(q, m, kb, n, out, act, pad):
    _check_epilogues(q, m, kb, n, out, act, pad)


@pytest.mark.parametrize("tile,splits", [(tile, splits) for tile in sorted(SMALL) for splits in (1, 2)])
@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("act", ["none", "gelu_erf", "gelu_tanh"])
@pytest.mark.parametrize("pad", [0, 1])
def test_epilogues_of_every_tile(tile, splits, out, act, pad):
    with _forced(tile, splits):
        _check_epilogues(2, 136, 128, 200, out, act, pad)


def _check_epilogues(q, m, kb, n, out, act, pad):
    gen = torch.Generator().manual_seed(q + pad)
    desc = share_desc(q, 1, m, kb, n, "bf16", out)
    odt = torch.bfloat16 if out == "bf16" else torch.float32
    # bf16 outputs: half an ulp (2^-9) and the tails of the GELU, in which the value itself is tiny;
    # fp32 outputs: sums of at most 2048 terms in fp32
    tol = 4e-3 if out == "bf16" else 5e-6
    draw = lambda r, c, s: (torch.randn(q, r, c, generator=gen) * s).to(torch.bfloat16)  # noqa: E731
    x, w, dy = draw(m, kb, 1.0), draw(kb, n, 0.05), draw(m, n, 1.0)
    bias = torch.randn(n, generator=gen).to(torch.bfloat16)
    room = lambda r, c: torch.full((r, c + pad), float("nan"), dtype=odt, device="cuda:0")[:, :c]  # noqa: E731
    y, z, dz = room(m, n), room(m, n), room(m, kb)
    xd, wd, dyd = list(x.cuda()), list(w.cuda()), list(dy.cuda())
    tess.linear_fwd(desc, xd, wd, bias.cuda(), ACT[act], y, preact_out=z, workspace=workspace(desc, B.OP_FWD))
    want_y, want_z = orc.fwd_panels([f64(a) for a in x], [f64(a) for a in w], bias=f64(bias), act=ORC_ACT[act], want_z=True)
    assert rel_err(y, want_y) <= tol and rel_err(z, want_z) <= tol
    # dX through the activation of a layer whose pre-activation is [m, kb]
    zin = torch.randn(m, kb, generator=gen).to(torch.bfloat16)
    tess.linear_bwd_dx_act(desc, dyd, wd, zin.cuda(), ACT[act], dz, workspace=workspace(desc, B.OP_BWD_DX))
    dx = orc.bwd_dx_panels([f64(a) for a in dy], [f64(a) for a in w])
    zt = torch.from_numpy(f64(zin)).requires_grad_()
    if act != "none":
        torch.nn.functional.gelu(zt, approximate="tanh" if act == "gelu_tanh" else "none").sum().backward()
        dx = dx * zt.grad.numpy()
    assert rel_err(dz, dx) <= tol
