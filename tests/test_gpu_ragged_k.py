"""bf16 panels whose contraction is a multiple of 8 but not of 64: the last stage of every panel
reaches past the panel's end, and what lies there (other columns of the parent matrix, here NaN)
must read as zero.  Both tile sizes, whole and split contractions, small integers: bit exact."""
import numpy as np
import pytest
import torch

import paper_2105_14500_amd as tess
from paper_2105_14500_amd import binding as B
from oracle import tess_oracle as orc
from gpu_util import f64, share_desc, workspace

pytestmark = pytest.mark.gpu


def _panels(q, rows, cols, gen):
    """q integer panels with eight NaN columns beside them and eight NaN rows below."""
    host = torch.randint(-2, 3, (q, rows, cols), generator=gen).to(torch.bfloat16)
    room = torch.full((q, rows + 8, cols + 8), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    room[:, :rows, :cols] = host.cuda()
    return [f64(h) for h in host], [room[t, :rows, :cols] for t in range(q)]


Q = 3
TILES = [(128, 1), (128, 3), (256, 1), (256, 2)]
SHAPES = [(264, 328, 456), (312, 264, 376), (520, 1016, 264)]
# outputs of more than 256 workgroups: rows, columns, K parts, contraction of a panel, panels
MANY = [(2056, 2104, 1, 8, 1), (2056, 2104, 1, 72, 2), (2056, 2104, 1, 200, 3), (1544, 1672, 2, 72, 2), (1544, 1672, 2, 200, 3)]


@pytest.mark.parametrize("tile,splits", TILES)
@pytest.mark.parametrize("m,kb,n", SHAPES)
def test_stages_past_the_panel_end_read_as_zero(tile, splits, m, kb, n):
    q = Q
    gen = torch.Generator().manual_seed(tile + splits + m)
    desc = share_desc(q, 1, m, kb, n, "bf16", "f32")
    xs, xd = _panels(q, m, kb, gen)
    ws, wd = _panels(q, kb, n, gen)
    dys, dyd = _panels(q, m, n, gen)
    out = lambda r, c: torch.full((r, c), float("nan"), dtype=torch.float32, device="cuda:0")  # noqa: E731
    y, dx, dw, db = out(m, n), out(m, kb), out(kb, n), torch.empty((n,), dtype=torch.float32, device="cuda:0")
    try:
        B.set_plan_override(tile=tile, k_splits=splits)
        for op in (B.OP_FWD, B.OP_BWD_DX, B.OP_BWD_DW):
            assert tess.plan(desc, op) == (tile, tile, splits)
        tess.linear_fwd(desc, xd, wd, None, B.ACT_NONE, y, workspace=workspace(desc, B.OP_FWD))
        tess.linear_bwd_dx(desc, dyd, wd, dx, workspace=workspace(desc, B.OP_BWD_DX))
        tess.linear_bwd_dw_bias(desc, xd, dyd, dw, db, workspace=workspace(desc, B.OP_BWD_DW))
    finally:
        B.set_plan_override(0, 0)
    assert np.array_equal(f64(y), orc.fwd_panels(xs, ws))
    assert np.array_equal(f64(dx), orc.bwd_dx_panels(dys, ws))
    assert np.array_equal(f64(dw), orc.bwd_dw_panels(xs, dys))
    assert np.array_equal(f64(db), sum(d.sum(0) for d in dys))


@pytest.mark.parametrize("op", ["fwd", "dx", "dw"])
@pytest.mark.parametrize("rows,cols,splits,k,q", MANY)
def test_more_workgroups_than_compute_units(op, rows, cols, splits, k, q):
    """Two stages in the LDS in place of three, two workgroups per compute unit: 289 tiles, and 156 in two
    parts; contractions of one stage, fewer stages than the ring holds, and more."""
    m, kb, n = {"fwd": (rows, k, cols), "dx": (rows, cols, k), "dw": (k, rows, cols)}[op]
    gen = torch.Generator().manual_seed(rows + k)
    desc = share_desc(q, 1, m, kb, n, "bf16", "f32")
    code = {"fwd": B.OP_FWD, "dx": B.OP_BWD_DX, "dw": B.OP_BWD_DW}[op]
    out = torch.full((rows, cols), float("nan"), dtype=torch.float32, device="cuda:0")
    first = _panels(q, *((m, n) if op == "dx" else (m, kb)), gen)
    second = _panels(q, *((m, n) if op == "dw" else (kb, n)), gen)
    db = torch.empty((n,), dtype=torch.float32, device="cuda:0")
    try:
        B.set_plan_override(tile=128, k_splits=splits)
        assert tess.plan(desc, code) == (128, 128, splits)
        ws = workspace(desc, code)
        if op == "fwd":
            tess.linear_fwd(desc, first[1], second[1], None, B.ACT_NONE, out, workspace=ws)
        elif op == "dx":
            tess.linear_bwd_dx(desc, first[1], second[1], out, workspace=ws)
        else:
            tess.linear_bwd_dw_bias(desc, first[1], second[1], out, db, workspace=ws)
    finally:
        B.set_plan_override(0, 0)
    want = {"fwd": orc.fwd_panels, "dx": orc.bwd_dx_panels, "dw": orc.bwd_dw_panels}[op](first[0], second[0])
    assert np.array_equal(f64(out), want)
    if op == "dw":
        assert np.array_equal(f64(db), sum(d.sum(0) for d in second[0]))
