"""bf16 panels of about 2 GiB and more whose contraction is no multiple of 64: every row is read, the
last ones among them, and what lies past a panel's end reads as zero.  Small integers: bit exact.
Every address of such calls is checked on the host by test_loader_addresses.py."""
import pytest
import torch

import paper_2105_14500_amd as tess
from paper_2105_14500_amd import binding as B
from gpu_util import share_desc, workspace

pytestmark = pytest.mark.gpu

CHUNK = 1 << 20


def _panel(rows, cols, ld):
    """Integers in [-1, 1] with NaN in the columns beside them."""
    room = torch.full((rows, ld), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    gen = torch.Generator(device="cuda:0").manual_seed(rows + cols)
    for r in range(0, rows, CHUNK):
        part = room[r:r + CHUNK, :cols]
        part.copy_(torch.randint(-1, 2, part.shape, generator=gen, device="cuda:0", dtype=torch.int8))
    return room[:, :cols]


# bytes of the large operand (rows x 160): 2^31 - 2528, and 2^31 + 12.5 M
ROWS = [13421757, 13499965]


@pytest.mark.parametrize("rows", ROWS)
@pytest.mark.parametrize("op", ["fwd", "dx"])
@pytest.mark.parametrize("tile", [0, 128, 256])
def test_many_rows(rows, op, tile):
    k, n = 72, 256 if tile == 256 else 64
    a = _panel(rows, k, 80)
    b = _panel(k, n, n + 8) if op == "fwd" else _panel(n, k, 80)
    desc = share_desc(1, 1, rows, k, n, "bf16", "bf16") if op == "fwd" else share_desc(1, 1, rows, n, k, "bf16", "bf16")
    code = B.OP_FWD if op == "fwd" else B.OP_BWD_DX
    out = torch.full((rows, n), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    try:
        B.set_plan_override(tile=tile, k_splits=0)
        assert B.plan(desc, code)[0] == (tile or B.plan(desc, code)[0]) != 0
        if op == "fwd":
            tess.linear_fwd(desc, [a], [b], None, B.ACT_NONE, out, workspace=workspace(desc, code))
        else:
            tess.linear_bwd_dx(desc, [a], [b], out, workspace=workspace(desc, code))
    finally:
        B.set_plan_override(0, 0)
    right = (b if op == "fwd" else b.t()).float().contiguous()
    for r in range(0, rows, CHUNK):      # integers of at most 72: exact in bf16
        assert torch.equal(out[r:r + CHUNK].float(), a[r:r + CHUNK].float() @ right)


@pytest.mark.parametrize("rows", ROWS)
@pytest.mark.parametrize("tile", [0, 128])
def test_a_long_contraction(rows, tile):
    kb, n = 72, 64
    x, dy = _panel(rows, kb, 80), _panel(rows, n, 72)
    desc = share_desc(1, 1, rows, kb, n, "bf16", "f32")
    dw = torch.full((kb, n), float("nan"), dtype=torch.float32, device="cuda:0")
    db = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda:0")
    try:
        B.set_plan_override(tile=tile, k_splits=0)
        assert B.plan(desc, B.OP_BWD_DW)[0] != 0
        tess.linear_bwd_dw_bias(desc, [x], [dy], dw, db, workspace=workspace(desc, B.OP_BWD_DW))
    finally:
        B.set_plan_override(0, 0)
    want, want_b = torch.zeros((kb, n), dtype=torch.float64, device="cuda:0"), torch.zeros((n,), dtype=torch.float64, device="cuda:0")
    for r in range(0, rows, CHUNK):      # sums of some 10^4: exact in fp32
        part = dy[r:r + CHUNK].double()
        want += x[r:r + CHUNK].double().t().contiguous() @ part
        want_b += part.sum(0)
    assert torch.equal(dw.double(), want) and torch.equal(db.double(), want_b)
