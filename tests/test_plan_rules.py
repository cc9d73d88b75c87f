"""Host-only: launch plans where the cost model alone chose a kernel that measures slower, one shape for
each rule beside it (tess_api.cpp has both sides' times)."""
import pytest

from paper_2105_14500_amd import binding as B

OPS = {"fwd": B.OP_FWD, "dx": B.OP_BWD_DX, "dw": B.OP_BWD_DW}


def _plan(op, q, m, kb, n):
    return B.plan(B.make_desc(q, 1, 0, 0, 0, m * q, kb * q, n * q, B.BF16, B.BF16), OPS[op])


@pytest.mark.parametrize("op,q,m,kb,n,tile", [
    ("dw", 1, 152, 3632, 4952, 128), ("fwd", 8, 4216, 16, 4840, 128), ("fwd", 3, 4992, 32, 3568, 128),      # few stages
    ("fwd", 1, 5664, 1200, 1696, 256), ("dw", 1, 1672, 3024, 4096, 256), ("dx", 4, 4032, 3160, 104, 256),      # many, plain drain
    ("fwd", 1, 4104, 1000, 4096, 128), ("dw", 2, 1000, 4104, 4096, 128)])                                   # a second round
def test_256_tiles_of_ragged_contractions(op, q, m, kb, n, tile):
    assert _plan(op, q, m, kb, n) == (tile, tile, 1)


@pytest.mark.parametrize("op,q,m,kb,n,tile", [
    ("dx", 1, 2304, 2816, 64, 128), ("dx", 3, 2112, 640, 64, 128), ("fwd", 1, 4224, 64, 512, 128),          # few stages, many tiles
    ("dx", 2, 3616, 1296, 120, 128), ("dw", 1, 16, 1344, 3376, 128),
    ("dw", 3, 64, 3968, 1216, 64), ("dx", 2, 1600, 640, 192, 64), ("fwd", 3, 5568, 128, 192, 64),           # the other side of the line
    ("dw", 8, 704, 1024, 576, 128), ("dw", 1, 5760, 1472, 576, 128), ("dw", 8, 448, 1408, 704, 64)])        # many stages of dW
def test_64_tiles(op, q, m, kb, n, tile):
    assert _plan(op, q, m, kb, n)[0] == tile
