"""Host-only: which kernel variant each shape of the GPU suite takes.  The launch plan is
pure host arithmetic (tess_linear_plan), so this runs without a GPU and fails when a
retuned cost model silently moves the GPU tests off a code path: every combination of
{256 x 256, 128 x 128 with three stages and with two, 64 x 64, 64 x 32} x {whole panels, ragged ones}
x {no K split, K split} x {forward, input gradient, weight gradient} must be taken by at least one GPU
test shape (the two-stage ring serves ragged panels only)."""
import itertools

import tess_workloads as wl
from paper_2105_14500_amd import binding as B

import test_gpu_configs
import test_gpu_parity
import test_gpu_ragged_k
import test_gpu_small_tiles
import test_gpu_tile_grids


def _variants(q, d, m, kb, n):
    desc = B.make_desc(q, d, 0, 0, 0, m * q * d, kb * q, n * q, B.BF16, B.BF16)
    out = []
    for op, name, (M, N, kp) in ((B.OP_FWD, "fwd", (m, n, kb)), (B.OP_BWD_DX, "dx", (m, kb, n)), (B.OP_BWD_DW, "dw", (kb, n, m))):
        bm, bn, splits = B.plan(desc, op)
        if bm:
            panels = "ragged" if kp % 64 else "whole"
            tile = bm if bm == bn else (bm, bn)
            if (tile, panels) == (128, "ragged") and -(-M // bm) * -(-N // bn) * splits > 256:
                tile = "128 two stages"
            out.append(((tile, panels), "split" if splits > 1 else "whole", name))
    return out


def test_gpu_suite_reaches_every_kernel_variant():
    seen = {}
    for q, d, m, kb, n, dtype in test_gpu_parity.SHAPES:
        if dtype == "bf16":
            for v in _variants(q, d, m, kb, n):
                seen.setdefault(v, ("test_gpu_parity.SHAPES", (q, d, m, kb, n)))
    for wname, lname in test_gpu_configs.CASES:
        w = wl.workload_by_name(wname)
        L = next(l for l in w.layers if l.name == lname)
        for v in _variants(w.q, w.d, L.m, L.kb, L.n):
            seen.setdefault(v, ("test_gpu_configs.CASES", (wname, lname)))
    try:
        forced = [(t, s, shape, "test_gpu_parity.FORCED") for t, s, shape in test_gpu_parity.FORCED]
        forced += [(t, s, (q, 1, *shape), "test_gpu_small_tiles.FORCED") for t, s, (q, *shape) in test_gpu_small_tiles.FORCED]
        forced += [(t, s, (test_gpu_ragged_k.Q, 1, *shape), "test_gpu_ragged_k.TILES") for t, s in test_gpu_ragged_k.TILES
                   for shape in test_gpu_ragged_k.SHAPES]
        for tile, splits, shape, where in forced:
            B.set_plan_override(tile=tile, k_splits=splits)
            for v in _variants(*shape):
                assert v[0][0] == (64 if tile == (64, 64) else tile) and (v[1] == "split") == (splits > 1)
                seen.setdefault(v, (where, (tile, splits, shape)))
        for rows, cols, splits, k, q in test_gpu_ragged_k.MANY:
            B.set_plan_override(tile=128, k_splits=splits)
            for name, shape in (("fwd", (rows, k, cols)), ("dx", (rows, cols, k)), ("dw", (k, rows, cols))):
                for v in _variants(q, 1, *shape):
                    if v[2] == name:
                        seen.setdefault(v, ("test_gpu_ragged_k.MANY", (splits, q, shape)))
    finally:
        B.set_plan_override(0, 0)
    tiles = list(itertools.product([256, 128, 64, (64, 32)], ["whole", "ragged"])) + [("128 two stages", "ragged")]
    want = set(itertools.product(tiles, ["whole", "split"], ["fwd", "dx", "dw"]))
    missing = sorted(want - set(seen), key=str)
    assert not missing, missing


def test_full_size_plans_of_the_configurations_match_the_exact_grid_tests():
    """The whole-output exact tests force the K-split count that the full-size call of the
    same output shape takes; if the cost model changes that count, this says which."""
    planned = set()
    for w in wl.WORKLOADS:
        if w.dtype != "bf16" or w.name.startswith("cfg2"):
            continue
        for L in w.layers:
            desc = B.make_desc(w.q, w.d, 0, 0, 0, L.a, L.b, L.c, B.BF16, B.BF16)
            for op, name, (M, N) in ((B.OP_FWD, "fwd", (L.m, L.n)), (B.OP_BWD_DX, "dx", (L.m, L.kb)),
                                     (B.OP_BWD_DW, "dw", (L.kb, L.n))):
                tile, _, splits = B.plan(desc, op)
                assert tile == 256
                planned.add((name, w.q, M, N, splits))
    assert planned == set(test_gpu_tile_grids.GRIDS), sorted(planned ^ set(test_gpu_tile_grids.GRIDS))
