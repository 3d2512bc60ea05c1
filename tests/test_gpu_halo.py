"""The forward / backward-data kernel of unit-stride layers with equal maps, which splits the gathered pixels once for all
taps: its tiles at the edges of what they hold, against the oracle."""
import numpy as np
import pytest

import paper_2305_08819_amd as mc
from tests import gpu_util as gu
from tests.test_gpu_products import far_from_one, inputs, run

pytestmark = pytest.mark.gpu
CODE = {"fwd": mc.OP_FWD, "bwd_data": mc.OP_BWD_DATA}
BOTH = ("fwd", "bwd_data")


@pytest.fixture(autouse=True)
def _restore():
    yield
    mc.conv2d_set_tuning(mc.VARIANT_AUTO, 0)


# (N, H, W, IC, OC, FH, FW, stride, pad), forced slices (0: the planner's), operators
CASES = [
    ((333, 8, 8, 64, 128, 3, 3, 1, 1), 0, BOTH),         # 256-row tiles of whole images, a partial last one
    ((333, 8, 8, 64, 128, 3, 3, 1, 1), 100, BOTH),       # as many slices as chunks
    ((39, 32, 32, 64, 64, 3, 3, 1, 1), 0, BOTH),         # whole rows and the rows above and below: exactly 320 pixels
    ((24, 31, 31, 64, 64, 3, 3, 1, 1), 0, BOTH),         # any run of rows: exactly 320 pixels
    ((24, 31, 31, 64, 64, 3, 3, 1, 1), 2, BOTH),
    ((130, 16, 16, 32, 32, 3, 3, 1, 1), 0, BOTH),        # one chunk: every filter stage is of the same pixels
    ((3, 64, 64, 64, 128, 3, 3, 1, 1), 0, ("fwd",)),     # 128-row tiles: exactly 256 pixels of whole rows
    ((4, 40, 63, 64, 128, 3, 3, 1, 1), 0, ("fwd",)),     # and of any rows
    ((3, 64, 64, 64, 128, 3, 3, 1, 1), 100, BOTH),
    ((6, 48, 48, 64, 256, 3, 3, 1, 1), 100, BOTH),
    ((200, 6, 6, 36, 156, 3, 3, 1, 1), 0, BOTH),         # channels that are not multiples of 32 or 64, on either side
    ((37, 13, 11, 68, 132, 3, 3, 1, 1), 100, BOTH),
    ((50, 14, 14, 36, 60, 5, 5, 1, 2), 100, BOTH),       # 25 taps
    ((8, 32, 32, 64, 100, 5, 5, 1, 2), 100, BOTH),       # 25 taps, 128-row tiles: two rows above and below
    ((40, 24, 20, 64, 64, 3, 5, 1, (1, 2)), 0, BOTH),    # filters that are not square
    ((400, 1, 100, 32, 64, 1, 7, 1, (0, 3)), 0, BOTH),   # one row, and as few taps as the tile's loads allow
    ((400, 90, 1, 64, 64, 7, 1, 1, (3, 0)), 0, BOTH),    # one column
    ((150, 9, 5, 64, 256, 3, 3, 1, 1), 0, BOTH),
    ((2000, 3, 4, 32, 32, 3, 3, 1, 1), 2, BOTH),         # tiles over many small images
]


def plan(op, d):
    p = mc.conv2d_query_plan(CODE[op], d)
    assert p.order == mc.ORDER_CONTIGUOUS and mc.conv2d_query_products(CODE[op], d) == mc.PRODUCTS_TERMS, (op, p.order, p.tile_m)
    return p


@pytest.mark.parametrize("shp,split,ops", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_tiles(shp, split, ops):
    d = mc.make_desc(*shp)
    mc.conv2d_set_tuning(mc.VARIANT_AUTO, split)
    for op in ops:
        p = plan(op, d)
        print("halo", shp, op, p.tile_m, p.tile_n, p.split, p.grid, flush=True)
    gu.check_all_ops(d, *inputs(d, 21), ops=ops, label=str(shp), twice=True)


@pytest.mark.parametrize("shp,split,ops", [CASES[i] for i in (2, 8, 10)], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
@pytest.mark.parametrize("kind", ["1e-37", "1e-42", "hidden", "2^-133"])
def test_small_operand_with_a_large_partner(shp, split, ops, kind):
    """Operands that three bf16 terms do not hold (see test_gpu_products), against the oracle at the parity tests' bar."""
    d = mc.make_desc(*shp)
    mc.conv2d_set_tuning(mc.VARIANT_AUTO, split)
    for op in ops:
        p = plan(op, d)
        print("halo small", shp, op, kind, p.tile_m, p.split, flush=True)
        a, b = far_from_one(op, *gu.operands(op, *inputs(d, 11)), kind)
        ref = gu.run_oracle(op, d, a, b)
        got = run(op, d, a, b).astype(np.float64)
        assert np.linalg.norm((got - ref).ravel()) <= 1e-5 * np.linalg.norm(ref.ravel()), op


@pytest.mark.parametrize("shp,split,ops", [CASES[i] for i in (0, 3, 8, 10)], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_operands_reach_what_their_taps_reach(shp, split, ops, value):
    """Exactly the elements whose taps inside the image read the infinity or NaN are not finite, and the others are what they
    are without it: an infinite filter element does not reach the border pixels at which its tap lies outside."""
    d = mc.make_desc(*shp)
    mc.conv2d_set_tuning(mc.VARIANT_AUTO, split)
    for op in ops:
        p = plan(op, d)
        print("halo non-finite", shp, op, value, p.tile_m, p.split, flush=True)
        a, b = gu.operands(op, *inputs(d, 3))
        a.reshape(-1)[a.size // 3] = value
        b.reshape(-1)[5] = float("inf")               # filter row 0, column 0: outside the image at the first rows and columns
        ref = gu.run_oracle(op, d, a, b)
        got = run(op, d, a, b)
        assert np.isnan(got).any() or np.isinf(got).any()
        assert np.isfinite(got).sum() == np.isfinite(ref).sum() > 0
        for f in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(f(got), f(ref)), op
        ok = np.isfinite(ref)
        assert np.linalg.norm(got[ok].astype(np.float64) - ref[ok]) <= 1e-5 * np.linalg.norm(ref[ok])


def test_fused_bias_and_activation():
    """Unsliced (in the epilogue) and sliced (in the combine pass), columns past the last one, rows past the last one."""
    import torch
    for shp, split in [((200, 6, 6, 36, 156, 3, 3, 1, 1), 1), ((200, 6, 6, 36, 156, 3, 3, 1, 1), 2), ((3, 64, 64, 64, 128, 3, 3, 1, 1), 1)]:
        d = mc.make_desc(*shp)
        mc.conv2d_set_tuning(mc.VARIANT_AUTO, split)
        assert plan("fwd", d).split == split
        X, W, _ = inputs(d, 5)
        bias = np.linspace(-1, 1, d.OC + 1).astype(np.float32)
        ref = gu.run_oracle("fwd", d, X, W) + bias[1:]
        ref = np.where(ref > 0, ref, ref * np.float32(0.125))
        buf, Y = gu.guarded((d.N, d.OH, d.OW, d.OC))
        tb = torch.from_numpy(bias).cuda()[1:]        # aligned to 4 bytes only
        mc.conv2d_fwd_bias_act(gu.nan_fenced(X), gu.nan_fenced(W), tb, Y, d, 0.125)
        torch.cuda.synchronize()
        assert gu.guards_intact(buf)
        rel, mx = gu.errors(Y.cpu().numpy(), ref)
        assert rel <= gu.REL_L2_TOL and mx <= gu.MAX_ABS_TOL, (shp, split, rel, mx)


@pytest.mark.parametrize("n", [128, 129])
def test_results_around_32_mb(n):
    """Below: plain stores; from there on nontemporal ones, the last tile partial."""
    d = mc.make_desc(n, 33, 31, 64, 64, 3, 3, 1, 1)
    assert (d.N * d.OH * d.OW * d.OC * 4 >= 32 << 20) == (n == 129) and plan("fwd", d).split == 1
    print("halo large", n, flush=True)
    gu.check_all_ops(d, *inputs(d, 9), ops=("fwd",), label=str(n), twice=True)
