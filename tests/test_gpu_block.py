"""The kernel of small results with long sums (forward and backward-data in 32 x 32 blocks, one launch) at the edges of its blocks,
items, taps and row orders, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2305_08819_amd as mc
from tests import gpu_util as gu
from tests.test_gpu_products import far_from_one, inputs, run

pytestmark = pytest.mark.gpu
CODE = {"fwd": mc.OP_FWD, "bwd_data": mc.OP_BWD_DATA}

# N, IH, IW, IC, OC, F, stride, pad
CASES = {
    "fwd": [
        (128, 2, 2, 512, 512, 3, 1, 1),    # one block a CU, one position a block, sixteen waves
        (33, 4, 4, 64, 64, 3, 1, 1),       # blocks that span two positions, half a block at the end
        (20, 11, 11, 96, 32, 3, 2, 1),
        (32, 2, 2, 124, 216, 5, 1, 2),     # last item and last block of columns partly empty, most taps padding
        (352, 10, 10, 32, 32, 3, 2, 1),    # more blocks than CUs, about one item a wave
        (2, 41, 41, 76, 28, 3, 1, 1),      # rows that cross images
        (1, 36, 44, 32, 268, 3, 1, 0),     # no padding, (n, y, x) rows
        (256, 1, 1, 1024, 512, 1, 1, 0),   # a matrix product
    ],
    "bwd_data": [
        (128, 2, 2, 512, 512, 3, 1, 1),
        (33, 4, 4, 64, 64, 3, 1, 1),
        (20, 11, 11, 96, 32, 3, 2, 1),     # four stride phases of odd extents
        (32, 6, 6, 96, 64, 3, 2, 0),       # rows and columns of the map that no tap reaches
        (32, 2, 2, 124, 216, 5, 1, 2),
        (32, 7, 6, 96, 76, 5, 2, 0),
        (16, 8, 8, 144, 228, 3, 2, 1),     # rows that cross positions of two phases
        (7, 15, 15, 48, 60, 3, 1, 1),      # 28 channels in the last item
        (2, 41, 41, 76, 28, 3, 1, 1),
    ],
}
BOTH = [(op, c) for op in CASES for c in CASES[op]]
IDS = ["%s-%s" % (op, "x".join(map(str, c))) for op, c in BOTH]


def desc(op, case):
    n, h, w, ic, oc, f, s, p = case
    d = mc.make_desc(n, h, w, ic, oc, f, f, s, p)
    q = mc.conv2d_query_plan(CODE[op], d)
    assert (q.kernel, q.tile_m, q.tile_n) == (mc.KERNEL_DIRECT, 32, 32) and mc.conv2d_query_products(CODE[op], d) == mc.PRODUCTS_TERMS
    print("block", op, case, q.grid, q.pos_major, flush=True)
    return d


@pytest.mark.parametrize("op,case", BOTH, ids=IDS)
def test_blocks(op, case):
    gu.check_all_ops(desc(op, case), *inputs(desc(op, case), 31), ops=(op,), label=str(case), twice=True)


@pytest.mark.parametrize("op,case", BOTH, ids=IDS)
def test_no_less_exact_than_the_tiled_kernels(op, case):
    """2-norm error against 64-bit sums, here and with the fp32 products that the call would take otherwise."""
    d = desc(op, case)
    t = inputs(d, 7)
    block = gu.check_all_ops(d, *t, ops=(op,))[op][0]
    mc.conv2d_set_products(mc.PRODUCTS_FP32)
    try:
        tiled = gu.check_all_ops(d, *t, ops=(op,))[op][0]
    finally:
        mc.conv2d_set_products(mc.PRODUCTS_AUTO)
    print("%.2e %.2e" % (block, tiled), flush=True)
    assert block <= tiled


@pytest.mark.parametrize("op", ["fwd", "bwd_data"])
@pytest.mark.parametrize("kind", ["1e-37", "1e-42", "hidden", "2^-133"])
def test_small_operand_with_a_large_partner(op, kind):
    """Operands that three bf16 terms do not hold (see test_gpu_products), in either operand, at the parity tests' bar."""
    d = desc(op, (33, 4, 4, 64, 64, 3, 1, 1))
    a, b = far_from_one(op, *gu.operands(op, *inputs(d, 11)), kind)
    ref = gu.run_oracle(op, d, a, b)
    got = run(op, d, a, b).astype(np.float64)
    assert np.linalg.norm((got - ref).ravel()) <= 1e-5 * np.linalg.norm(ref.ravel())


@pytest.mark.parametrize("op", ["fwd", "bwd_data"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_operands_reach_what_their_taps_reach(op, value):
    for case in ((20, 11, 11, 96, 32, 3, 2, 1), (33, 4, 4, 64, 64, 3, 1, 1)):
        d = desc(op, case)
        for which in (0, 1):
            ab = list(gu.operands(op, *inputs(d, 3)))
            ab[which].reshape(-1)[ab[which].size // 3] = value
            ref, got = gu.run_oracle(op, d, *ab), run(op, d, *ab)
            assert 0 < np.isfinite(ref).sum() < ref.size
            for f in (np.isnan, np.isposinf, np.isneginf):
                assert np.array_equal(f(got), f(ref)), (case, which)
            ok = np.isfinite(ref)
            assert np.linalg.norm(got[ok].astype(np.float64) - ref[ok]) <= 1e-5 * np.linalg.norm(ref[ok])


def test_fused_bias_and_activation():
    for case in (CASES["fwd"][0], CASES["fwd"][3]):
        d = desc("fwd", case)
        X, W, _ = inputs(d, 5)
        bias = np.linspace(-1, 1, d.OC + 1).astype(np.float32)
        ref = gu.run_oracle("fwd", d, X, W) + bias[1:]
        ref = np.where(ref > 0, ref, ref * np.float32(0.125))
        buf, Y = gu.guarded((d.N, d.OH, d.OW, d.OC))
        tb = torch.from_numpy(bias).cuda()[1:]        # aligned to 4 bytes only
        ws = torch.empty(mc.conv2d_workspace_bytes(mc.OP_FWD, d), dtype=torch.uint8, device="cuda")
        mc.conv2d_fwd_bias_act(gu.nan_fenced(X), gu.nan_fenced(W), tb, Y, d, 0.125, ws=ws)
        torch.cuda.synchronize()
        assert gu.guards_intact(buf)
        rel, mx = gu.errors(Y.cpu().numpy(), ref)
        assert rel <= gu.REL_L2_TOL and mx <= gu.MAX_ABS_TOL, (case, rel, mx)
