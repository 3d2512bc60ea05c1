"""The 32 x 32 block kernel on channel counts off the grid of four: the last quad of a tap starts at the fourth channel from the end, and
a block's last columns are any number.  Against the oracle; short calls and large 1x1 results stay where they were."""
import numpy as np
import pytest
import torch

import paper_2305_08819_amd as mc
from tests import gpu_util as gu
from tests.test_gpu_block import CODE
from tests.test_gpu_products import far_from_one, inputs, run

pytestmark = pytest.mark.gpu

# N, IH, IW, IC, OC, F, stride, pad
CASES = {
    "fwd": [
        (32, 9, 9, 65, 64, 3, 1, 1),       # an item of one channel: its quad starts in the item before
        (32, 7, 7, 30, 96, 5, 1, 2),       # two channels twice
        (96, 7, 7, 63, 62, 3, 1, 1),       # three channels in the last quad; 30 of 32 columns
        (5, 31, 31, 97, 127, 3, 1, 1),     # more blocks than CUs, rows that cross images
        (32, 18, 21, 90, 53, 3, 2, 1),
        (224, 4, 3, 107, 112, 3, 1, 0),    # sixteen waves
        (1, 105, 105, 19, 25, 5, 1, 2),    # a map of more than 2^13 pixels, one chunk
        (100, 29, 29, 65, 66, 3, 1, 1),    # over 2^16 rows
        (33, 5, 5, 64, 41, 3, 1, 1),       # whole quads, odd columns
    ],
    "bwd_data": [
        (32, 10, 10, 90, 72, 3, 1, 1),
        (35, 14, 15, 58, 65, 3, 1, 1),     # an item of one channel
        (29, 13, 13, 123, 94, 3, 2, 1),    # the four stride phases, 27 of 32 columns
        (32, 6, 5, 461, 63, 3, 1, 1),
        (32, 4, 2, 318, 61, 5, 1, 2),      # most taps padding
        (10, 29, 29, 34, 33, 3, 2, 1),
        (64, 9, 9, 94, 22, 3, 2, 1),       # less than one item
    ],
}
BOTH = [(op, c) for op in CASES for c in CASES[op]]
IDS = ["%s-%s" % (op, "x".join(map(str, c))) for op, c in BOTH]


def plan(op, case):
    n, h, w, ic, oc, f, s, p = case
    d = mc.make_desc(n, h, w, ic, oc, f, f, s, p)
    return d, mc.conv2d_query_plan(CODE[op], d), mc.conv2d_query_products(CODE[op], d)


def desc(op, case):
    d, q, products = plan(op, case)
    assert (q.kernel, q.tile_m, q.tile_n, products) == (mc.KERNEL_DIRECT, 32, 32, mc.PRODUCTS_TERMS), (q.kernel, q.tile_m, products)
    print("block", op, case, q.grid, q.pos_major, flush=True)
    return d


@pytest.mark.parametrize("op,case", BOTH, ids=IDS)
def test_channels(op, case):
    gu.check_all_ops(desc(op, case), *inputs(desc(op, case), 51), ops=(op,), label=str((op, case)), twice=True)


@pytest.mark.parametrize("case", [CASES["fwd"][2], CASES["fwd"][5]], ids=lambda c: "x".join(map(str, c)))
def test_bias_and_activation(case):
    d = desc("fwd", case)
    X, W, _ = inputs(d, 5)
    bias = np.random.default_rng(6).standard_normal(d.OC + 1).astype(np.float32)
    y = gu.run_oracle("fwd", d, X, W) + bias[1:]
    ref = np.where(y > 0, y, y * 0.125)
    buf, Y = gu.guarded((d.N, d.OH, d.OW, d.OC))
    mc.conv2d_fwd_bias_act(gu.nan_fenced(X), gu.nan_fenced(W), torch.from_numpy(bias).cuda()[1:], Y, d, 0.125)
    torch.cuda.synchronize()
    assert gu.guards_intact(buf)
    rel, mx = gu.errors(Y.cpu().numpy(), ref)
    assert rel <= gu.REL_L2_TOL and mx <= gu.MAX_ABS_TOL, (case, rel, mx)


@pytest.mark.parametrize("kind", ["1e-37", "1e-42", "hidden", "2^-133"])
def test_small_operand_with_a_large_partner(kind):
    """Operands that three bf16 terms do not hold (see test_gpu_products), in either operand, at the parity tests' bar."""
    for op, case in (("fwd", CASES["fwd"][1]), ("bwd_data", CASES["bwd_data"][1])):
        d = desc(op, case)
        a, b = far_from_one(op, *gu.operands(op, *inputs(d, 11)), kind)
        ref = gu.run_oracle(op, d, a, b)
        got = run(op, d, a, b).astype(np.float64)
        assert np.linalg.norm((got - ref).ravel()) <= 1e-5 * np.linalg.norm(ref.ravel())


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_operands_reach_what_their_taps_reach(value):
    """In the last channels of a pixel and of the filter, which a tap's last two quads share."""
    for op, case in (("fwd", CASES["fwd"][0]), ("fwd", CASES["fwd"][2]), ("bwd_data", CASES["bwd_data"][1]), ("bwd_data", CASES["bwd_data"][5])):
        d = desc(op, case)
        for which in (0, 1):
            for back in (1, 2, 4):
                a, b = (v.copy() for v in gu.operands(op, *inputs(d, 3)))
                if which == 0:
                    a[a.shape[0] // 2, a.shape[1] // 2, 0, -back] = value
                elif op == "fwd":
                    b[b.shape[0] // 2, 0, 0, -back] = value
                else:
                    b[-back, 0, 0, b.shape[3] // 2] = value
                ref, got = gu.run_oracle(op, d, a, b), run(op, d, a, b)
                assert 0 < np.isfinite(ref).sum() < ref.size
                for f in (np.isnan, np.isposinf, np.isneginf):
                    assert np.array_equal(f(got), f(ref)), (op, case, which, back)
                ok = np.isfinite(ref)
                assert np.linalg.norm(got[ok].astype(np.float64) - ref[ok]) <= 1e-5 * np.linalg.norm(ref[ok])


@pytest.mark.parametrize("op,case", [("fwd", (32, 75, 63, 55, 64, 1, 1, 0)), ("fwd", (3, 27, 27, 337, 32, 5, 2, 2)), ("bwd_data", (32, 10, 12, 39, 64, 1, 1, 0)),
                                     ("fwd", (4, 9, 9, 3, 40, 3, 2, 1))])
def test_calls_that_stay(op, case):
    """Large 1x1 results, long sums of few blocks, short calls, fewer than four channels."""
    _, q, products = plan(op, case)
    assert products == mc.PRODUCTS_FP32 or q.kernel == mc.KERNEL_FIRST_LAYER, (q.kernel, products)
