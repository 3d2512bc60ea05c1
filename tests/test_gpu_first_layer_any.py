"""First-layer backward-data whose output channels are a multiple of 4 but not of 32, on the kernel that forms the products of all filter
elements of a pixel at once: the edges of its chunks of 64 channels and steps of 16, of its tiles and of the rule that chooses it."""
import numpy as np
import pytest

import paper_2305_08819_amd as mc
from tests import gpu_util as gu
from tests.test_gpu_products import far_from_one, inputs, run

pytestmark = pytest.mark.gpu

# N, IH, IW, IC, OC, F, pad, tile rows
CASES = [
    (40, 33, 31, 3, 4, 3, 1, 8),        # one quad of channels
    (160, 16, 17, 2, 12, 3, 0, 8),
    (18, 16, 16, 3, 36, 3, 1, 4),       # the last step has 4 of 16 channels
    (7, 9, 70, 3, 60, 3, 1, 4),         # the last quad missing; tiles that end inside the row
    (300, 32, 32, 3, 68, 3, 1, 8),      # a second chunk of one quad
    (5, 33, 20, 1, 84, 3, 2, 4),        # padding of a whole filter; a second chunk of two steps, the last of one quad
    (33, 28, 28, 2, 120, 2, 1, 8),
    (200, 30, 30, 4, 20, 2, 0, 8),
    (600, 20, 20, 3, 60, 1, 0, 8),
    (30, 18, 18, 3, 196, 3, 1, 4),      # more than 192 channels: enough pixels
]


def desc(case):
    n, h, w, ic, oc, f, pad, rows = case
    d = mc.make_desc(n, h, w, ic, oc, f, f, 1, pad)
    p = mc.conv2d_query_plan(mc.OP_BWD_DATA, d)
    assert (p.kernel, p.tile_m, p.tile_n, p.grid) == (mc.KERNEL_DIRECT, 32 * rows, 32, n * -(-h // rows) * -(-w // 32)), \
        (p.kernel, p.tile_m, p.tile_n, p.grid)
    assert p.variant == mc.VARIANT_MFMA and mc.conv2d_query_products(mc.OP_BWD_DATA, d) == mc.PRODUCTS_TERMS
    print("first layer", case, p.grid, flush=True)
    return d


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_any_quads(case):
    gu.check_all_ops(desc(case), *inputs(desc(case), 41), ops=("bwd_data",), label=str(case), twice=True)


@pytest.mark.parametrize("shape", [(18, 16, 16, 3, 36, 3, 1), (4, 32, 32, 3, 44, 3, 1), (160, 7, 7, 3, 36, 3, 0)])
def test_former_short_calls_need_no_workspace(shape):
    n, h, w, ic, oc, f, pad = shape
    d = mc.make_desc(n, h, w, ic, oc, f, f, 1, pad)
    p = mc.conv2d_query_plan(mc.OP_BWD_DATA, d)
    assert p.tile_m > 32 and p.split == 1 and mc.conv2d_workspace_bytes(mc.OP_BWD_DATA, d) == 0
    gu.check_all_ops(d, *inputs(d, 43), ops=("bwd_data",), label=str(shape))


@pytest.mark.parametrize("kind", ["1e-37", "1e-42", "hidden", "2^-133"])
def test_small_operand_with_a_large_partner(kind):
    """Operands that three bf16 terms do not hold (see test_gpu_products), in either operand, at the parity tests' bar."""
    for case in (CASES[3], CASES[5]):
        d = desc(case)
        a, b = far_from_one("bwd_data", *gu.operands("bwd_data", *inputs(d, 11)), kind)
        ref = gu.run_oracle("bwd_data", d, a, b)
        got = run("bwd_data", d, a, b).astype(np.float64)
        assert np.linalg.norm((got - ref).ravel()) <= 1e-5 * np.linalg.norm(ref.ravel())


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_operands_reach_what_their_taps_reach(value):
    for case in (CASES[2], CASES[9]):
        d = desc(case)
        for which in (0, 1):
            ab = list(gu.operands("bwd_data", *inputs(d, 3)))
            ab[which].reshape(-1)[ab[which].size // 3] = value
            ref, got = gu.run_oracle("bwd_data", d, *ab), run("bwd_data", d, *ab)
            assert 0 < np.isfinite(ref).sum() < ref.size
            for f in (np.isnan, np.isposinf, np.isneginf):
                assert np.array_equal(f(got), f(ref)), (case, which)
            ok = np.isfinite(ref)
            assert np.linalg.norm(got[ok].astype(np.float64) - ref[ok]) <= 1e-5 * np.linalg.norm(ref[ok])


@pytest.mark.parametrize("shape", [(57, 5, 4, 1, 432, 3, 1), (7, 32, 32, 2, 12, 3, 1), (4, 32, 32, 2, 268, 1, 0), (217, 33, 33, 3, 308, 1, 0), (40, 33, 31, 3, 30, 3, 1)])
def test_calls_that_stay(shape):
    """Few pixels under many channels, short calls, 1x1 filters of many channels, and channel counts off the grid of quads."""
    n, h, w, ic, oc, f, pad = shape
    p = mc.conv2d_query_plan(mc.OP_BWD_DATA, mc.make_desc(n, h, w, ic, oc, f, f, 1, pad))
    assert p.kernel != mc.KERNEL_DIRECT or p.tile_m == 32, (p.kernel, p.tile_m)
