"""Column passes of two stages with the tile in registers: every pair of radices the kernel is built for, row
strides of one and more, ascending and descending stages, every pair of element types (a float32
workspace between two passes of a bf16 matrix comes with a plan_V that has no half-precision form) and
widths with a ragged last tile."""
import sys

import numpy as np
import pytest

from oracle import harp_oracle as ho
from paper_2605_29843_amd import inputs as gi
from parity_util import assert_parity, to_device, to_host64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rv", [None, [8, 8, 4], [4, 5, 7]])     # 256 and 140 columns with plan_V, 260 without
@pytest.mark.parametrize("ru", [[7, 4], [8, 3], [8, 4], [8, 5], [8, 6], [8, 7], [8, 8],
                                [8, 8, 8, 4], [8, 7, 7, 4], [3, 7, 4, 8, 5],
                                [2] * 6, [2] * 12, [2, 4, 2, 3], [4, 2, 5, 2, 2, 2, 7]])
def test_column_pass_of_two_stages(ru, rv, dtype):
    from paper_2605_29843_amd import harp
    do, cols = int(np.prod(ru)), int(np.prod(rv)) if rv else 260
    rng = np.random.default_rng(do + cols)
    bu, su = gi.make_blocks(do, ru, "qr", rng), gi.make_signs(do, rng)
    pu, pv = harp.Plan(do, ru, bu, su), None
    if rv:
        bv, sv = gi.make_blocks(cols, rv, "qr", rng), gi.make_signs(cols, rng)
        pv = harp.Plan(cols, rv, bv, sv)
    print("two-stage pass", ru, rv, dtype, file=sys.stderr, flush=True)
    W = rng.standard_normal((do, cols)).astype(np.float32)
    if dtype == "bf16":
        W = gi.round_to_bf16(W)
    Wd = to_device(W, dtype)
    W64 = W.astype(np.float64)
    for fn, rows_fn in ((harp.harp_rotate_weight, ho.apply_staged), (harp.harp_rotate_weight_inverse, ho.apply_transpose_staged)):
        M = rows_fn(W64, cols, rv, bv, sv) if rv else W64
        ref = rows_fn(np.ascontiguousarray(M.T), do, ru, bu, su).T
        rho = np.linalg.norm(M, axis=0, keepdims=True) / np.sqrt(do)
        assert_parity(to_host64(fn(pu, pv, Wd)), ref, dtype, fn.__name__, rho=rho)
    pu.destroy()
    if pv:
        pv.destroy()


@pytest.mark.parametrize("ru", [[2] * 12, [8, 8, 8, 7]])
def test_a_new_plan_is_ready_on_every_stream(ru):
    """The block values of these passes are made by a kernel while the plan is created: they are there when
    the call returns, for a stream that does not wait for any other."""
    import torch
    from paper_2605_29843_amd import harp
    do, cols = int(np.prod(ru)), 128
    rng = np.random.default_rng(do)
    bu, su = gi.make_blocks(do, ru, "qr", rng), gi.make_signs(do, rng)
    W = to_device(gi.round_to_bf16(rng.standard_normal((do, cols)).astype(np.float32)), "bf16")
    side = torch.cuda.Stream()
    for _ in range(5):
        torch.cuda.synchronize()
        plan = harp.Plan(do, ru, bu, su)
        with torch.cuda.stream(side):
            first = harp.harp_rotate_weight(plan, None, W)
        torch.cuda.synchronize()
        again = harp.harp_rotate_weight(plan, None, W)
        assert torch.equal(first, again)
        plan.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cols", [130, 260, 380, 2, 66])
@pytest.mark.parametrize("ru", [[2] * 6, [2] * 9, [2, 4, 2, 3], [8, 7]])
def test_equal_columns_give_equal_results(ru, cols, dtype):
    """Whatever the column's place: a ragged last tile takes the arithmetic of the whole ones."""
    from paper_2605_29843_amd import harp
    do = int(np.prod(ru))
    rng = np.random.default_rng(do + cols)
    plan = harp.Plan(do, ru, gi.make_blocks(do, ru, "qr", rng), gi.make_signs(do, rng))
    two = rng.standard_normal((do, 2)).astype(np.float32)
    W = to_device(gi.round_to_bf16(np.tile(two, (1, cols // 2))), dtype)
    for fn in (harp.harp_rotate_weight, harp.harp_rotate_weight_inverse):
        got = fn(plan, None, W)
        assert bool((got.view(do, cols // 2, 2) == got[:, :2].reshape(do, 1, 2)).all()), fn.__name__
    plan.destroy()
