"""Column passes (rotation along the row index of a matrix) of every height up to 128.  On the LDS-tile kernel,
at every number of row steps per wave it is built for: heights that fill the steps and heights that
repeat rows, float32 on both sides, and half-precision workspaces (bf16, two-sided).  Pairs of radix 8 and
3 .. 8 and of 7 and 4 with a float32 workspace run on the kernel of two-stage passes instead; the same heights
with the radices the other way round keep the LDS tile."""
import sys

import numpy as np
import pytest

from oracle import harp_oracle as ho
from paper_2605_29843_amd import inputs as gi
from parity_util import assert_parity, to_device, to_host64

pytestmark = pytest.mark.gpu


# the rows of one pass (all stages of the plan), or of each of two passes (the last four plans; a float32
# workspace where each of them is a pair or a single stage, else halves for bf16)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("radices", [
    [2, 3], [2, 4], [3, 3], [2, 7], [3, 5], [2, 8], [3, 7], [8, 3], [5, 5], [4, 7], [3, 3, 4], [8, 5], [7, 6], [8, 6], [7, 7],
    [8, 7], [3, 4, 5], [8, 8], [5, 7, 2], [8, 3, 3], [8, 5, 2], [3, 3, 3, 3], [6, 4, 4], [7, 2, 7], [8, 7, 2],
    [8, 3, 5], [8, 2, 8], [5, 5, 5], [3, 8], [5, 8], [6, 8], [7, 8],
    [8, 3, 8, 3, 8], [8, 5, 8, 5], [8, 7, 8, 7], [8, 7, 2, 8, 5, 2]])
def test_column_pass_heights(radices, dtype):
    import torch
    from paper_2605_29843_amd import harp
    do, cols = int(np.prod(radices)), 256
    rng = np.random.default_rng(do)
    blocks, signs = gi.make_blocks(do, radices, "orth", rng), gi.make_signs(do, rng)
    plan = harp.Plan(do, radices, blocks, signs)
    W = rng.standard_normal((do, cols)).astype(np.float32)
    if dtype == "bf16":
        W = gi.round_to_bf16(W)
    print("column pass heights", radices, dtype, file=sys.stderr, flush=True)
    Wd = to_device(W, dtype)
    out, back = harp.harp_rotate_weight(plan, None, Wd), harp.harp_rotate_weight_inverse(plan, None, Wd)
    # columns of U^T W and U W: rows of W^T through the processor and its transpose
    W64 = W.astype(np.float64)
    fwd = ho.apply_staged(np.ascontiguousarray(W64.T), do, radices, blocks, signs).T
    inv = ho.apply_transpose_staged(np.ascontiguousarray(W64.T), do, radices, blocks, signs).T
    rho = np.linalg.norm(W64, axis=0, keepdims=True) / np.sqrt(do)   # the transformed vectors are columns
    assert_parity(to_host64(out), fwd, dtype, "U^T W", rho=rho)
    assert_parity(to_host64(back), inv, dtype, "U W", rho=rho)
    plan.destroy()


# heights of one pass (and of two) with the halves between it and plan_V's kernel
@pytest.mark.parametrize("rv", [[2] * 10, [2] * 11])
@pytest.mark.parametrize("ru", [[3, 8], [8, 3], [8, 5], [8, 6], [8, 7], [7, 8], [8, 8], [7, 4], [3, 3, 4], [8, 7, 2],
                                [8, 3, 8, 3, 8], [8, 7, 8, 7]])
def test_column_pass_heights_on_halves(ru, rv):
    from paper_2605_29843_amd import harp
    do, cols = int(np.prod(ru)), int(np.prod(rv))
    rng = np.random.default_rng(do + cols)
    bu, su, bv, sv = (f(d, r, "orth", rng) if f is gi.make_blocks else f(d, rng)
                      for d, r in ((do, ru), (cols, rv)) for f in (gi.make_blocks, gi.make_signs))
    pu, pv = harp.Plan(do, ru, bu, su), harp.Plan(cols, rv, bv, sv)
    print("column pass heights on halves", ru, rv, file=sys.stderr, flush=True)
    W = gi.round_to_bf16(rng.standard_normal((do, cols)).astype(np.float32))
    Wd, W64 = to_device(W, "bf16"), W.astype(np.float64)
    for fn, rows_fn in ((harp.harp_rotate_weight, ho.apply_staged), (harp.harp_rotate_weight_inverse, ho.apply_transpose_staged)):
        M = rows_fn(W64, cols, rv, bv, sv)
        ref = rows_fn(np.ascontiguousarray(M.T), do, ru, bu, su).T
        rho = np.linalg.norm(M, axis=0, keepdims=True) / np.sqrt(do)
        assert_parity(to_host64(fn(pu, pv, Wd)), ref, "bf16", fn.__name__, rho=rho)
    pu.destroy()
    pv.destroy()
