"""Column passes (rotation along the row index of a matrix) on the LDS-tile kernel at every number of
row steps per wave it is built for: heights that fill the steps and heights that repeat rows, with
float32 and (bf16, two passes) half-precision workspaces."""
import sys

import numpy as np
import pytest

from oracle import harp_oracle as ho
from paper_2605_29843_amd import inputs as gi
from parity_util import assert_parity, to_device, to_host64

pytestmark = pytest.mark.gpu


# the rows of one pass (all stages of the plan), or of each of two passes (the last four plans)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("radices", [
    [2, 3], [2, 4], [3, 3], [2, 7], [3, 5], [2, 8], [3, 7], [8, 3], [5, 5], [4, 7], [3, 3, 4], [8, 5], [7, 6], [8, 6], [7, 7],
    [8, 7], [3, 4, 5], [8, 8], [5, 7, 2], [8, 3, 3], [8, 5, 2], [3, 3, 3, 3], [6, 4, 4], [7, 2, 7], [8, 7, 2],
    [8, 3, 5], [8, 2, 8], [5, 5, 5],
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
