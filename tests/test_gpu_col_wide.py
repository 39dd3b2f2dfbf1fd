"""Column passes of 512 rows: alone and beside other passes, row strides of one and more, ascending and
descending stages, with and without plan_V's radix-2 stage riding along, widths that do and do not
fill whole tiles (those fall back to passes of up to 128 rows), in place and with row pitches."""
import sys

import numpy as np
import pytest

from oracle import harp_oracle as ho
from paper_2605_29843_amd import inputs as gi
from parity_util import assert_parity, to_device, to_host64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ru,rv,cols", [
    ([8, 8, 8], None, 32), ([8, 8, 8], None, 96), ([8, 8, 8], None, 100), ([8, 8, 8], [2] * 5, 32),
    ([8, 8, 8, 3, 3, 3], None, 64),           # 512 and 27 rows
    ([7, 8, 8, 8, 8], [8, 4], 32),            # row stride 56
    ([8, 8, 8], [8, 8, 8, 5, 2], 5120),       # plan_V's stage on the top digit beside the pass of 512 rows
    ([8, 8, 8], [8, 8, 8, 8, 2], 8192),
])
def test_column_pass_of_512_rows(ru, rv, cols, dtype):
    import torch
    from paper_2605_29843_amd import harp
    do = int(np.prod(ru))
    rng = np.random.default_rng(do + cols)
    bu, su = gi.make_blocks(do, ru, "qr", rng), gi.make_signs(do, rng)
    pu, pv = harp.Plan(do, ru, bu, su), None
    if rv:
        bv, sv = gi.make_blocks(cols, rv, "qr", rng), gi.make_signs(cols, rng)
        pv = harp.Plan(cols, rv, bv, sv)
    print("512-row pass", ru, rv, cols, dtype, file=sys.stderr, flush=True)
    W = rng.standard_normal((do, cols)).astype(np.float32)
    if dtype == "bf16":
        W = gi.round_to_bf16(W)
    Wd = to_device(W, dtype)
    pitched = torch.zeros(do, cols + 8, dtype=Wd.dtype, device="cuda")[:, :cols]
    fwd = to_host64(harp.harp_rotate_weight(pu, pv, Wd, pitched))
    back = Wd.clone()
    back = to_host64(harp.harp_rotate_weight_inverse(pu, pv, back, back))
    W64 = W.astype(np.float64)
    for got, rows_fn, what in ((fwd, ho.apply_staged, "U^T W V"), (back, ho.apply_transpose_staged, "U W V^T")):
        M = rows_fn(W64, cols, rv, bv, sv) if rv else W64
        # every column of narrow matrices, else a hundred spread over both halves of the row
        pick = np.unique(np.linspace(0, cols - 1, 100).astype(int))
        ref = rows_fn(np.ascontiguousarray(M[:, pick].T), do, ru, bu, su).T
        rho = np.linalg.norm(M[:, pick], axis=0, keepdims=True) / np.sqrt(do)
        assert_parity(got[:, pick], ref, dtype, what, rho=rho)
    pu.destroy()
    if pv:
        pv.destroy()
