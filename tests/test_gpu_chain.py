"""Chains of radices 8, 8, 8, 3..8 on the float32 matrix instruction: every radix of the last stage, as a
whole row and as the chunk of a split program, row counts around the tile of eight (and of four rows,
the operand of one instruction), both element types, both directions, in place, and rows that hold
infinities (a tile's rows must not mix)."""
import sys

import numpy as np
import pytest

from oracle import harp_oracle as ho
from paper_2605_29843_amd import inputs as gi
from parity_util import assert_parity, summand_magnitude, to_device, to_host64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("top", [[], [3], [2, 2]])     # whole rows; one streamed stage; two of radix 2
@pytest.mark.parametrize("r4", [3, 4, 5, 6, 7, 8])
def test_chain(r4, top, dtype):
    import torch
    from paper_2605_29843_amd import harp
    radices = [8, 8, 8, r4] + top
    d = int(np.prod(radices))
    if top and d <= 4096:
        pytest.skip("the whole row is one chunk of other radices")
    rng = np.random.default_rng(d)
    kind = "qr" if r4 % 2 else "generic"
    blocks, signs = gi.make_blocks(d, radices, kind, rng), gi.make_signs(d, rng)
    plan = harp.Plan(d, radices, blocks, signs)
    for n in (1, 4, 5, 8, 19):
        print("chain", radices, dtype, n, file=sys.stderr, flush=True)
        X = rng.standard_normal((n, d)).astype(np.float32)
        X *= np.exp2(rng.integers(-20, 20, size=(n, 1))).astype(np.float32)
        if dtype == "bf16":
            X = gi.round_to_bf16(X)
        Xd = to_device(X, dtype)
        wide = torch.zeros(n, d + 16, dtype=Xd.dtype, device="cuda")[:, 8:8 + d]   # rows with a pitch
        out = harp.harp_apply(plan, Xd, wide)
        mag = summand_magnitude(X, d, radices, blocks) if kind == "generic" else None
        assert_parity(to_host64(out), ho.apply_staged(X, d, radices, blocks, signs), dtype, f"apply n={n}", mag=mag)
        back = Xd.clone()
        harp.harp_apply_transpose(plan, back, back)
        mag = summand_magnitude(X, d, radices, blocks, True) if kind == "generic" else None
        assert_parity(to_host64(back), ho.apply_transpose_staged(X, d, radices, blocks, signs), dtype,
                      f"transposed n={n}", mag=mag)
    # an infinity stays in its row, and in its block's outputs at the first stage
    bad = Xd.clone()
    bad[3, 5] = float("inf")
    for fn in (harp.harp_apply, harp.harp_apply_transpose):
        good, got = fn(plan, Xd), fn(plan, bad)
        assert not torch.isfinite(got[3]).all()
        keep = [r for r in range(Xd.shape[0]) if r != 3]
        assert torch.equal(got[keep], good[keep])
    plan.destroy()
