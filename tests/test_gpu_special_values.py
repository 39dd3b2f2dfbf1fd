"""Infinities, NaN and subnormal numbers through the kernels on the float32 matrix instruction (chains of rows, column
passes of two stages and of 512 rows) and the single-stage column kernel."""
import sys

import numpy as np
import pytest

from paper_2605_29843_amd import inputs as gi
from parity_util import to_device

pytestmark = pytest.mark.gpu

COLUMNS = [[8], [8, 8], [8, 7], [7, 4], [2] * 6, [8, 8, 8], [8, 8, 8, 7]]


def _plan(radices, seed=0):
    from paper_2605_29843_amd import harp
    d = int(np.prod(radices))
    rng = np.random.default_rng(d + seed)
    return d, harp.Plan(d, radices, gi.make_blocks(d, radices, "qr", rng), gi.make_signs(d, rng))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("radices", COLUMNS)
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_columns_do_not_mix(radices, value, dtype):
    """What is not finite stays in its column, whichever tile of 32 or 128 columns that shares with others."""
    import torch
    from paper_2605_29843_amd import harp
    d, plan = _plan(radices)
    rng = np.random.default_rng(1)
    W = to_device(gi.round_to_bf16(rng.standard_normal((d, 160)).astype(np.float32)), dtype)
    bad, cols = W.clone(), [0, 33, 130]
    for k, c in enumerate(cols):
        bad[(5 * k + 3) % d, c] = value
    keep = [c for c in range(160) if c not in cols]
    for fn in (harp.harp_rotate_weight, harp.harp_rotate_weight_inverse):
        print("columns do not mix", radices, value, dtype, fn.__name__, file=sys.stderr, flush=True)
        good, got = fn(plan, None, W), fn(plan, None, bad)
        assert torch.equal(got[:, keep], good[:, keep])
        assert not torch.isfinite(got[:, cols]).all(dim=0).any()
    plan.destroy()


@pytest.mark.parametrize("radices,rotate", [([8, 8, 8, 8], False), ([8, 8, 8, 4], False), ([8, 8, 8, 8, 7], False)] +
                         [(r, True) for r in COLUMNS])
def test_subnormal_numbers(radices, rotate):
    """Results of integers below 128 times a power of two that makes them subnormal: not flushed.  A float32 sum
    rounds by half a unit of 2^-149 per product, at most eight per stage, and later stages at most add
    sqrt(8) times an error; 64 units per stage bound that.  bf16: the results are around the least normal number."""
    import torch
    from paper_2605_29843_amd import harp
    d, plan = _plan(radices)
    g = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randint(-127, 128, (d, 130) if rotate else (9, d), device="cuda", generator=g).float()
    fns = [lambda x, f=f: f(plan, None, x) for f in (harp.harp_rotate_weight, harp.harp_rotate_weight_inverse)] if rotate \
        else [lambda x, f=f: f(plan, x) for f in (harp.harp_apply, harp.harp_apply_transpose)]
    for fn in fns:
        print("subnormal numbers", radices, rotate, file=sys.stderr, flush=True)
        ref = fn(X).double() * 2.0 ** -140
        assert float(ref.abs().median()) > 1e-41
        assert float((fn(X * 2.0 ** -140).double() - ref).abs().max()) <= 64 * len(radices) * 2.0 ** -149
        ref = fn(X).double() * 2.0 ** -130
        got = fn((X * 2.0 ** -130).bfloat16()).double()
        assert bool(((got - ref).abs() <= ref.abs() * 2.0 ** -8 + 2.0 ** -133).all())
    plan.destroy()
