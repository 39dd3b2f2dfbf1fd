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
    assert plan.kernel_name(8, harp.HARP_BF16 if dtype == "bf16" else harp.HARP_F32) == \
        ("chain_radix8" if not top else "split_chain_stream" if d // np.prod(top[1:], dtype=int) > 4096
         else "split_chunk_stream")   # (a fifth stage that still fits the chunk is no chain: 1536 or 2048 times 2)
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ru", [[8, 3], [7, 4], [5, 11]])     # 24 and 28 rows along the columns, 55 by way of the transpose
@pytest.mark.parametrize("r4", [3, 4, 5, 6, 7, 8])
def test_rotation_with_a_chain_on_whole_rows(r4, ru, dtype):
    """plan_V is one chain: bf16 rows in, float32 rows out, in both directions."""
    from paper_2605_29843_amd import harp
    rv = [8, 8, 8, r4]
    do, cols = int(np.prod(ru)), int(np.prod(rv))
    rng = np.random.default_rng(do + cols)
    bu, su = gi.make_blocks(do, ru, "qr", rng), gi.make_signs(do, rng)
    bv, sv = gi.make_blocks(cols, rv, "qr", rng), gi.make_signs(cols, rng)
    pu, pv = harp.Plan(do, ru, bu, su), harp.Plan(cols, rv, bv, sv)
    print("rotation with a chain", ru, rv, dtype, file=sys.stderr, flush=True)
    W = rng.standard_normal((do, cols)).astype(np.float32)
    if dtype == "bf16":
        W = gi.round_to_bf16(W)
    Wd, W64 = to_device(W, dtype), W.astype(np.float64)
    for fn, rows_fn in ((harp.harp_rotate_weight, ho.apply_staged), (harp.harp_rotate_weight_inverse, ho.apply_transpose_staged)):
        M = rows_fn(W64, cols, rv, bv, sv)
        ref = rows_fn(np.ascontiguousarray(M.T), do, ru, bu, su).T
        rho = np.linalg.norm(M, axis=0, keepdims=True) / np.sqrt(do)
        assert_parity(to_host64(fn(pu, pv, Wd)), ref, dtype, fn.__name__, rho=rho)
    pu.destroy()
    pv.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("radices,counts", [([8, 8, 8, r], (1, 2, 4, 5, 7, 8, 13)) for r in range(3, 9)] +
                         [([8, 8, 8, 7, 4], (1, 3, 6, 9)), ([8, 8, 8, 8, 7], (1, 6)),
                          # the last batch in tiles of four rows on 256 compute units, and the first in tiles of eight
                          ([8, 8, 8, 3], (1024, 1025)), ([8, 8, 8, 5, 2], (512, 513))])
def test_tiles_of_four_and_eight_rows(radices, counts, dtype):
    """The same sums in the same order whatever the tile: rows per tile given (three, eight) and chosen."""
    import torch
    from paper_2605_29843_amd import harp
    d = int(np.prod(radices))
    rng = np.random.default_rng(d)
    blocks, signs = gi.make_blocks(d, radices, "qr", rng), gi.make_signs(d, rng)
    plan = harp.Plan(d, radices, blocks, signs)
    for n in counts:
        print("tiles of four and eight rows", radices, dtype, n, file=sys.stderr, flush=True)
        X = rng.standard_normal((n, d)).astype(np.float32)
        X = gi.round_to_bf16(X) if dtype == "bf16" else X
        Xd = to_device(X, dtype)
        for fn, oracle in ((harp.harp_apply, ho.apply_staged), (harp.harp_apply_transpose, ho.apply_transpose_staged)):
            outs = []
            for rows in (0, 3, 8):
                plan.set_rows_per_tile(rows)
                Y = torch.full((n + 1, d), 7.0, dtype=Xd.dtype, device="cuda")
                outs.append(fn(plan, Xd, Y[:n]))
                assert bool((Y[n] == 7).all())
            assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]), (n, fn.__name__)
            some = np.unique(np.linspace(0, n - 1, 9).astype(int))
            assert_parity(to_host64(outs[2])[some], oracle(X[some], d, radices, blocks, signs), dtype, f"{fn.__name__} n={n}")
    plan.destroy()


# The stage above the chunk on the way in (transposed, not in place): its radices 2 .. 4 over every last radix of a chain, rows
# that fill the last tile of four or eight and rows that do not, pitches; against the oracle, and against the same call in place, which
# takes two launches (the same sums in the same order: equal bits).
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("r4,top", [(r4, top) for r4 in range(3, 9) for top in (2, 3, 4)
                                    if 512 * r4 * top > 4096])   # (shorter rows are one chunk of other radices)
def test_chain_takes_the_stage_above_along(r4, top, dtype):
    import torch
    from paper_2605_29843_amd import harp
    radices = [8, 8, 8, r4, top]
    d = int(np.prod(radices))
    rng = np.random.default_rng(d)
    kind = "qr" if r4 % 2 else "generic"
    blocks, signs = gi.make_blocks(d, radices, kind, rng), gi.make_signs(d, rng)
    plan = harp.Plan(d, radices, blocks, signs)
    for n in (1, 7, 1024 // top + 8, 1024 // top + 13):   # tiles of four rows; more of them than compute units: of eight
        print("chain with the stage above", radices, n, dtype, file=sys.stderr, flush=True)
        X = rng.standard_normal((n, d)).astype(np.float32)
        if dtype == "bf16":
            X = gi.round_to_bf16(X)
        Xd = to_device(X, dtype)
        wide = torch.zeros(n, d + 16, dtype=Xd.dtype, device="cuda")
        got = harp.harp_apply_transpose(plan, Xd, wide[:, 8:8 + d])
        two = Xd.clone()
        harp.harp_apply_transpose(plan, two, two)
        assert torch.equal(got, two)
        assert bool((wide[:, :8] == 0).all()) and bool((wide[:, 8 + d:] == 0).all())
        rows = np.unique(np.r_[0:min(8, n), max(n - 14, 0):n])
        mag = summand_magnitude(X[rows], d, radices, blocks, True) if kind == "generic" else None
        assert_parity(to_host64(got)[rows], ho.apply_transpose_staged(X[rows], d, radices, blocks, signs), dtype,
                      f"transposed n={n}", mag=mag)
    plan.destroy()


def test_in_place_call_is_captured_after_one_out_of_place():
    """Out of place a transposed call with a stage above the chain needs no intermediate; in place it does.  Running the
    plan once either way is enough for a captured call in place."""
    import torch
    from paper_2605_29843_amd import harp
    d, radices, n = 8192, [8, 8, 8, 8, 2], 70
    rng = np.random.default_rng(9)
    plan = harp.Plan(d, radices, gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng))
    X = torch.randn(n, d, device="cuda")
    Y, Z = torch.zeros_like(X), X.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        harp.harp_apply_transpose(plan, X, Y, side)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            harp.harp_apply_transpose(plan, Z, Z, side)
    for _ in range(3):
        Z.copy_(X)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(Z, Y)
    plan.destroy()
