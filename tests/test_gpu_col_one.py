"""Column passes of a single stage (rotation along the row index of a matrix): every radix they are
built for, four-column accesses at their edges, and the fused radix-2 stage of the row side."""
import sys

import numpy as np
import pytest

from oracle import harp_oracle as ho
from paper_2605_29843_amd import inputs as gi
from parity_util import assert_parity, to_device, to_host64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def harp():
    import torch
    assert torch.cuda.is_available()
    from paper_2605_29843_amd import harp as h
    return h


def _plan(harp, d, radices, rng):
    blocks, signs = gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng)
    return harp.Plan(d, radices, blocks, signs), (d, radices, blocks, signs)


def _references(W64, u, v=None):
    """U^T W V and U W V^T in float64."""
    E = np.eye(u[0])
    fwd, inv = ho.apply_transpose_staged(E, *u) @ W64, ho.apply_staged(E, *u) @ W64
    if v is not None:
        fwd, inv = ho.apply_staged(fwd, *v), ho.apply_transpose_staged(inv, *v)
    return fwd, inv


# [b]: the one pass of the plan (stride 1); [8, 8, b]: b = 4 .. 8 gives passes of 8 and 8 b rows.
# Columns: one access, a workgroup's 1024 plus a remainder, and 70: no multiple of four (tile kernel)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("radices", [[2], [3], [4], [5], [6], [7], [8], [8, 8, 7], [8, 8, 8]])
@pytest.mark.parametrize("cols", [4, 1028, 70])
def test_single_stage_column_pass(harp, radices, cols, dtype):
    import torch
    do = int(np.prod(radices))
    rng = np.random.default_rng(do + cols)
    pu, u = _plan(harp, do, radices, rng)
    W = rng.standard_normal((do, cols)).astype(np.float32)
    if dtype == "bf16":
        W = gi.round_to_bf16(W)
    fwd, inv = _references(W.astype(np.float64), u)
    print("single-stage column pass", radices, cols, dtype, file=sys.stderr, flush=True)
    # rows at a pitch and start that keep (8, 0) or break (3, 1) the accesses of four columns
    for pad, off in ((0, 0), (8, 0), (3, 1)):
        big = torch.full((do, cols + pad + off), 7.0, device="cuda", dtype=to_device(W, dtype).dtype)
        out_big = big.clone()
        win, wout = big[:, off:off + cols], out_big[:, off:off + cols]
        win.copy_(to_device(W, dtype))
        harp.harp_rotate_weight(pu, None, win, wout)
        assert_parity(to_host64(wout.contiguous()), fwd, dtype, "U^T W")
        assert bool((out_big[:, :off] == 7.0).all()) and bool((out_big[:, off + cols:] == 7.0).all())
        inv_out = harp.harp_rotate_weight_inverse(pu, None, to_device(W, dtype))
        assert_parity(to_host64(inv_out), inv, dtype, "U W")
    pu.destroy()


# row side of two on-chip chunks and one streamed radix-2 stage on the top digit
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ru,rv", [([8, 8, 7], [8, 8, 8, 8, 2]), ([8, 8, 7], [2] * 13), ([3], [8, 8, 8, 8, 2]),
                                   ([8, 8, 8, 8], [8, 8, 8, 8, 2])])   # the last: passes of 64 rows, not fused
def test_single_stage_column_pass_with_radix2_row_stage(harp, ru, rv, dtype):
    import torch
    do, di = int(np.prod(ru)), int(np.prod(rv))
    rng = np.random.default_rng(do + di)
    pu, u = _plan(harp, do, ru, rng)
    pv, v = _plan(harp, di, rv, rng)
    W = (rng.standard_normal((do, di)) * 0.1).astype(np.float32)
    if dtype == "bf16":
        W = gi.round_to_bf16(W)
    print("with a radix-2 row stage", ru, rv, dtype, file=sys.stderr, flush=True)
    Wd = to_device(W, dtype)
    rows = sorted({0, 1, do // 3, do - 1})
    E = np.zeros((len(rows), do))
    E[np.arange(len(rows)), rows] = 1.0
    W64 = W.astype(np.float64)
    fwd = ho.apply_staged(ho.apply_transpose_staged(E, *u) @ W64, *v)
    inv = ho.apply_transpose_staged(ho.apply_staged(E, *u) @ W64, *v)
    out, back = harp.harp_rotate_weight(pu, pv, Wd), harp.harp_rotate_weight_inverse(pu, pv, Wd)
    idx = torch.tensor(rows).cuda()
    assert_parity(to_host64(out[idx]), fwd, dtype, "U^T W V rows")
    assert_parity(to_host64(back[idx]), inv, dtype, "U W V^T rows")
    W2 = Wd.clone()
    harp.harp_rotate_weight(pu, pv, W2, W2)
    assert torch.equal(W2, out)
    pu.destroy()
    pv.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ru,rv,cols", [([8], None, 128), ([7], None, 132), ([8, 8, 8, 7], None, 256), ([8, 8, 7, 4], None, 128),
                                        ([8], [8, 8, 8, 5, 2], 5120)])
def test_rows_on_four_byte_boundaries(ru, rv, cols, dtype):
    """Rows of a view: every float32 pitch, every even bf16 one.  The same bits as rows side by side, and
    nothing beside them is written."""
    import torch
    from paper_2605_29843_amd import harp
    do = int(np.prod(ru))
    rng = np.random.default_rng(do + cols)
    pu = harp.Plan(do, ru, gi.make_blocks(do, ru, "qr", rng), gi.make_signs(do, rng))
    pv = harp.Plan(cols, rv, gi.make_blocks(cols, rv, "qr", rng), gi.make_signs(cols, rng)) if rv else None
    W = to_device(gi.round_to_bf16(rng.standard_normal((do, cols)).astype(np.float32)), dtype)
    unit = 1 if dtype == "f32" else 2

    def view(pad, off):
        big = torch.full((do * (cols + pad) + off,), 7.0, device="cuda", dtype=W.dtype)
        return big[off:].view(do, cols + pad), big[:off]

    for fn in (harp.harp_rotate_weight, harp.harp_rotate_weight_inverse):
        # (the first: rows on 16-byte boundaries in float32)
        ref = None
        for pi, oi, po, oo in ((4, 0, 4, 0), (unit, 0, unit, unit), (3 * unit, unit, 8, 0), (8, 0, unit, 3 * unit)):
            print("rows on four-byte boundaries", ru, rv, dtype, fn.__name__, pi, oi, po, oo, file=sys.stderr, flush=True)
            src, dst = view(pi, oi)[0], view(po, oo)
            src[:, :cols] = W
            fn(pu, pv, src[:, :cols], dst[0][:, :cols])
            got = dst[0][:, :cols].clone()
            assert bool((dst[0][:, cols:] == 7).all()) and bool((dst[1] == 7).all())
            ref = got if ref is None else ref
            if rv is None:
                assert torch.equal(got, ref), (pi, oi, po, oo)
            else:   # plan_V's kernels follow the alignment: two results, each rounded to bf16 (2^-9) or by float32 sums
                assert float((got.double() - ref.double()).norm() / ref.double().norm()) < (1e-6 if dtype == "f32" else 4e-3)
    pu.destroy()
    if pv:
        pv.destroy()
