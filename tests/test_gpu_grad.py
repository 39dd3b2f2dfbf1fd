"""GPU parity of harp_grad_blocks (gradient through Y = X U with respect to the blocks and X)
against the float64 oracle, through the C ABI."""
import sys

import numpy as np
import pytest

from oracle import harp_oracle as ho
from paper_2605_29843_amd import inputs as gi
from parity_util import assert_parity, summand_magnitude, to_device, to_host64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def harp():
    import torch
    assert torch.cuda.is_available()
    from paper_2605_29843_amd import harp as h
    return h


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def assert_dk_parity(dK, ref, X, G, what):
    """dK is a float32 sum of n products of float32 numbers.  Per entry the oracle's value is
    bounded by sqrt(sum x^2 sum g^2) <= ||X||_max-col ||G||_max-col; the float32 path (one rounding
    per product and per partial sum, chunks of <= 32..n/128 rows, then <= 128 chunk sums) stays
    within 2e-5 of that scale for the n used here, and must be finite.  With non-orthogonal blocks
    the inner activations x_t and gradients g_t are no longer of the size of X and G; the largest
    entry of the stage's own reference then joins the scale."""
    scale = float(np.sqrt((X.astype(np.float64) ** 2).sum(axis=0).max() *
                          (G.astype(np.float64) ** 2).sum(axis=0).max()))
    for t, (a, r) in enumerate(zip(dK, ref)):
        a = a.detach().cpu().numpy().astype(np.float64)
        assert a.shape == r.shape, (a.shape, r.shape)
        assert np.all(np.isfinite(a))
        err = np.abs(a - r)
        tol = 2e-5 * max(scale, float(np.abs(r).max())) + 1e-5 * np.abs(r)
        assert np.all(err <= tol), f"{what}: stage {t}: max err {err.max():.3e} vs tol {tol.min():.3e}"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,radices,n,kind", [
    (256, [2] * 8, 64, "orth"), (240, [5, 6, 8], 37, "orth"), (96, [3, 2, 2, 2, 4], 1, "generic"),
    (1024, [8, 8, 4, 4], 200, "orth"), (672, [7, 2, 2, 2, 2, 2, 3], 33, "generic"),
    (4096, [2] * 12, 130, "orth"),
    # a stage of radix above 8 (leftover prime): first, last, in the middle, with signs on it
    (44, [4, 11], 9, "generic"), (344, [2, 2, 2, 43], 70, "orth"), (572, [13, 4, 11], 21, "generic"),
    (1376, [2] * 5 + [43], 130, "orth"), (128, [2, 64], 5, "generic"),
    # ... at a stride that is a multiple of 16, in the middle: the stage and the gradient passed
    # back through it both run on the matrix cores
    (704, [4, 4, 11, 2, 2], 50, "generic"), (1408, [2] * 4 + [11, 8], 33, "orth"),
    (320, [4, 4, 20], 75, "generic"), (1024, [2, 2, 2, 2, 64], 12, "orth")])
def test_grad_blocks_matches_the_oracle(harp, d, radices, n, kind, dtype):
    import torch
    rng = np.random.default_rng(d + n)
    blocks = gi.make_blocks(d, radices, kind, rng)
    signs = gi.make_signs(d, rng)
    X = rng.standard_normal((n, d)).astype(np.float32)
    G = rng.standard_normal((n, d)).astype(np.float32)
    if dtype == "bf16":
        X, G = gi.round_to_bf16(X), gi.round_to_bf16(G)
    plan = harp.Plan(d, radices, blocks, signs)
    say("grad_blocks", d, radices, n, kind, dtype)
    dK, dX = harp.harp_grad_blocks(plan, to_device(X, dtype), to_device(G, dtype))
    torch.cuda.synchronize()
    rK, rX = ho.grad_blocks(X, G, d, radices, blocks, signs)
    assert_dk_parity(dK, rK, X, G, "dK")
    mag = None
    if kind == "generic":    # the blocks really are non-orthogonal, and the tolerance follows the summands
        assert max(float(np.abs(np.swapaxes(K, 1, 2) @ K - np.eye(K.shape[1])).max()) for K in blocks) > 0.05
        mag = summand_magnitude(G, d, radices, blocks, transpose=True)
    assert_parity(to_host64(dX), rX, dtype, "dX", mag=mag)
    # dX is apply_transpose of G
    Z = harp.harp_apply_transpose(plan, to_device(G, dtype))
    assert_parity(to_host64(Z), rX, dtype, "apply_transpose(G)", mag=mag)
    # the same call again gives the same bits (fixed summation order)
    dK2, _ = harp.harp_grad_blocks(plan, to_device(X, dtype), to_device(G, dtype), want_dX=False)
    torch.cuda.synchronize()
    for a, b in zip(dK, dK2):
        assert torch.equal(a, b)
    plan.destroy()


# Row chunks of the backward kernels: 4, 8, 16 and 32 rows per workgroup of four groups, at the counts
# where the next one is taken (n x workgroups per row = 256, 1024, 4096), with groups and chunks that are
# not full; rows of 128 blocks, of fewer, and of several workgroups with a last one that is not full.
# (assert_dk_parity's bound: at most 16 rows a group here, then up to 129 chunks, so its 2e-5 holds.)
@pytest.mark.parametrize("d,radices,counts", [
    (512, [8, 8, 8], (2, 5, 256, 257, 1024, 1025)), (280, [5, 8, 7], (3, 255, 259, 4097)),
    (2688, [6, 7, 8, 8], (64, 65, 86, 257)), (1536, [3, 4, 2, 8, 8], (51, 129, 1366)),
    (2048, [2] * 11, (33, 63, 129, 513)), (3125, [5] * 5, (52, 205))])
def test_grad_row_chunks(harp, d, radices, counts):
    rng = np.random.default_rng(d)
    kind = "generic" if d % 2 else "orth"
    blocks, signs = gi.make_blocks(d, radices, kind, rng), gi.make_signs(d, rng)
    plan = harp.Plan(d, radices, blocks, signs)
    for n in counts:
        say("grad row chunks", radices, n)
        X, G = rng.standard_normal((n, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
        dK, dX = harp.harp_grad_blocks(plan, to_device(X, "f32"), to_device(G, "f32"))
        rK, rX = ho.grad_blocks(X, G, d, radices, blocks, signs)
        assert_dk_parity(dK, rK, X, G, f"dK, {n} rows")
        mag = summand_magnitude(G, d, radices, blocks, transpose=True) if kind == "generic" else None
        assert_parity(to_host64(dX), rX, "f32", f"dX, {n} rows", mag=mag)
    plan.destroy()


def test_grad_blocks_without_signs_and_with_padded_rows(harp):
    import torch
    d, radices, n = 512, [2, 4, 8, 8], 70
    rng = np.random.default_rng(9)
    blocks = gi.make_blocks(d, radices, "orth", rng)
    X = rng.standard_normal((n, d)).astype(np.float32)
    G = rng.standard_normal((n, d)).astype(np.float32)
    plan = harp.Plan(d, radices, blocks, None)
    bigx = torch.zeros(n, d + 24, device="cuda")
    bigg = torch.zeros(n, d + 8, device="cuda")
    bigx[:, 3:3 + d] = torch.from_numpy(X).cuda()
    bigg[:, 5:5 + d] = torch.from_numpy(G).cuda()
    dK, dX = harp.harp_grad_blocks(plan, bigx[:, 3:3 + d], bigg[:, 5:5 + d])
    torch.cuda.synchronize()
    rK, rX = ho.grad_blocks(X, G, d, radices, blocks, None)
    assert_dk_parity(dK, rK, X, G, "dK (views)")
    assert_parity(to_host64(dX), rX, "f32", "dX (views)")
    plan.destroy()


def test_grad_blocks_empty_batch(harp):
    import torch
    d, radices = 64, [4, 4, 4]
    rng = np.random.default_rng(1)
    plan = harp.Plan(d, radices, gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng))
    X = torch.empty(0, d, device="cuda")
    dK, dX = harp.harp_grad_blocks(plan, X, X.clone())
    torch.cuda.synchronize()
    assert all(float(k.abs().max()) == 0.0 for k in dK) and dX.shape == (0, d)
    plan.destroy()


def test_grad_blocks_llama7b_shape_sampled(harp):
    """2048 x 4096 bf16, 12 radix-2 stages (the benchmark's shape): every block of every stage
    against the oracle on the same rows."""
    import torch
    w = gi.workload("llama7b_4096_r2")
    d, radices, n = w["d"], w["radices"], w["n"]
    rng = np.random.default_rng(4)
    X = w["X"]
    G = gi.round_to_bf16((rng.standard_normal((n, d)) * 0.05).astype(np.float32))
    plan = harp.Plan(d, radices, w["blocks"], w["signs"])
    say("grad_blocks full size", n, d)
    dK, dX = harp.harp_grad_blocks(plan, to_device(X, "bf16"), to_device(G, "bf16"))
    torch.cuda.synchronize()
    rK, rX = ho.grad_blocks(X, G, d, radices, w["blocks"], w["signs"])
    assert_dk_parity(dK, rK, X, G, "dK full size")
    rows = np.arange(0, n, 97)
    assert_parity(to_host64(dX)[rows], rX[rows], "bf16", "dX rows")
    plan.destroy()


def assert_dk_accuracy(dK, ref, X, G, d, radices, blocks, signs, what):
    """How far a float32 sum may be from the float64 one where the block decides the scale, not the
    largest column: every entry within 5e-7 of |x_t[:, i]| |g_{t+1}[:, j]| of its own two columns, and
    every stage within 1e-6 of its norm.  One rounding (2^-24 = 6e-8) per product and per sum gives
    about 1e-7 and 2e-7 (measured, with and without the segment, 64 to 20000 rows: at most 1.6e-7
    and 3.3e-7); operands or partial sums of 16 bits would show 2e-3."""
    st = ho.strides(radices)
    x, g = [np.asarray(X, dtype=np.float64) * signs[None, :]], np.asarray(G, dtype=np.float64)
    for t, b in enumerate(radices):
        x.append(ho.stage_apply_rows(x[t].copy(), b, st[t], np.asarray(blocks[t], dtype=np.float64)))
    for t in range(len(radices) - 1, -1, -1):
        b, s = radices[t], st[t]

        def norms(a):   # of the columns, [d / b, b]: block alpha s + beta, coordinate alpha b s + r s + beta
            return np.sqrt((a ** 2).sum(axis=0)).reshape(-1, b, s).transpose(0, 2, 1).reshape(-1, b)
        scale = norms(x[t])[:, :, None] * norms(g)[:, None, :]
        err = np.abs(dK[t].detach().cpu().numpy().astype(np.float64) - ref[t])
        assert np.all(err <= 5e-7 * scale), f"{what}: stage {t}: an entry is {(err / scale).max():.2e} of its columns off"
        rel = np.linalg.norm(err) / np.linalg.norm(ref[t])
        assert rel <= 1e-6, f"{what}: stage {t}: {rel:.2e} of the norm"
        g = ho.stage_apply_rows(g.copy(), b, s, np.asarray(blocks[t], dtype=np.float64), transpose_blocks=True)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,radices,n", [
    # one stage behind the leading segment of 64 coordinates, at the fewest rows it takes
    (128, [2] * 7, 64), (512, [8, 8, 8], 64),
    # ragged runs of rows: a wave with one row, a wave with none, more than one workgroup per group
    (320, [2] * 6 + [5], 65), (704, [8, 8, 11], 71), (2048, [8, 8, 8, 4], 297), (4096, [2] * 12, 1033)])
def test_leading_segment_and_stage_by_stage_agree_with_the_oracle(harp, d, radices, n, dtype):
    """The first 64 coordinates' stages as one segment (n >= 64), rows on boundaries of four elements and
    rows that are not (here: shifted by one element), both against the oracle: within the tolerance of
    every call, and within the one that follows from float32 sums entry by entry."""
    import torch
    rng = np.random.default_rng(7 * d + n)
    blocks, signs = gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng)
    X = rng.standard_normal((n, d)).astype(np.float32)
    X[:, :: 97] *= 20.0
    G = rng.standard_normal((n, d)).astype(np.float32)
    if dtype == "bf16":
        X, G = gi.round_to_bf16(X), gi.round_to_bf16(G)
    plan = harp.Plan(d, radices, blocks, signs)
    say("grad leading segment", d, radices, n, dtype)
    rK, rX = ho.grad_blocks(X, G, d, radices, blocks, signs)
    Xd, Gd = to_device(X, dtype), to_device(G, dtype)
    wide = torch.zeros(n, d + 8, device="cuda", dtype=Xd.dtype)
    wide[:, 1:1 + d] = Xd
    for Xin in (Xd, wide[:, 1:1 + d]):
        dK, dX = harp.harp_grad_blocks(plan, Xin, Gd)
        dK2, none = harp.harp_grad_blocks(plan, Xin, Gd, want_dX=False)
        torch.cuda.synchronize()
        assert none is None
        assert_dk_parity(dK, rK, X, G, "dK")
        assert_dk_accuracy(dK, rK, X, G, d, radices, blocks, signs, "dK")
        assert_parity(to_host64(dX), rX, dtype, "dX")
        for a, b in zip(dK, dK2):
            assert torch.equal(a, b)
    plan.destroy()


# Two passes of one launch behind the leading segment: eight coordinates (one stage, or three of radix 2), then
# 2 .. 8 (one stage, or one, two, three of radix 2), at the end of the plan and with a stage behind them; rows that
# fill a workgroup's chunk, leave a set of four with one row, and leave whole sets empty; tiles of 16 groups that share
# lines with neighbours and that do not.  The last nine: chunks of 48 rows (the fewest rounds on 256 compute units), three steps of
# 16 rows for second passes of two, three and four coordinates, the last chunk's with a step that is not full.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("radices,n", [
    ([8, 8, 8, 2], 64), ([8, 8, 8, 3], 81), ([8, 8, 8, 4], 65), ([8, 8, 8, 5], 97), ([8, 8, 8, 6], 70),
    ([8, 8, 8, 7], 67), ([8, 8, 8, 8], 145), ([2] * 6 + [8, 3], 131), ([2] * 6 + [8, 2, 2], 66), ([2] * 6 + [8, 2], 79),
    ([2] * 10, 96), ([2] * 11, 161), ([2] * 12, 73), ([2] * 9 + [5], 64), ([8, 8] + [2] * 6, 99), ([8, 8, 2, 2, 2, 7], 77),
    ([8, 8, 8, 2, 3], 66), ([2] * 12 + [3], 65), ([8, 8, 8, 5, 2], 83), ([8, 8, 8, 3, 3], 70), ([2] * 6 + [8, 4, 2], 69),
    ([8, 8, 8, 6, 2], 64), ([8, 8, 8, 7, 2], 64),
    ([8, 8, 8, 2], 3001), ([8, 8, 8, 3], 3001), ([8, 8, 8, 4], 3001), ([8, 8, 8, 2, 3], 1501), ([8, 8, 8, 3, 2], 1501),
    ([8, 8, 8, 4, 2], 1501), ([2] * 10 + [5], 1001), ([2] * 9 + [3, 3, 3], 601), ([2] * 11 + [7], 333)])
def test_pairs_of_passes_behind_the_leading_segment(harp, radices, n, dtype):
    d = int(np.prod(radices))
    rng = np.random.default_rng(d + n)
    blocks, signs = gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng)
    X, G = rng.standard_normal((n, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
    if dtype == "bf16":
        X, G = gi.round_to_bf16(X), gi.round_to_bf16(G)
    plan = harp.Plan(d, radices, blocks, signs)
    say("grad pairs of passes", radices, n, dtype)
    dK, dX = harp.harp_grad_blocks(plan, to_device(X, dtype), to_device(G, dtype))
    rK, rX = ho.grad_blocks(X, G, d, radices, blocks, signs)
    assert_dk_parity(dK, rK, X, G, "dK")
    assert_dk_accuracy(dK, rK, X, G, d, radices, blocks, signs, "dK")
    assert_parity(to_host64(dX), rX, dtype, "dX")
    plan.destroy()


# A stage of radix 9 .. 48 at a stride that is a multiple of 16: operand tiles one to three, full and not, steps of 16 rows
# and chunks that are full, short by one and longer by one (one workgroup per compute unit: D / 16 tiles across, so the
# counts beyond 4096 rows of D = 16 take chunks of more than a step), the stage last, in the middle, and twice; chunks added by one
# thread, by four (25 and 33 chunks: the last of them one or none) and by sixteen; chunks that fill the chip twice.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,radices,kind,counts", [
    (144, [4, 4, 9], "generic", (1, 15, 16, 17, 400, 520, 4097, 8200, 33000)), (256, [8, 2, 16], "orth", (31, 4096)), (272, [4, 4, 17], "orth", (33, 4113)),
    (1024, [8, 4, 32], "generic", (16, 130)), (528, [2, 8, 33], "orth", (47, 4100)), (688, [4, 4, 43], "generic", (64, 8193)),
    (768, [8, 2, 48], "orth", (5, 4098)), (11008, [8, 8, 4, 43], "orth", (81, 257)), (1408, [4, 4, 11, 8], "generic", (65,)),
    (1936, [16, 11, 11], "orth", (40,))])
def test_large_radix_on_the_matrix_cores(harp, d, radices, kind, counts, dtype):
    rng = np.random.default_rng(d)
    blocks, signs = gi.make_blocks(d, radices, kind, rng), gi.make_signs(d, rng)
    plan = harp.Plan(d, radices, blocks, signs)
    for n in counts:
        say("grad large radix", radices, n, dtype)
        X, G = rng.standard_normal((n, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
        if dtype == "bf16":
            X, G = gi.round_to_bf16(X), gi.round_to_bf16(G)
        dK, dX = harp.harp_grad_blocks(plan, to_device(X, dtype), to_device(G, dtype))
        rK, rX = ho.grad_blocks(X, G, d, radices, blocks, signs)
        assert_dk_parity(dK, rK, X, G, f"dK, {n} rows")
        if kind == "orth":
            assert_dk_accuracy(dK, rK, X, G, d, radices, blocks, signs, f"dK, {n} rows")
        mag = summand_magnitude(G, d, radices, blocks, transpose=True) if kind == "generic" else None
        assert_parity(to_host64(dX), rX, dtype, f"dX, {n} rows", mag=mag)
    plan.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1, 65, 130])
def test_last_stage_of_large_radix_reads_gradient_rows_at_any_pitch(harp, n, dtype):
    """A last stage of radix above 8 at a stride that is a multiple of 16: G is read
    where it lies (pitch and start on boundaries of four elements) or from a copy (any other); both give the bits of a
    contiguous G."""
    import torch
    d, radices = 1408, [2] * 4 + [8, 11]
    rng = np.random.default_rng(n)
    blocks, signs = gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng)
    plan = harp.Plan(d, radices, blocks, signs)
    Xh, Gh = rng.standard_normal((n, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
    if dtype == "bf16":
        Xh, Gh = gi.round_to_bf16(Xh), gi.round_to_bf16(Gh)
    X, G = to_device(Xh, dtype), to_device(Gh, dtype)
    dK0, dX0 = harp.harp_grad_blocks(plan, X, G)
    ref, ref_dx = ho.grad_blocks(Xh.astype(np.float64), Gh.astype(np.float64), d, radices, blocks, signs)
    assert_dk_parity(dK0, ref, Xh, Gh, "contiguous")
    assert_parity(to_host64(dX0), ref_dx, dtype, "dX")
    for pad, off in ((4, 0), (4, 4), (3, 0), (4, 1)):
        big = torch.zeros(n, d + pad + off, device="cuda", dtype=G.dtype)
        view = big[:, off:off + d]
        view.copy_(G)
        dK, dX = harp.harp_grad_blocks(plan, X, view)
        assert torch.equal(dX, dX0) and all(torch.equal(a, b) for a, b in zip(dK, dK0)), (pad, off)
    plan.destroy()


# plans whose chunks get fewer as n grows: the leading segment's (64 coordinates) where its rows per
# chunk step up by 32, and those of a radix above 8 beyond 16384 rows
@pytest.mark.parametrize("d,radices", [(2048, [2] * 11), (4096, [2] * 12), (5120, [2] * 10 + [5]), (512, [8, 8, 8]),
                                       (704, [8, 8, 11]), (44, [4, 11]), (11008, [8, 8, 4, 43])])
def test_workspace_size_does_not_fall_as_the_batch_grows(harp, d, radices):
    rng = np.random.default_rng(d)
    plan = harp.Plan(d, radices, gi.make_blocks(d, radices, "orth", rng), None)
    sizes = [harp.harp_grad_blocks_workspace_size(plan, n) for n in range(18000)]
    sizes += [harp.harp_grad_blocks_workspace_size(plan, n) for n in range(65535 * 128 - 2, 65535 * 128 + 3)]
    assert all(b >= a for a, b in zip(sizes, sizes[1:]))
    plan.destroy()


def test_workspace_of_a_larger_batch_serves_a_smaller_one(harp):
    import torch
    d, radices = 4096, [2] * 12
    rng = np.random.default_rng(5)
    plan = harp.Plan(d, radices, gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng))
    ws = torch.empty(harp.harp_grad_blocks_workspace_size(plan, 513), dtype=torch.uint8, device="cuda")
    for n in (513, 512, 63):
        X = torch.from_numpy(rng.standard_normal((n, d)).astype(np.float32)).cuda()
        G = torch.from_numpy(rng.standard_normal((n, d)).astype(np.float32)).cuda()
        dK, dX = harp.harp_grad_blocks(plan, X, G, workspace=ws)
        ref, ref_dx = harp.harp_grad_blocks(plan, X, G)
        assert torch.equal(dX, ref_dx) and all(torch.equal(a, b) for a, b in zip(dK, ref))
    plan.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,radices,n", [(128, [2] * 7, 64), (512, [8, 8, 8], 71), (2048, [8, 8, 8, 4], 297),
                                         (704, [8, 8, 11], 130), (1376, [2] * 5 + [43], 65), (4096, [2] * 12, 200),
                                         (512, [8, 8, 8], 63)])
def test_bits_do_not_depend_on_where_the_matrices_lie(harp, d, radices, n, dtype):
    """The same values in views that break the boundaries of four elements or of 16 bytes, for each of
    the matrices and the workspace, with and without dX."""
    import ctypes
    import torch
    rng = np.random.default_rng(3 * d + n)
    plan = harp.Plan(d, radices, gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng))
    X, G = rng.standard_normal((n, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
    if dtype == "bf16":
        X, G = gi.round_to_bf16(X), gi.round_to_bf16(G)
    X, G = to_device(X, dtype), to_device(G, dtype)
    dK0, dX0 = harp.harp_grad_blocks(plan, X, G)
    need = harp.harp_grad_blocks_workspace_size(plan, n)
    ws = torch.empty(need + 64, dtype=torch.uint8, device="cuda")
    code = 0 if dtype == "f32" else 1

    def placed(x, pad, off):
        big = torch.zeros(n, d + pad + off, device="cuda", dtype=x.dtype)
        big[:, off:off + d] = x
        return big[:, off:off + d]

    # (pad, off) of X, G, dX (None: no dX), bytes by which the workspace starts late
    for px, pg, pdx, late in (((8, 1), (0, 0), (0, 0), 0), ((4, 0), (0, 0), (0, 0), 0), ((3, 0), (5, 2), (1, 0), 0),
                              ((0, 0), (8, 1), (8, 1), 0), ((0, 0), (0, 0), (7, 0), 0), ((0, 0), (0, 0), None, 0),
                              ((4, 4), (4, 4), (4, 4), 0), ((0, 0), (0, 0), (0, 0), 4), ((8, 1), (0, 0), None, 12)):
        xv, gv = placed(X, *px), placed(G, *pg)
        dxv = None if pdx is None else placed(torch.full_like(X, 7.0), *pdx)
        dK = [torch.full_like(a, 7.0) for a in dK0]
        ptrs = (ctypes.c_void_p * len(dK))(*[a.data_ptr() for a in dK])
        st = harp.lib.harp_grad_blocks(plan.handle, xv.data_ptr(), xv.stride(0), gv.data_ptr(), gv.stride(0), n, code,
                                       ptrs, None if dxv is None else dxv.data_ptr(),
                                       0 if dxv is None else dxv.stride(0), ws.data_ptr() + late, need,
                                       torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        where = (px, pg, pdx, late)
        assert st == 0, where
        assert all(torch.equal(a, b) for a, b in zip(dK, dK0)), where
        assert dxv is None or torch.equal(dxv, dX0), where
        # nothing beside the rows of dX was written
        if dxv is not None:
            full = torch.as_strided(dxv, (n, dxv.stride(0)), (dxv.stride(0), 1), dxv.storage_offset() - pdx[1])
            assert bool((full[:, :pdx[1]] == 0).all()) and bool((full[:, pdx[1] + d:] == 0).all()), where
    plan.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("radices", [[2] * 12, [8, 8, 8, 4]])
def test_bits_do_not_depend_on_a_pitch_beyond_32_bit_offsets(harp, radices, dtype):
    """Gradient rows 2^25 elements apart and more: read with 64-bit offsets, or copied first."""
    import torch
    d, n = int(np.prod(radices)), 67
    rng = np.random.default_rng(d)
    plan = harp.Plan(d, radices, gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng))
    X, G = torch.randn(n, d, device="cuda"), torch.randn(n, d, device="cuda")
    if dtype == "bf16":
        X, G = X.bfloat16(), G.bfloat16()
    dK0, dX0 = harp.harp_grad_blocks(plan, X, G)
    big = torch.empty(n, (1 << 25) + 8, device="cuda", dtype=G.dtype)
    view = big[:, :d]
    view.copy_(G)
    say("gradient rows far apart", radices, dtype)
    dK, dX = harp.harp_grad_blocks(plan, X, view)
    torch.cuda.synchronize()
    assert torch.equal(dX, dX0) and all(torch.equal(a, b) for a, b in zip(dK, dK0))
    plan.destroy()


# One stage of each way in which block gradients are written: the matrix cores' (9, 16 with one operand tile, 43 with three), the
# pairs' and the first 64 coordinates', a run of radix-2 stages, a single stage, a stride that is no multiple of 16
@pytest.mark.parametrize("d,radices,n", [(144, [4, 4, 9], 20), (256, [8, 2, 16], 33), (688, [4, 4, 43], 65), (512, [8, 8, 8], 64),
                                         (4096, [8, 8, 8, 8], 70), (4096, [2] * 12, 64), (240, [5, 6, 8], 37), (44, [4, 11], 9)])
def test_block_gradients_may_lie_at_any_float(harp, d, radices, n):
    import ctypes
    import torch
    rng = np.random.default_rng(d + n)
    plan = harp.Plan(d, radices, gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng))
    X, G = torch.randn(n, d, device="cuda"), torch.randn(n, d, device="cuda")
    dK0, dX0 = harp.harp_grad_blocks(plan, X, G)
    need = harp.harp_grad_blocks_workspace_size(plan, n)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    for shift in (1, 2, 3):   # one array for all stages, each `shift` floats behind a boundary of 16 bytes
        sizes = [(a.numel() + 7) // 4 * 4 for a in dK0]
        flat = torch.full((sum(sizes) + 4,), 7.0, device="cuda")
        at = [sum(sizes[:t]) + shift for t in range(len(sizes))]
        ptrs = (ctypes.c_void_p * len(dK0))(*[flat.data_ptr() + 4 * a for a in at])
        dX = torch.empty_like(X)
        say("block gradients at", shift, radices, n)
        st = harp.lib.harp_grad_blocks(plan.handle, X.data_ptr(), d, G.data_ptr(), d, n, harp.HARP_F32, ptrs, dX.data_ptr(), d,
                                       ws.data_ptr(), need, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert st == 0 and torch.equal(dX, dX0)
        beside = torch.ones_like(flat, dtype=torch.bool)
        for a, ref in zip(at, dK0):
            assert torch.equal(flat[a:a + ref.numel()], ref.reshape(-1)), shift
            beside[a:a + ref.numel()] = False
        assert bool((flat[beside] == 7.0).all())
    plan.destroy()


# dX written over X or G: a leading segment (radix 2, radix 8), a run of radix-2 stages, a single
# stage at either end, one run and nothing else
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,radices,n", [(512, [2] * 9, 133), (512, [8, 8, 8], 133), (512, [2] * 9, 20), (176, [2] * 4 + [11], 70),
                                         (8, [2] * 3, 300), (240, [5, 6, 8], 37), (11, [11], 5)])
def test_dX_may_be_X_or_G(harp, d, radices, n, dtype):
    import ctypes
    import torch
    rng = np.random.default_rng(d + n)
    plan = harp.Plan(d, radices, gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng))
    X, G = rng.standard_normal((n, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
    if dtype == "bf16":
        X, G = gi.round_to_bf16(X), gi.round_to_bf16(G)
    X, G = to_device(X, dtype), to_device(G, dtype)
    dK0, dX0 = harp.harp_grad_blocks(plan, X, G)
    need = harp.harp_grad_blocks_workspace_size(plan, n)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    for over in ("X", "G"):
        x, g = X.clone(), G.clone()
        out = x if over == "X" else g
        dK = [torch.empty_like(a) for a in dK0]
        ptrs = (ctypes.c_void_p * len(dK))(*[a.data_ptr() for a in dK])
        st = harp.lib.harp_grad_blocks(plan.handle, x.data_ptr(), d, g.data_ptr(), d, n, 0 if dtype == "f32" else 1,
                                       ptrs, out.data_ptr(), d, ws.data_ptr(), need,
                                       torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert st == 0
        assert torch.equal(out, dX0) and all(torch.equal(a, b) for a, b in zip(dK, dK0)), over
    plan.destroy()


def test_four_pairs_of_passes_behind_the_leading_segment(harp):
    """2^22 coordinates, the smallest row with four pairs (ten sums at the end of the call): 64 rows at once against
    the same rows 32 at a time, which go stage by stage, block gradients added."""
    import torch
    radices, n = [8, 8] + [8, 2] * 4, 64
    d = int(np.prod(radices))
    rng = np.random.default_rng(4)
    blocks = [np.tile(gi.qr_blocks(512, b, rng), (d // b // 512, 1, 1)) for b in radices]
    plan = harp.Plan(d, radices, blocks, gi.make_signs(d, rng))
    say("grad", radices, n)
    gen = torch.Generator(device="cuda").manual_seed(7)
    X = torch.randn(n, d, device="cuda", generator=gen)
    G = torch.randn(n, d, device="cuda", generator=gen)
    dK, dX = harp.harp_grad_blocks(plan, X, G)
    halves = [harp.harp_grad_blocks(plan, X[r:r + 32], G[r:r + 32]) for r in (0, 32)]
    # float32 both ways, sums of up to 64 terms after up to 10 stages: about 3e-7 of the norm each
    rel = lambda a, b: float((a.double() - b.double()).norm() / b.double().norm())
    assert rel(dX, torch.cat([h[1] for h in halves])) < 2e-6
    for t in range(len(radices)):
        assert rel(dK[t], halves[0][0][t].double() + halves[1][0][t].double()) < 2e-6, t
    plan.destroy()
