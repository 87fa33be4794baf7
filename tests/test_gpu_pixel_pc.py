"""Pixel-resolution phase correlation (Eq. 4-1 on full-resolution luma) through the C ABI
against the oracle: the response surface element by element, the integer peak exactly,
the sub-pixel displacement to 1e-9 px, and the selection with align_pixel bit-exact
(strict harness, no tolerated decision mismatch)."""
import numpy as np
import pytest
import torch

import fcdata
from oracle import select as osel
from tests import fcutil

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fc():
    import paper_2604_24391_amd as fc
    fc.lib()
    return fc


def ctx_for(fc, B, H, W):
    return fc.Context(fc.Caps(max_batch=B, max_height=H, max_width=W, max_tokens=1024,
                              max_seq=64, max_d_model=64, max_ffn=64, max_qkv=64))


def run_pc(fc, ctx, prev, cur):
    B, _, H, W = cur.shape
    sp = torch.empty(B, 2, dtype=torch.float64, device="cuda")
    pk = torch.empty(B, 2, dtype=torch.int32, device="cuda")
    rs = torch.empty(B, H, W, dtype=torch.float64, device="cuda")
    fc.fc_phase_correlate(ctx, None if prev is None else torch.from_numpy(prev).cuda(),
                          torch.from_numpy(cur).cuda(), sp, pk, rs)
    torch.cuda.synchronize()
    return sp.cpu().numpy(), pk.cpu().numpy(), rs.cpu().numpy()


def compare_pc(prev, cur, sp, pk, rs):
    for b in range(cur.shape[0]):
        yp = osel.luma(prev[b]) if prev is not None else np.zeros(cur.shape[2:])
        (di, dj), (pi, pj), r = osel.pixel_phase_correlation(yp, osel.luma(cur[b]))
        np.testing.assert_allclose(rs[b], r, rtol=0, atol=1e-9 * max(1.0, np.abs(r).max()),
                                   err_msg=f"pair {b}: response")
        assert tuple(pk[b]) == (pi, pj), f"pair {b}: peak {tuple(pk[b])} vs {(pi, pj)}"
        np.testing.assert_allclose(sp[b], (di, dj), rtol=0, atol=1e-9, err_msg=f"pair {b}")


@pytest.mark.parametrize("H,W", [(28, 56), (112, 224), (224, 224), (448, 448), (896, 448),
                                 (14, 896)])
def test_surface_peak_and_shift_random_rolls(fc, H, W):
    """Random frames rolled by random (also fractional, band-limited) amounts, at every
    transform length the kernels are built for."""
    rng = np.random.default_rng(H * 1000 + W)
    B = 3
    prev = rng.random((B, 3, H, W)).astype(np.float32)
    cur = np.empty_like(prev)
    for b in range(B):
        cur[b] = np.roll(prev[b], (int(rng.integers(-H // 3, H // 3 + 1)),
                                   int(rng.integers(-W // 3, W // 3 + 1))), axis=(1, 2))
    # the last pair: a fractional shift through the Fourier shift theorem
    u = np.fft.fftfreq(H)[:, None]
    v = np.fft.fftfreq(W)[None, :]
    ramp = np.exp(-2j * np.pi * (u * 2.3 + v * -1.6))
    cur[-1] = np.clip(np.real(np.fft.ifft2(np.fft.fft2(prev[-1]) * ramp)), 0, 1).astype(np.float32)
    ctx = ctx_for(fc, B, H, W)
    try:
        sp, pk, rs = run_pc(fc, ctx, prev, cur)
    finally:
        ctx.close()
    compare_pc(prev, cur, sp, pk, rs)


@pytest.mark.parametrize("H,W", [(14, 14), (28, 28), (56, 14), (14, 56), (112, 112), (56, 224),
                                 (224, 28), (448, 896), (896, 896), (896, 14)])
def test_every_transform_length_both_ways(fc, H, W):
    """Every length as rows and as columns (one to 32 sequences in a wave, the last strip of
    columns 1, 5, 7 or 8 wide), more items than one; the shift and peak are the same bytes
    whether or not the surface is asked for."""
    rng = np.random.default_rng(H * 1009 + W)
    B = 2
    prev = rng.random((B, 3, H, W)).astype(np.float32)
    cur = np.stack([np.roll(prev[b], (H // 5 + b, -(W // 4)), axis=(1, 2)) for b in range(B)])
    cur = np.clip(cur + rng.normal(0, 0.02, cur.shape), 0, 1).astype(np.float32)
    ctx = ctx_for(fc, B, H, W)
    try:
        sp, pk, rs = run_pc(fc, ctx, prev, cur)
        sp2 = torch.empty(B, 2, dtype=torch.float64, device="cuda")
        fc.fc_phase_correlate(ctx, torch.from_numpy(prev).cuda(), torch.from_numpy(cur).cuda(), sp2)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    compare_pc(prev, cur, sp, pk, rs)
    np.testing.assert_array_equal(sp, sp2.cpu().numpy())


@pytest.mark.parametrize("axis", [2, 3])
@pytest.mark.parametrize("H,W,period", [(224, 224, 1), (448, 448, 1), (448, 448, 2), (448, 448, 7),
                                        (448, 448, 14), (448, 448, 56), (448, 224, 2),
                                        (224, 448, 7), (448, 224, 7), (896, 112, 2)])
def test_frames_that_repeat_along_an_axis(fc, H, W, period, axis):
    """Bands (period 1) and tiles of random content have a surface of equal maxima: the first of
    them in row order is the peak, as in the oracle, whatever the rounding of the others."""
    rng = np.random.default_rng(H * 7 + W + 100 * period + axis)
    B = 8
    tile = rng.random((B, 3, period, W) if axis == 2 else (B, 3, H, period)).astype(np.float32)
    reps = (1, 1, H // period, 1) if axis == 2 else (1, 1, 1, W // period)
    prev = np.tile(tile, reps)
    cur = np.roll(prev, 5, axis=5 - axis).copy()
    ctx = ctx_for(fc, B, H, W)
    try:
        sp, pk, rs = run_pc(fc, ctx, prev, cur)
    finally:
        ctx.close()
    compare_pc(prev, cur, sp, pk, rs)


def test_trajectory_pairs_and_missing_previous(fc):
    """Consecutive 448 x 448 frames of the benchmark trajectory, and batches without a
    previous frame or with an all-black one (shift 0, zero surface, as in the oracle)."""
    frames = fcdata.episode_frames(2024, size=448, n_frames=9)
    prev, cur = frames[:-1], frames[1:]
    ctx = ctx_for(fc, 8, 448, 448)
    try:
        sp, pk, rs = run_pc(fc, ctx, prev, cur)
        compare_pc(prev, cur, sp, pk, rs)
        sp0, pk0, rs0 = run_pc(fc, ctx, None, cur[:2])
        sp1, pk1, rs1 = run_pc(fc, ctx, np.zeros_like(cur[:2]), cur[:2])
    finally:
        ctx.close()
    # a missing and an all-black previous frame: zero spectrum, zero surface, shift 0
    for sp_, pk_, rs_ in ((sp0, pk0, rs0), (sp1, pk1, rs1)):
        assert not rs_.any() and not pk_.any() and not sp_.any()


def test_rejects_unsupported_sizes(fc):
    ctx = ctx_for(fc, 1, 448, 448)
    try:
        cur = torch.zeros(1, 3, 420, 448, device="cuda")
        sp = torch.empty(1, 2, dtype=torch.float64, device="cuda")
        with pytest.raises(fc.FcError, match="UNSUPPORTED"):
            fc.fc_phase_correlate(ctx, None, cur, sp)
        big = torch.zeros(2, 3, 448, 448, device="cuda")
        with pytest.raises(fc.FcError, match="CAPACITY"):
            fc.fc_phase_correlate(ctx, None, big, torch.empty(2, 2, dtype=torch.float64,
                                                              device="cuda"))
        prm = fc.SelectParams(merge=2, align_pixel=True)
        out = fc.SelectOut.alloc(1, 1024)
        st = fc.select_state_alloc(1, 448, 448)
        with pytest.raises(fc.FcError, match="UNSUPPORTED"):
            fc.fc_select_carry(ctx, prm, None, torch.zeros(1, 3, 448, 448, device="cuda"), st, out)
    finally:
        ctx.close()


@pytest.mark.parametrize("case", ["trajectory_merge2", "shear_free_merge1"])
def test_selection_with_pixel_alignment(fc, case):
    """fc_select with align_pixel on consecutive trajectory frames, every output against
    the oracle's selection with the same variant (strict: no tolerated mismatch)."""
    if case == "trajectory_merge2":
        frames = fcdata.episode_frames(2024, size=448, n_frames=9)
        prm = fc.SelectParams(merge=2, align_pixel=True)
    else:
        frames = fcdata.episode_frames(99, size=224, n_frames=9, shear=0.0)
        prm = fc.SelectParams(merge=1, align_pixel=True)
    op = fcutil.oracle_select_params(prm)
    B, _, H, W = frames[1:].shape
    ctx = ctx_for(fc, B, H, W)
    try:
        fr = torch.from_numpy(frames).cuda()
        gh, gw = fc.token_grid(H, W, prm)
        out = fc.SelectOut.alloc(B, gh * gw)
        fc.fc_select(ctx, prm, fr[:-1], fr[1:], out)
        torch.cuda.synchronize()
        o = fcutil.select_out_np(out)
    finally:
        ctx.close()
    shifts = set()
    for b in range(B):
        res = osel.select_item(frames[b], frames[b + 1], op)
        mg, esc = fcutil.check_select(o, res, op, b)
        assert not esc, f"pair {b}: {esc}"
        shifts.add(res.shift)
    assert len(shifts) > 1          # the trajectory exercises several displacements


def test_noalloc_with_pixel_alignment(fc):
    """fc_select_noalloc with align_pixel gives the bytes fc_select gives."""
    frames = fcdata.episode_frames(5, size=224, n_frames=3)
    prm = fc.SelectParams(merge=2, align_pixel=True)
    fr = torch.from_numpy(frames).cuda()
    ctx = ctx_for(fc, 2, 224, 224)
    try:
        a = fc.SelectOut.alloc(2, 64)
        b = fc.SelectOut.alloc(2, 64)
        fc.fc_select(ctx, prm, fr[:-1], fr[1:], a)
        fc.fc_select_noalloc(prm, fr[:-1], fr[1:], b)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    oa, ob = fcutil.select_out_np(a), fcutil.select_out_np(b)
    for k in oa:
        np.testing.assert_array_equal(oa[k], ob[k], err_msg=k)


# ------------------------------------------------------ rotation (log-polar spectra)
def rotated_pair(size, angle, roll):
    """A shear-free trajectory frame and the same frame rotated by `angle` about its
    centre (per channel, bilinear) and rolled by `roll` pixels."""
    prev = fcdata.episode_frames(11, size=size, n_frames=1, shear=0.0)[0]
    cur = np.stack([np.roll(osel.rotate_image(prev[c].astype(np.float64), -angle), roll,
                            axis=(0, 1)) for c in range(3)]).astype(np.float32)
    return prev, cur


@pytest.mark.parametrize("size", [224, 448])
def test_rotation_against_oracle(fc, size):
    """fc_phase_correlate_rotation on pairs rotated by 0.0 / 0.06 / -0.12 rad and moved:
    angle to 1e-8 rad and the centre's displacement to 1e-6 px of the oracle's."""
    pairs = [rotated_pair(size, a, r) for a, r in ((0.0, (3, -7)), (0.06, (0, 0)),
                                                   (-0.12, (-11, 5)))]
    prev = np.stack([p for p, _ in pairs])
    cur = np.stack([c for _, c in pairs])
    B = len(pairs)
    ctx = ctx_for(fc, B, size, size)
    try:
        sp = torch.empty(B, 2, dtype=torch.float64, device="cuda")
        ang = torch.empty(B, dtype=torch.float64, device="cuda")
        fc.fc_phase_correlate_rotation(ctx, torch.from_numpy(prev).cuda(),
                                       torch.from_numpy(cur).cuda(), sp, ang)
        torch.cuda.synchronize()
        sp, ang = sp.cpu().numpy(), ang.cpu().numpy()
    finally:
        ctx.close()
    for b in range(B):
        a_o, d_o, _ = osel.rotation_phase_correlation(osel.luma(prev[b]), osel.luma(cur[b]))
        assert abs(ang[b] - a_o) < 1e-8, (b, ang[b], a_o)
        np.testing.assert_allclose(sp[b], d_o, rtol=0, atol=1e-6, err_msg=f"pair {b}")


def test_selection_with_rotation(fc):
    """fc_select with align_pixel and align_rotation on rotated-and-moved pairs and on
    trajectory pairs, bit-exact against the oracle's selection (strict)."""
    rot = [rotated_pair(224, a, r) for a, r in ((0.08, (28, 0)), (-0.05, (0, -30)))]
    traj = fcdata.episode_frames(99, size=224, n_frames=3)
    prev = np.concatenate([np.stack([p for p, _ in rot]), traj[:-1]])
    cur = np.concatenate([np.stack([c for _, c in rot]), traj[1:]])
    prm = fc.SelectParams(merge=2, align_pixel=True, align_rotation=True)
    op = fcutil.oracle_select_params(prm)
    B = prev.shape[0]
    ctx = ctx_for(fc, B, 224, 224)
    try:
        out = fc.SelectOut.alloc(B, 64)
        fc.fc_select(ctx, prm, torch.from_numpy(prev).cuda(), torch.from_numpy(cur).cuda(), out)
        torch.cuda.synchronize()
        o = fcutil.select_out_np(out)
    finally:
        ctx.close()
    for b in range(B):
        res = osel.select_item(prev[b], cur[b], op)
        mg, esc = fcutil.check_select(o, res, op, b)
        assert not esc, f"pair {b}: {esc}"


def test_rotation_rejects_small_frames(fc):
    ctx = ctx_for(fc, 1, 448, 448)
    try:
        sp = torch.empty(1, 2, dtype=torch.float64, device="cuda")
        with pytest.raises(fc.FcError, match="UNSUPPORTED"):
            fc.fc_phase_correlate_rotation(ctx, None, torch.zeros(1, 3, 14, 28, device="cuda"), sp)
        out = fc.SelectOut.alloc(1, 4)
        with pytest.raises(fc.FcError, match="INVALID_ARG"):
            fc.fc_select(ctx, fc.SelectParams(merge=1, align_rotation=True), None,
                         torch.zeros(1, 3, 28, 28, device="cuda"), out)
    finally:
        ctx.close()
