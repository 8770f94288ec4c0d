"""GPU parity: flow field, per-patch motion and gate against the fp64 oracle, through the C ABI.
Tolerance 1e-3 relative + 1e-4 absolute on u, v and Delta P; gate counts may differ only on
patches whose oracle margin to tau_t is inside that tolerance."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import flow as of
from paper_2602_14236_amd import synth

from _util import FLOW_ATOL, FLOW_RTOL, close, lib_config, params

pytestmark = pytest.mark.gpu


def _run(ctx, prev, cur):
    from paper_2602_14236_amd import binding
    h, w, _ = prev.shape
    d_prev, d_cur = torch.from_numpy(prev).cuda(), torch.from_numpy(cur).cuda()
    uv = torch.full((2, h, w), 99.0, dtype=torch.float32, device="cuda")
    dp = torch.full((576,), -1.0, dtype=torch.float32, device="cuda")
    gate = torch.zeros(4, dtype=torch.int32, device="cuda")
    ctx.flow_score(d_prev, d_cur, uv, dp, gate)
    torch.cuda.synchronize()
    g = gate.cpu().numpy()
    return uv.cpu().numpy(), dp.cpu().numpy(), (int(g[0]), float(g[1:2].view(np.float32)[0]), int(g[2]))


def _check(ctx, prev, cur, levels, tau_t=0.5, theta_r=0.9, label=""):
    uv, dp, gate = _run(ctx, prev, cur)
    d = of.flow(prev, cur, levels)
    edp = of.patch_motion(d)
    n, r, red, margin = of.gate(edp, tau_t, theta_r)
    ok_u, ok_v = close(uv[0], d[..., 0]), close(uv[1], d[..., 1])
    err = max(np.abs(uv[0] - d[..., 0]).max(), np.abs(uv[1] - d[..., 1]).max())
    print(f"{label}: max |flow err| {err:.3e}, max |flow| {np.abs(d).max():.3f}, gate margin {margin:.3e}", flush=True)
    assert ok_u.all() and ok_v.all(), f"{(~ok_u).sum() + (~ok_v).sum()} flow values out of tolerance, max err {err}"
    assert close(dp, edp).all()
    # gate: only patches within tolerance of tau_t may be counted differently
    fragile = int(np.count_nonzero(np.abs(edp - tau_t) <= FLOW_ATOL + FLOW_RTOL * tau_t))
    assert abs(gate[0] - n) <= fragile
    if fragile == 0:
        assert gate == (n, float(r), int(red))
    return gate, (n, r, red)


def test_config1_pairs():
    from paper_2602_14236_amd import binding
    ctx = binding.SaliContext(lib_config(params()))
    v = synth.video(1)
    for t in (1, 2, 5):
        _check(ctx, v.frame(t - 1), v.frame(t), 3, label=f"cfg1 {t - 1}->{t}")
    ctx.close()


def test_identical_frames_are_exactly_static():
    from paper_2602_14236_amd import binding
    ctx = binding.SaliContext(lib_config(params()))
    v = synth.video(1)
    uv, dp, gate = _run(ctx, v.frame(2), v.frame(3))          # byte copies
    assert not uv.any() and not dp.any()
    assert gate == (576, 1.0, 1)
    ctx.set_gate_thresholds(0.0, 0.9)                         # strict '<': nothing is below zero
    _, _, gate0 = _run(ctx, v.frame(2), v.frame(3))
    assert gate0 == (0, 0.0, 0)
    ctx.close()


# with three updates a level: 360x640 is too large for updates in one launch and takes 32x32 tiles; 300x500 does so with
# ragged ones; the other levels fit the chip and have their three updates in one launch, 200x200 and 200x264 with ragged
# 16x16 tiles, the smaller ones with 16x8 (test_updates_per_launch goes along both rules)
@pytest.mark.parametrize("h,w,levels", [(24, 24, 1), (50, 77, 2), (97, 131, 3), (360, 640, 3), (200, 264, 5),
                                        (200, 200, 2), (300, 500, 3)])
def test_ragged_sizes_and_level_counts(h, w, levels):
    from paper_2602_14236_amd import binding
    ctx = binding.SaliContext(lib_config(params(h, w, flow_levels=levels)))
    rng = np.random.default_rng(h + w)
    yy, xx = np.meshgrid(np.arange(h + 8, dtype=np.float64), np.arange(w + 8, dtype=np.float64), indexing="ij")
    tex = np.zeros_like(yy)
    for _ in range(8):
        fx, fy = rng.uniform(-0.8, 0.8, 2)
        tex += rng.uniform(0.4, 1.0) * np.sin(fx * xx + fy * yy + rng.uniform(0, 6.28))
    big = np.clip(np.rint(128 + 30 * tex), 0, 255).astype(np.uint8)
    sy, sx = (1, 2) if levels > 1 else (0, 1)
    prev = np.repeat(big[4:4 + h, 4:4 + w, None], 3, axis=2).copy()
    cur = np.repeat(big[4 - sy:4 - sy + h, 4 - sx:4 - sx + w, None], 3, axis=2).copy()
    cur[..., 1] = np.clip(cur[..., 1].astype(np.int64) + rng.integers(-2, 3, (h, w)), 0, 255).astype(np.uint8)
    _check(ctx, prev, cur, levels, label=f"{h}x{w} L{levels}")
    ctx.close()


def test_gate_rational_boundary_on_device():
    """theta_R = 0.75 with exactly 432 static patches: R equals the threshold, so not redundant."""
    from paper_2602_14236_amd import binding
    v = synth.video(5, 60)
    prev, cur = v.frame(57), v.frame(58)
    d = of.flow(prev, cur, 3)
    edp = of.patch_motion(d)
    n, r, red, margin = of.gate(edp, 0.5, 0.75)
    assert n == 432 and not red and margin > 10 * (FLOW_ATOL + FLOW_RTOL * 0.5)
    ctx = binding.SaliContext(lib_config(params(theta_r=0.75)))
    _, _, gate = _run(ctx, prev, cur)
    assert gate == (432, 0.75, 0)
    ctx.set_gate_thresholds(0.5, 0.7499)
    _, _, gate = _run(ctx, prev, cur)
    assert gate[2] == 1
    ctx.close()


@pytest.mark.parametrize("h,w", [(97, 131), (336, 336)])
def test_image_address_does_not_matter(h, w):
    """The gray conversion takes 16 pixels per thread from a 16-byte aligned image and single pixels
    otherwise (and for the last pixels of a frame whose size is no multiple of 16): both give the same bits."""
    from paper_2602_14236_amd import binding
    ctx = binding.SaliContext(lib_config(params(h, w)))
    rng = np.random.default_rng(7)
    prev = rng.integers(0, 256, (h, w, 3), dtype=np.uint8)
    cur = np.roll(prev, (1, 2), axis=(0, 1))
    cur[..., 0] = np.clip(cur[..., 0].astype(np.int64) + rng.integers(-3, 4, (h, w)), 0, 255).astype(np.uint8)
    ref = _run(ctx, prev, cur)
    n = h * w * 3
    for off in (1, 3, 8):
        buf = torch.zeros(2 * n + 64, dtype=torch.uint8, device="cuda")
        d_prev = buf[off:off + n].view(h, w, 3)
        d_cur = buf[n + 32 + off:n + 32 + off + n].view(h, w, 3)
        assert d_prev.data_ptr() % 16 == off
        d_prev.copy_(torch.from_numpy(prev))
        d_cur.copy_(torch.from_numpy(cur))
        uv = torch.full((2, h, w), 99.0, dtype=torch.float32, device="cuda")
        dp = torch.full((576,), -1.0, dtype=torch.float32, device="cuda")
        gate = torch.zeros(4, dtype=torch.int32, device="cuda")
        ctx.flow_score(d_prev, d_cur, uv, dp, gate)
        torch.cuda.synchronize()
        assert np.array_equal(uv.cpu().numpy(), ref[0]) and np.array_equal(dp.cpu().numpy(), ref[1]), off
    ctx.close()


@pytest.mark.parametrize("h,w", [(24, 24), (100, 131), (384, 384), (384, 387), (401, 640)])
def test_patch_motion_of_small_and_large_patches(h, w):
    """Patch motion and the flow planes where the kernel changes its shape (a wave per patch up to 256 pixels a
    patch, a block beyond) and patches are ragged: the motions must be the RMS of the very planes the call
    returns (float64 reference; fp32 sums of at most 4096 terms in 64 or more partial sums: 1e-5), and the gate their count."""
    from paper_2602_14236_amd import binding
    ctx = binding.SaliContext(lib_config(params(h, w, flow_levels=1)))
    rng = np.random.default_rng(h)
    cur = rng.integers(0, 256, (h, w, 3), dtype=np.uint8)
    uv, dp, gate = _run(ctx, np.roll(cur, 1, axis=1), cur)
    assert not np.any(uv == 99.0)
    ys, xs = [i * h // 24 for i in range(25)], [i * w // 24 for i in range(25)]
    sq = (uv.astype(np.float64) ** 2).sum(0)
    exp = np.array([np.sqrt(sq[ys[r]:ys[r + 1], xs[c]:xs[c + 1]].mean()) for r in range(24) for c in range(24)])
    assert np.all(np.abs(dp - exp) <= 1e-5 * exp)
    n = int((dp < 0.5).sum())
    assert gate == (n, float(np.float32(n) / np.float32(576)), int(np.float32(n) / np.float32(576) > np.float32(0.9)))
    ctx.close()


@pytest.mark.parametrize("h,w,levels,shift", [
    (64, 65, 4, 0), (65, 64, 4, 1), (131, 70, 5, 0), (33, 203, 4, 3),      # more than three levels: odd sizes, one tile and a bit
    (400, 401, 2, 0), (402, 400, 3, 2),                                    # large enough for the same path with fewer levels
])
def test_pyramid_in_pairs_of_levels(h, w, levels, shift):
    """Gray image and pyramid two levels at a time: borders of the 64-pixel tiles, last levels without a
    second one, rows that are no multiple of four pixels and images at any address (`shift` bytes into an
    allocation), against the oracle's flow."""
    from paper_2602_14236_amd import binding
    ctx = binding.SaliContext(lib_config(params(h, w, flow_levels=levels)))
    yy, xx = np.mgrid[0:h, 0:w].astype(np.float64)
    rng = np.random.default_rng(h * w)
    frames = []
    for d in (0.0, 1.5):
        x, y = xx - d, yy - 0.7 * d
        img = 128 + 50 * np.sin(x / 3.1) * np.sin(y / 2.7) + 40 * np.sin((x + y) / 9.0)
        frames.append(np.clip(np.rint(img[..., None] + rng.normal(0, 1, (h, w, 3))), 0, 255).astype(np.uint8))
    dev = []
    for f in frames:
        buf = torch.empty(f.size + shift, dtype=torch.uint8, device="cuda")
        dev.append(buf[shift:].view(h, w, 3).copy_(torch.from_numpy(f)))
    uv = torch.empty((2, h, w), dtype=torch.float32, device="cuda")
    dp, gate = torch.empty(576, device="cuda"), torch.zeros(4, dtype=torch.int32, device="cuda")
    ctx.flow_score(dev[0], dev[1], uv, dp, gate)
    d = of.flow(frames[0], frames[1], levels)
    got = uv.cpu().numpy()
    print(f"{h}x{w}, {levels} levels: largest error {max(np.abs(got[0] - d[..., 0]).max(), np.abs(got[1] - d[..., 1]).max()):.2e}", flush=True)
    assert close(got[0], d[..., 0]).all() and close(got[1], d[..., 1]).all()
    ctx.close()


@pytest.mark.parametrize("h,w,levels,iters", [
    (24, 25, 1, 3), (49, 33, 2, 3), (128, 129, 1, 4), (170, 168, 2, 3),                       # three in one: 16x8 tiles
    (181, 243, 1, 3), (240, 433, 2, 3),                                                       # 16x16; 32x16, then 16x8
    (100, 90, 3, 1), (100, 90, 3, 2), (100, 90, 3, 7), (430, 440, 1, 3),                      # single updates, both mixed, too large
    (199, 200, 1, 2), (200, 200, 1, 2), (200, 264, 2, 1), (211, 199, 1, 2),                   # a launch each: 16x16 tiles (the larger tiles: test_single_updates_of_larger_levels)
])
def test_updates_per_launch(h, w, levels, iters):
    """Three updates of a small level in one launch, over its tile shapes, ragged tiles, frames smaller than the
    halo, and update counts that are no multiple of three, against the oracle."""
    from paper_2602_14236_amd import binding
    ctx = binding.SaliContext(lib_config(params(h, w, flow_levels=levels, flow_iters=iters)))
    yy, xx = np.mgrid[0:h, 0:w].astype(np.float64)
    rng = np.random.default_rng(h + w + iters)
    frames = []
    for d in (0.0, 1.0):
        x, y = xx - 1.2 * d, yy + 0.8 * d
        img = 128 + 50 * np.sin(x / 2.9) * np.sin(y / 3.3) + 40 * np.sin((x - y) / 7.0)
        frames.append(np.clip(np.rint(img[..., None] + rng.normal(0, 1, (h, w, 3))), 0, 255).astype(np.uint8))
    uv, _, _ = _run(ctx, frames[0], frames[1])
    d = of.flow(frames[0], frames[1], levels, iters)
    print(f"{h}x{w}, {levels} levels, {iters} updates: largest error "
          f"{max(np.abs(uv[0] - d[..., 0]).max(), np.abs(uv[1] - d[..., 1]).max()):.2e}", flush=True)
    assert close(uv[0], d[..., 0]).all() and close(uv[1], d[..., 1]).all()
    ctx.close()


@pytest.mark.parametrize("h,w,shift", [
    (353, 577, (0.9, -1.3)), (383, 607, (-2.6, 3.4)), (512, 481, (6.0, 5.0)),      # 32x32 tiles: one row and column over, ragged, exact rows
    (270, 929, (0.9, -1.3)), (259, 947, (-2.6, 3.4)),                              # 32x16: a column over, three rows over
    (480, 97, (3.0, -6.0)), (97, 480, (-6.0, 3.0)), (2050, 43, (0.9, -1.3)),       # 16x16, 210 blocks; 387, a round and a half
])
def test_single_updates_of_larger_levels(h, w, shift):
    """Two updates, a launch each, in every tile shape, with windows and warped samples that reach past all four borders
    (samples in the last row and column included), against the oracle."""
    from paper_2602_14236_amd import binding
    ctx = binding.SaliContext(lib_config(params(h, w, flow_levels=1, flow_iters=2)))
    yy, xx = np.mgrid[0:h, 0:w].astype(np.float64)
    rng = np.random.default_rng(h * w)
    frames = []
    for d in (0.0, 1.0):
        x, y = xx - shift[0] * d, yy - shift[1] * d
        img = 128 + 60 * np.sin(x / 9.1) * np.sin(y / 8.3) + 40 * np.sin((x - y) / 15.0)
        frames.append(np.clip(np.rint(img[..., None] + rng.normal(0, 1, (h, w, 3))), 0, 255).astype(np.uint8))
    uv, _, _ = _run(ctx, frames[0], frames[1])
    d = of.flow(frames[0], frames[1], 1, 2)
    print(f"{h}x{w}: largest error {max(np.abs(uv[0] - d[..., 0]).max(), np.abs(uv[1] - d[..., 1]).max()):.2e}", flush=True)
    assert close(uv[0], d[..., 0]).all() and close(uv[1], d[..., 1]).all()
    ctx.close()


def test_flow_score_next_to_analyses_on_another_stream():
    """The stand-alone flow call has scratch of its own: next to batched analyses of the same context on another stream,
    in either order of issue, both give the bits that they give alone."""
    from paper_2602_14236_amd import binding
    h, w, n = 200, 264, 8
    ctx = binding.SaliContext(lib_config(params(h, w, max_frames=n)))
    rng = np.random.default_rng(3)
    base = np.kron(rng.integers(0, 256, (h // 4 + 4, w // 4 + 4, 3), dtype=np.uint8), np.ones((4, 4, 1), dtype=np.uint8))
    rgb = [torch.from_numpy(base[t:t + h, 2 * t % 5:2 * t % 5 + w].copy()).cuda() for t in range(n)]
    pairs = [(0, 1), (5, 2), (3, 7)]
    a, b = torch.cuda.Stream(), torch.cuda.Stream()

    def outputs():
        return [(torch.full((2, h, w), 9.0, device="cuda"), torch.full((576,), 9.0, device="cuda"),
                 torch.zeros(4, dtype=torch.int32, device="cuda")) for _ in pairs]

    def flows(out):
        with torch.cuda.stream(b):
            for (i, j), o in zip(pairs, out):
                ctx.flow_score(rgb[i], rgb[j], *o)

    def analyses():
        ctx.analyze_batch(rgb[:4], 0, a)
        ctx.analyze_batch(rgb[4:], 4, a)

    def analysed():
        torch.cuda.synchronize()
        return [ctx.read_analysis(t) for t in range(n)], [r.as_tuple() for r in ctx.read_frame_table(0, n)]

    alone = outputs()
    flows(alone)
    torch.cuda.synchronize()
    analyses()
    ref, ref_rows = analysed()
    for first in (flows, None):
        for _ in range(4):
            ctx.reset()
            out = outputs()
            torch.cuda.synchronize()
            if first is not None:
                flows(out)
            analyses()
            if first is None:
                flows(out)
            got, rows = analysed()
            assert rows == ref_rows
            for (dp, gate, sc), (dp0, gate0, sc0) in zip(got, ref):
                assert np.array_equal(dp, dp0) and gate.n_static == gate0.n_static and not gate.redundant and np.array_equal(sc, sc0)
            for x, y in zip(out, alone):
                assert all(torch.equal(p, q) for p, q in zip(x, y))
    ctx.close()
