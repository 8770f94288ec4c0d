"""GPU parity of sali_attend_decode (single-query attention that dequantises the mixed-precision
pools on the fly) against the attention oracle, through the C ABI.

Tolerance: the kernel works in fp32 on the same dequantised values as the oracle (float64; codes
times scales, never rounded to fp16).  A logit is a sum of 128 products of fp16 and small-integer
factors, the softmax sums run over up to ~10^5 tokens; both stay far below the 1e-3 relative +
1e-4 absolute bound used for floating-point results here (the largest error met is printed)."""
import math

import numpy as np
import pytest
import torch

from oracle.attention import attend_decode
from oracle.cache import SaliCacheOracle
from paper_2602_14236_amd import synth

from _util import fp16_operand_bounds as _fp16_operand_bounds, lib_config, oracle_config, params, pool_arrays, workload_params

pytestmark = pytest.mark.gpu

RTOL, ATOL = 1e-3, 1e-4


def _check(ctx, orc, layer, q, lo, hi, scale, what):
    n_heads = q.shape[0]
    out = torch.full((n_heads, 128), 7.0, dtype=torch.float32, device="cuda")
    lse = torch.full((n_heads,), 7.0, dtype=torch.float32, device="cuda")
    ctx.attend_decode(layer, q, lo, hi, scale, out, lse)
    torch.cuda.synchronize()
    exp_out, exp_lse = attend_decode(orc, layer, q.cpu().numpy(), lo, hi, scale)
    got, got_lse = out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    err = np.abs(got - exp_out)
    assert np.all(err <= ATOL + RTOL * np.abs(exp_out)), f"{what}: out, max error {err.max():.3e}"
    if np.all(np.isneginf(exp_lse)):
        assert np.all(np.isneginf(got_lse)) and not got.any(), f"{what}: empty range"
    else:
        assert np.all(np.abs(got_lse - exp_lse) <= ATOL + RTOL * np.abs(exp_lse)), f"{what}: lse"
    return float(err.max())


def _q(seed, n_heads):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return torch.randn((n_heads, 128), generator=g).to(torch.float16).cuda()


def test_attend_after_chained_steps_all_tiers_pointers_and_cuts():
    """Config 5 frames 0..11: threshold tiers (FP16, INT8, INT4 and pruned tokens), exact duplicates
    5..8 (pointer entries), two layers and three heads; whole range, ranges that start inside the
    pointer run, a pointer frame alone, an empty range."""
    from paper_2602_14236_amd import binding
    wl = synth.WORKLOADS[5]
    n, nl, nh = 12, 2, 3
    v = synth.video(5, 32)
    p = workload_params(wl, frames=n, n_layers=nl, n_heads=nh)
    scale_c = synth.kv_channel_scale(wl, nl, nh)
    ctx = binding.SaliContext(lib_config(p))
    orc = SaliCacheOracle(oracle_config(p))
    for t in range(n):
        print(f"frame {t} ({v.kind(t)})", flush=True)
        kv = synth.kv_frame(wl, t, device="cuda", n_layers=nl, n_heads=nh, scale=scale_c)
        ctx.step(torch.from_numpy(v.frame(t)).cuda(), kv, t)
        orc.step(v.frame(t), kv.cpu().numpy(), t)
    torch.cuda.synchronize()
    stored = [orc.rows[t].stored for t in range(n)]
    assert stored[5:9] == [0, 0, 0, 0] and stored[4] == 1
    assert any(int((orc.tier[t] == 3).sum()) > 0 for t in orc.tier) and any(int((orc.tier[t] == 2).sum()) > 0 for t in orc.tier)
    sm = 1.0 / math.sqrt(128.0)
    worst = 0.0
    for layer in range(nl):
        q = _q(100 + layer, nh)
        for lo, hi in ((0, n), (6, 9), (5, 6), (7, n), (0, 1), (3, 3), (4, 10)):
            worst = max(worst, _check(ctx, orc, layer, q, lo, hi, sm, f"layer {layer} frames [{lo}, {hi})"))
    # a large softmax scale: one token dominates
    worst = max(worst, _check(ctx, orc, 0, _q(7, nh), 0, n, 4.0, "sharp softmax"))
    print(f"largest |out - oracle| = {worst:.3e}", flush=True)
    assert ctx.get_status() == 0
    ctx.close()


def test_attend_long_range_many_frames_per_block():
    """150 stored frames of one head (top-k tiers 173 / 259 / 100, 44 pruned): more frames than
    partial slots, so a block walks several frames; also a range that is not a multiple of the
    chunk size."""
    from paper_2602_14236_amd import binding
    n = 150
    p = params(96, 96, tier_mode=1, k_fp16=173, k_int8=259, k_int4=100, n_layers=1, n_heads=1, cap_fp16=173 * n,
               cap_int8=259 * n, cap_int4=100 * n, max_frames=n)
    ctx = binding.SaliContext(lib_config(p))
    orc = SaliCacheOracle(oracle_config(p))
    g = torch.Generator(device="cpu").manual_seed(5)
    for t in range(n):
        kv = (torch.randn((1, 2, 1, 576, 128), generator=g) * 0.7).to(torch.float16)
        scores = torch.rand(576, generator=g)
        ctx.kv_compress(kv.cuda(), scores.cuda(), t)
        orc.kv_compress(kv.numpy(), scores.numpy(), t)
    torch.cuda.synchronize()
    q = _q(9, 1)
    sm = 1.0 / math.sqrt(128.0)
    worst = max(_check(ctx, orc, 0, q, 0, n, sm, "150 frames"), _check(ctx, orc, 0, q, 11, 140, sm, "129 frames"),
                _check(ctx, orc, 0, q, 20, 33, sm, "13 frames"))
    print(f"largest |out - oracle| = {worst:.3e}", flush=True)
    # the matrix-core path over the same cache: 32 queries on the one K/V head; several frames per
    # wave, ranges that end inside a tile, all three tiers
    q32 = _q(77, 32)
    out = torch.empty((32, 128), dtype=torch.float32, device="cuda")
    lse = torch.empty((32,), dtype=torch.float32, device="cuda")
    for lo, hi in ((0, n), (11, 140), (20, 21)):
        ctx.attend_decode_gqa(0, q32, 32, lo, hi, sm, out, lse)
        torch.cuda.synchronize()
        exp_out, exp_lse = attend_decode(orc, 0, q32.cpu().numpy(), lo, hi, sm, q_per_kv=32)
        bound, lse_bound = _fp16_operand_bounds(orc, q32.cpu().numpy(), lo, hi, sm, 32)
        err = np.abs(out.cpu().numpy().astype(np.float64) - exp_out)
        assert np.all(err <= bound), f"32 queries, frames [{lo}, {hi}): max error {err.max():.3e}"
        assert np.all(np.abs(lse.cpu().numpy() - exp_lse) <= lse_bound)
        rms = math.sqrt(float((err ** 2).mean())) / math.sqrt(float((exp_out ** 2).mean()))
        assert rms <= 1e-3, rms
        print(f"32 queries, frames [{lo}, {hi}): largest error {err.max():.3e}, relative rms {rms:.2e}", flush=True)
    ctx.close()


def test_attend_full_shape_sampled_layers():
    """The benchmark's K/V shape (32 layers x 32 heads, config 2's 173 fp16 / 403 int8 split) for 8
    frames in the launch configuration bench.py times; the oracle holds one sampled layer at a time."""
    from paper_2602_14236_amd import binding
    wl = synth.WORKLOADS[2]
    n = 8
    p = workload_params(wl, frames=n)
    ctx = binding.SaliContext(lib_config(p))
    scale_c = synth.kv_channel_scale(wl, wl.n_layers)
    g = torch.Generator(device="cpu").manual_seed(3)
    scores = [torch.rand(576, generator=g) for _ in range(n)]
    layers = (0, 17, 31)
    p1 = dict(p)
    p1["n_layers"] = 1
    orcs = {L: SaliCacheOracle(oracle_config(p1)) for L in layers}
    for t in range(n):
        print(f"frame {t}", flush=True)
        kv = synth.kv_frame(wl, t, device="cuda", scale=scale_c)
        ctx.kv_compress(kv, scores[t].cuda(), t)
        for L in layers:
            orcs[L].kv_compress(kv[L:L + 1].cpu().numpy(), scores[t].numpy(), t)
        del kv
    torch.cuda.synchronize()
    sm = 1.0 / math.sqrt(128.0)
    worst = 0.0
    for L in layers:
        q = _q(40 + L, wl.n_heads)
        n_heads = wl.n_heads
        out = torch.empty((n_heads, 128), dtype=torch.float32, device="cuda")
        lse = torch.empty((n_heads,), dtype=torch.float32, device="cuda")
        ctx.attend_decode(L, q, 0, n, sm, out, lse)
        torch.cuda.synchronize()
        exp_out, exp_lse = attend_decode(orcs[L], 0, q.cpu().numpy(), 0, n, sm)
        err = np.abs(out.cpu().numpy().astype(np.float64) - exp_out)
        assert np.all(err <= ATOL + RTOL * np.abs(exp_out)), f"layer {L}: max error {err.max():.3e}"
        assert np.all(np.abs(lse.cpu().numpy().astype(np.float64) - exp_lse) <= ATOL + RTOL * np.abs(exp_lse))
        worst = max(worst, float(err.max()))
    print(f"largest |out - oracle| = {worst:.3e}", flush=True)
    # the same cache through the matrix-core path as bench.py times it: 32 queries on each of the 32 K/V heads
    L, qpk = 17, 32
    q = _q(90, wl.n_heads * qpk)
    out = torch.empty((wl.n_heads * qpk, 128), dtype=torch.float32, device="cuda")
    lse = torch.empty((wl.n_heads * qpk,), dtype=torch.float32, device="cuda")
    for lo, hi in ((0, n), (2, 7)):
        ctx.attend_decode_gqa(L, q, qpk, lo, hi, sm, out, lse)
        torch.cuda.synchronize()
        exp_out, exp_lse = attend_decode(orcs[L], 0, q.cpu().numpy(), lo, hi, sm, q_per_kv=qpk)
        bound, lse_bound = _fp16_operand_bounds(orcs[L], q.cpu().numpy(), lo, hi, sm, qpk)
        err = np.abs(out.cpu().numpy().astype(np.float64) - exp_out)
        assert np.all(err <= bound), f"32 queries per head, frames [{lo}, {hi}): max error {err.max():.3e}"
        assert np.all(np.abs(lse.cpu().numpy() - exp_lse) <= lse_bound)
        rms = math.sqrt(float((err ** 2).mean())) / math.sqrt(float((exp_out ** 2).mean()))
        assert rms <= 1e-3, rms
        print(f"32 queries per head, frames [{lo}, {hi}): largest error {err.max():.3e}, relative rms {rms:.2e}", flush=True)
    assert ctx.get_status() == 0
    ctx.close()


@pytest.mark.parametrize("q_per_kv", [2, 4, 8, 16, 32, 40, 64])
def test_attend_grouped_queries(q_per_kv):
    """Several queries per K/V head: 2 K/V heads, q_per_kv queries each; threshold tiers (all four
    tiers), a duplicate frame stored through the chained step.  Up to 8 queries run in the streaming
    kernel against the usual tolerance.  More run on the matrix cores, whose operands are fp16: K^, V^
    and the softmax weights each carry a relative rounding error of at most u = 2^-11.  To first order
    a logit moves by at most u * S_j, S_j = softmax_scale * sum_d |q_d K^_jd|, a weight by twice the
    largest such shift (numerator and normaliser), so
        |out_d - exact_d| <= u * (2 + 2 max_j S_j) * sum_j p_j |V^_jd|,   |lse - exact| <= u * (1 + max_j S_j),
    which is the tolerance used here (with the factor doubled for the second-order terms and the
    fp32 accumulation, plus 1e-6); the largest error met is printed next to the bound."""
    from paper_2602_14236_amd import binding
    wl = synth.WORKLOADS[1]
    n, nh = 6, 2
    v = synth.video(1)
    p = workload_params(wl, frames=n, n_layers=1, n_heads=nh)
    scale_c = synth.kv_channel_scale(wl, 1, nh)
    ctx = binding.SaliContext(lib_config(p))
    orc = SaliCacheOracle(oracle_config(p))
    for t in range(n):
        kv = synth.kv_frame(wl, t, device="cuda", n_layers=1, n_heads=nh, scale=scale_c)
        ctx.step(torch.from_numpy(v.frame(t)).cuda(), kv, t)
        orc.step(v.frame(t), kv.cpu().numpy(), t)
    torch.cuda.synchronize()
    assert sum(1 for t in range(n) if not orc.rows[t].stored) == 1
    q = _q(200 + q_per_kv, nh * q_per_kv)
    sm = 1.0 / math.sqrt(128.0)
    out = torch.empty((nh * q_per_kv, 128), dtype=torch.float32, device="cuda")
    lse = torch.empty((nh * q_per_kv,), dtype=torch.float32, device="cuda")
    worst, tight, worst_rms = 0.0, np.inf, 0.0
    for lo, hi in ((0, n), (3, 5), (2, 2)):
        ctx.attend_decode_gqa(0, q, q_per_kv, lo, hi, sm, out, lse)
        torch.cuda.synchronize()
        exp_out, exp_lse = attend_decode(orc, 0, q.cpu().numpy(), lo, hi, sm, q_per_kv=q_per_kv)
        got = out.cpu().numpy().astype(np.float64)
        err = np.abs(got - exp_out)
        if q_per_kv <= 8 or lo == hi:
            bound = ATOL + RTOL * np.abs(exp_out)
            lse_bound = ATOL + RTOL * np.abs(exp_lse)
        else:
            bound, lse_bound = _fp16_operand_bounds(orc, q.cpu().numpy(), lo, hi, sm, q_per_kv)
        assert np.all(err <= bound), f"[{lo}, {hi}): max error {err.max():.3e}, bound there {bound.flat[err.argmax()]:.3e}"
        if lo < hi:       # the worst-case bound is loose; the typical error is far smaller
            rms = math.sqrt(float((err ** 2).mean())) / math.sqrt(float((exp_out ** 2).mean()))
            assert rms <= 1e-3, f"[{lo}, {hi}): relative rms error {rms:.3e}"
            worst_rms = max(worst_rms, rms)
        if lo < hi:
            assert np.all(np.abs(lse.cpu().numpy() - exp_lse) <= lse_bound)
        else:
            assert not got.any() and np.all(np.isneginf(lse.cpu().numpy()))
        worst = max(worst, float(err.max()))
        tight = min(tight, float((bound / np.maximum(err, 1e-30)).min()))
    print(f"q_per_kv={q_per_kv}: largest |out - oracle| = {worst:.3e}; bound / error at least {tight:.1f}; relative rms error {worst_rms:.2e}", flush=True)
    for bad in (3, 65):
        with pytest.raises(binding.SaliError) as e:
            ctx.attend_decode_gqa(0, q, bad, 0, n, sm, out, lse)
        assert e.value.code == -2
    ctx.close()


def test_attend_argument_checks():
    from paper_2602_14236_amd import binding
    p = params(96, 96, n_layers=2, n_heads=2, cap_fp16=576, cap_int8=576, cap_int4=576, max_frames=4)
    ctx = binding.SaliContext(lib_config(p))
    q = _q(1, 2)
    out = torch.empty((2, 128), dtype=torch.float32, device="cuda")
    for args in ((2, q, 0, 1), (-1, q, 0, 1), (0, q, 2, 1), (0, q, 0, 5), (0, q, -1, 2)):
        with pytest.raises(binding.SaliError) as e:
            ctx.attend_decode(args[0], args[1], args[2], args[3], 1.0, out)
        assert e.value.code == -2
    with pytest.raises(binding.SaliError) as e:
        ctx.attend_decode(0, None, 0, 1, 1.0, out)
    assert e.value.code == -1
    # nothing stored yet: zeros and -inf
    lse = torch.empty(2, dtype=torch.float32, device="cuda")
    ctx.attend_decode(1, q, 0, 4, 1.0, out, lse)
    torch.cuda.synchronize()
    assert not out.cpu().numpy().any() and np.all(np.isneginf(lse.cpu().numpy()))
    ctx.close()


@pytest.mark.parametrize("heads,q_per_kv,frames,counts", [
    (1, 9, 1, (1, 0, 0)),            # fewer tiles than waves, one row
    (2, 33, 2, (31, 32, 33)),        # tile edges; a second query tile with one query
    (3, 64, 5, (0, 65, 0)),          # one tier only
    (64, 10, 200, (3, 2, 2)),        # four parts of 50 frames
    (64, 10, 264, (3, 2, 2)),        # four parts of 66: a block looks up frames twice, two the second time
    (64, 40, 200, (33, 0, 1)),       # two parts of 100, two query tiles
    (129, 9, 5, (33, 2, 40)),        # more heads than half the compute units: three parts in two rounds
])
def test_many_queries_shares_of_the_range_and_pointer_runs(heads, q_per_kv, frames, counts):
    """The matrix-core path where its split of the work has edges: tiles with few rows, blocks whose share
    begins or ends inside a frame, more frames than are looked up at a time, runs of pointer frames across
    those limits and at the head of the range.  Reference: float64 attention over the values dequantise-on-
    read returns (the path's own operands), every frame counted as often as it is used.  What is left are
    the fp16 rounding of the softmax weights (2^-11 relative, 2^-25 absolute below the normal numbers) and
    fp32 accumulation (1e-5 relative covers n <= 50 000 rows' worth of it)."""
    from paper_2602_14236_amd import binding
    k16, k8, k4 = counts
    p = params(96, 96, tier_mode=1, k_fp16=k16, k_int8=k8, k_int4=k4, n_layers=1, n_heads=heads,
               cap_fp16=max(1, k16 * frames), cap_int8=max(1, k8 * frames), cap_int4=max(1, k4 * frames), max_frames=frames)
    ctx = binding.SaliContext(lib_config(p))
    g = torch.Generator(device="cuda").manual_seed(heads + frames)
    stored_at = [t for t in range(frames) if t in (0, 1) or t % 97 in (3, 4, 60, 63, 64)]
    rgb = torch.randint(0, 256, (96, 96, 3), generator=g, device="cuda", dtype=torch.uint8)
    for t in range(frames):
        # every frame with a predecessor is redundant under the first setting, none under the second
        ctx.set_gate_thresholds(*((1.0, 2.0) if t in stored_at else (1e9, 0.0)))
        kv = torch.randn((1, 2, heads, 576, 128), generator=g, device="cuda").to(torch.float16)
        ctx.step(rgb, kv, t)
    rows = ctx.read_frame_table(0, frames)
    assert [t for t in range(frames) if rows[t].stored] == stored_at
    dense, kept = {}, {}
    for t in stored_at:
        out, valid = torch.empty((1, 2, heads, 576, 128), dtype=torch.float16, device="cuda"), torch.empty(576, dtype=torch.uint8, device="cuda")
        ctx.kv_decompress(t, out, valid)
        kept[t] = valid.nonzero().flatten()
        dense[t] = out[0][:, :, kept[t]].double()
    q = torch.randn((heads * q_per_kv, 128), generator=g, device="cuda").to(torch.float16)
    sm = 128.0 ** -0.5
    got, lse = torch.empty((heads * q_per_kv, 128), device="cuda"), torch.empty(heads * q_per_kv, device="cuda")
    for lo, hi in ((0, frames), (min(2, frames - 1), frames), (frames // 3, frames - frames // 4)):
        ctx.attend_decode_gqa(0, q, q_per_kv, lo, hi, sm, got, lse)
        uses = [rows[t].src for t in range(lo, hi)]
        k = torch.cat([dense[t][0] for t in sorted(set(uses))], dim=1)
        v = torch.cat([dense[t][1] for t in sorted(set(uses))], dim=1)
        mult = torch.cat([torch.full((len(kept[t]),), float(uses.count(t)), dtype=torch.float64, device="cuda") for t in sorted(set(uses))])
        s = torch.bmm(q.double().view(heads, q_per_kv, 128), k.transpose(1, 2).contiguous()) * sm + mult.log()
        pr = torch.softmax(s, dim=-1)
        exp, exp_lse = torch.bmm(pr, v).reshape(-1, 128), torch.logsumexp(s, dim=-1).reshape(-1)
        top = pr.amax(-1, keepdim=True)
        bound = (2.0 ** -11 + 1e-5) * torch.bmm(pr, v.abs()) + 2.0 ** -24 * top * v.abs().sum(1, keepdim=True)
        err = (got.double() - exp).abs()
        print(f"heads {heads} q {q_per_kv} frames [{lo}, {hi}): largest error / bound {(err / bound.reshape(-1, 128)).max():.3f}", flush=True)
        assert bool((err <= bound.reshape(-1, 128)).all())
        assert bool(((lse.double() - exp_lse).abs() <= 1e-5 * (1 + exp_lse.abs())).all())
    assert ctx.get_status() == 0
    ctx.close()


@pytest.mark.parametrize("q_per_kv", [1, 2, 4, 8])
@pytest.mark.parametrize("frames,heads,counts", [
    (1, 1, (1, 0, 0)), (1, 3, (0, 0, 17)), (2, 2, (15, 16, 33)), (3, 1, (64, 65, 63)), (1, 2, (288, 144, 144)),   # groups of 16 rows
    (30, 2, (200, 180, 196)), (30, 5, (63, 65, 128)),                                                              # groups of 64
    (12, 5, (63, 65, 128)),                                                                                        # of 16, and of 64 with 8 queries
])
def test_few_queries_groups_of_rows(q_per_kv, frames, heads, counts):
    """The streaming kernel on both sides of its rule (groups of 16 rows for small ranges, of 64 otherwise) where
    groups end, tiers are empty and a frame has fewer groups than blocks.  fp32 sums of at most 20 000 terms
    in hundreds of partial ones against the float64 oracle: 1e-5 relative to the largest output."""
    from paper_2602_14236_amd import binding
    k16, k8, k4 = counts
    p = params(96, 96, tier_mode=1, k_fp16=k16, k_int8=k8, k_int4=k4, n_layers=1, n_heads=heads,
               cap_fp16=k16 * frames + 1, cap_int8=k8 * frames + 1, cap_int4=k4 * frames + 1, max_frames=frames)
    ctx = binding.SaliContext(lib_config(p))
    orc = SaliCacheOracle(oracle_config(p))
    g = torch.Generator(device="cpu").manual_seed(frames * 100 + heads)
    for t in range(frames):
        kv = torch.randn((1, 2, heads, 576, 128), generator=g).to(torch.float16)
        scores = torch.rand(576, generator=g)
        ctx.kv_compress(kv.cuda(), scores.cuda(), t)
        orc.kv_compress(kv.numpy(), scores.numpy(), t)
    q = _q(3, heads * q_per_kv)
    out, lse = torch.empty((heads * q_per_kv, 128), device="cuda"), torch.empty(heads * q_per_kv, device="cuda")
    for lo, hi in ((0, frames), (frames // 2, frames)):
        ctx.attend_decode_gqa(0, q, q_per_kv, lo, hi, 128.0 ** -0.5, out, lse)
        exp, exp_lse = attend_decode(orc, 0, q.cpu().numpy(), lo, hi, 128.0 ** -0.5, q_per_kv=q_per_kv)
        err = np.abs(out.cpu().numpy() - exp).max() / np.abs(exp).max()
        print(f"{frames} frames [{lo}, {hi}), {heads} heads, {q_per_kv} queries: relative error {err:.1e}", flush=True)
        assert err <= 1e-5
        assert np.all(np.abs(lse.cpu().numpy() - exp_lse) <= 1e-5 * (1 + np.abs(exp_lse)))
    ctx.close()


@pytest.mark.parametrize("stored_at", [(0,), (0, 100), (0, 33000)])
def test_many_queries_frames_counted_tens_of_thousands_of_times(stored_at):
    """The matrix-core path over a static camera's range: a stored frame with tens of thousands of pointer frames
    behind it, alone, next to a frame of few uses in the same block's share, and next to one of as many.  A count
    of more than 65 504 is no fp16 number, the operand type of the second product.  Reference and bounds as
    above: rounding of the weights to fp16 (2^-11 relative, 2^-25 of the largest weight below the normal numbers)
    and fp32 accumulation."""
    from paper_2602_14236_amd import binding
    n, q_per_kv, counts, sm = 70000, 9, (40, 70, 33), 128.0 ** -0.5
    p = params(24, 24, flow_levels=1, tier_mode=1, k_fp16=counts[0], k_int8=counts[1], k_int4=counts[2], n_layers=1, n_heads=1,
               cap_fp16=2 * counts[0], cap_int8=2 * counts[1], cap_int4=2 * counts[2], max_frames=n)
    ctx = binding.SaliContext(lib_config(p))
    g = torch.Generator(device="cuda").manual_seed(len(stored_at) + stored_at[-1])
    rgb = torch.randint(0, 256, (24, 24, 3), generator=g, device="cuda", dtype=torch.uint8)
    dense, t = {}, 0
    while t < n:
        if t in stored_at:
            ctx.set_gate_thresholds(1.0, 2.0)           # no frame is redundant
            kv = torch.randn((1, 2, 1, 576, 128), generator=g, device="cuda").to(torch.float16)
            ctx.step(rgb, kv, t)
            ctx.set_gate_thresholds(1e9, 0.0)           # every frame with a predecessor is
            out, valid = torch.empty_like(kv), torch.empty(576, dtype=torch.uint8, device="cuda")
            ctx.kv_decompress(t, out, valid)
            dense[t] = out[0, :, 0, valid.bool()].double()
            t += 1
        else:
            m = min([16, n - t] + [s - t for s in stored_at if s > t])
            ctx.analyze_batch([rgb] * m, t)
            t += m
    rows = ctx.read_frame_table(0, n)
    assert [t for t in range(n) if rows[t].stored] == list(stored_at)
    uses = {s: sum(1 for r in rows if r.src == s) for s in stored_at}
    assert sum(uses.values()) == n
    q = torch.randn((q_per_kv, 128), generator=g, device="cuda").to(torch.float16)
    got, lse = torch.empty((q_per_kv, 128), device="cuda"), torch.empty(q_per_kv, device="cuda")
    ctx.attend_decode_gqa(0, q, q_per_kv, 0, n, sm, got, lse)
    k, v = (torch.cat([dense[s][i] for s in stored_at]) for i in range(2))
    mult = torch.cat([torch.full((sum(counts),), float(uses[s]), dtype=torch.float64, device="cuda") for s in stored_at])
    s = q.double() @ k.t().contiguous() * sm + mult.log()
    pr = torch.softmax(s, dim=-1)
    exp, exp_lse = pr @ v, torch.logsumexp(s, dim=-1)
    bound = (2.0 ** -11 + 1e-5) * (pr @ v.abs()) + 2.0 ** -24 * pr.amax(-1, keepdim=True) * v.abs().sum(0)
    err = (got.double() - exp).abs()
    print(f"uses {uses}: largest error / bound {(err / bound).max():.3f}", flush=True)
    assert bool((err <= bound).all())
    assert bool(((lse.double() - exp_lse).abs() <= 1e-5 * (1 + exp_lse.abs())).all())
    ctx.close()


@pytest.mark.parametrize("q_per_kv", [1, 4, 8])
def test_few_queries_rows_other_than_the_tier_rule_in_force_says(q_per_kv):
    """The streaming kernel's launch is shaped by the rows a frame keeps under the present tier rule; a frame stored
    under another rule, with more or fewer rows or in other tiers, is read whole all the same.  Bounds as above."""
    from paper_2602_14236_amd import binding
    heads, frames = 2, 3
    p = params(96, 96, tier_mode=1, k_fp16=150, k_int8=90, k_int4=110, n_layers=1, n_heads=heads, cap_fp16=600, cap_int8=600,
               cap_int4=600, max_frames=frames)
    ctx = binding.SaliContext(lib_config(p))
    orc = SaliCacheOracle(oracle_config(p))
    g = torch.Generator(device="cpu").manual_seed(5)
    for t in range(frames):
        kv, scores = torch.randn((1, 2, heads, 576, 128), generator=g).to(torch.float16), torch.rand(576, generator=g)
        ctx.kv_compress(kv.cuda(), scores.cuda(), t)
        orc.kv_compress(kv.numpy(), scores.numpy(), t)
    q = _q(4, heads * q_per_kv)
    out, lse = torch.empty((heads * q_per_kv, 128), device="cuda"), torch.empty(heads * q_per_kv, device="cuda")
    exp, exp_lse = attend_decode(orc, 0, q.cpu().numpy(), 0, frames, 128.0 ** -0.5, q_per_kv=q_per_kv)
    for mode, counts in ((1, (150, 90, 110)), (1, (0, 0, 0)), (1, (0, 0, 16)), (1, (576, 0, 0)), (0, (0, 0, 0)), (2, (10, 10, 10))):
        ctx.set_tier_params(mode, k_fp16=counts[0], k_int8=counts[1], k_int4=counts[2])
        out.fill_(7.0)
        ctx.attend_decode_gqa(0, q, q_per_kv, 0, frames, 128.0 ** -0.5, out, lse)
        err = np.abs(out.cpu().numpy() - exp).max() / np.abs(exp).max()
        print(f"mode {mode} {counts}, {q_per_kv} queries: relative error {err:.1e}", flush=True)
        assert err <= 1e-5
        assert np.all(np.abs(lse.cpu().numpy() - exp_lse) <= 1e-5 * (1 + np.abs(exp_lse)))
    ctx.close()


@pytest.mark.parametrize("heads", [1, 15, 16, 51, 128, 129, 257, 600, 1100])
def test_parts_and_their_hand_over_by_number_of_heads(heads):
    """The number of heads decides how many parts the range is cut into, down to one part that nobody has to merge, and how the
    blocks are dealt; the last block of a head to finish merges its parts.  Calls with different numbers of queries follow each
    other on one context, so each finds the arrival counters as the ones before left them: every repetition gives the same
    bits.  Rows of the FP16 tier only: float64 attention over the stored values; fp32 sums of 200 terms (1e-5 relative) and, from nine
    queries on, softmax weights rounded to fp16 (2^-11, 2^-25 absolute below the normal numbers)."""
    from paper_2602_14236_amd import binding
    frames, k16 = 4, 50
    p = params(96, 96, tier_mode=1, k_fp16=k16, k_int8=0, k_int4=0, n_layers=1, n_heads=heads, cap_fp16=k16 * frames, cap_int8=1,
               cap_int4=1, max_frames=frames)
    ctx = binding.SaliContext(lib_config(p))
    g = torch.Generator(device="cuda").manual_seed(heads)
    dense = []
    for t in range(frames):
        kv = torch.randn((1, 2, heads, 576, 128), generator=g, device="cuda").to(torch.float16)
        scores = torch.rand(576, generator=g, device="cuda")
        ctx.kv_compress(kv, scores, t)
        dense.append(kv[0][:, :, torch.topk(scores, k16).indices].float())
    k, v = (torch.cat([d[i] for d in dense], dim=1).double() for i in (0, 1))
    first = {}
    for rep in range(3):
        for n in (1, 8, 33, 2, 9, 4):
            q = torch.randn((heads * n, 128), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda").to(torch.float16)
            out, lse = torch.full((heads * n, 128), 7.0, device="cuda"), torch.full((heads * n,), 7.0, device="cuda")
            ctx.attend_decode_gqa(0, q, n, 0, frames, 128.0 ** -0.5, out, lse)
            if rep > 0:
                assert torch.equal(out, first[n][0]) and torch.equal(lse, first[n][1]), f"{n} queries, repetition {rep}"
                continue
            first[n] = (out, lse)
            s = torch.bmm(q.double().view(heads, n, 128), k.transpose(1, 2).contiguous()) * 128.0 ** -0.5
            pr = torch.softmax(s, dim=-1)
            exp, size = torch.bmm(pr, v).reshape(-1, 128), torch.bmm(pr, v.abs()).reshape(-1, 128)
            bound = 1e-5 * size
            if n > 8:
                bound = (2.0 ** -11 + 1e-5) * size + 2.0 ** -24 * (pr.amax(-1, keepdim=True) * v.abs().sum(1, keepdim=True)).reshape(-1, 128)
            err = (out.double() - exp).abs()
            print(f"{heads} heads, {n} queries: largest error / bound {(err / bound).max():.3f}", flush=True)
            assert bool((err <= bound).all())
            assert bool(((lse.double() - torch.logsumexp(s, dim=-1).reshape(-1)).abs() <= 1e-5 * (1 + lse.double().abs())).all())
    assert ctx.get_status() == 0
    ctx.close()


@pytest.mark.parametrize("heads,frames,counts,tiles", [
    (1, 2, (20, 20, 24), 1), (1, 10, (20, 20, 24), 1), (1, 11, (20, 20, 24), 1),        # 12 parts, 60 of a group each, 33 of two
    (1, 24, (20, 20, 24), 1), (1, 60, (20, 20, 24), 1),                                 # 72 parts, 128 parts
    (2, 24, (1, 40, 17), 2), (5, 30, (33, 0, 50), 3), (8, 30, (100, 90, 77), 1), (40, 4, (33, 50, 17), 1), (70, 3, (17, 100, 30), 1),
])
def test_parts_that_cut_tiers_pointer_frames_and_tiles(heads, frames, counts, tiles):
    """Parts of the range begin and end inside tiers and frames, at pointer entries and among the tiles of a frame; their number, and with
    it who merges them (a block of the launch, or a launch with one, four or sixteen waves a query), goes from a few to 128.  Reference:
    float64 attention over the stored codes.  Up to eight queries fp32 sums, 1e-5 of the largest output; above, the bounds of fp16 operands."""
    from types import SimpleNamespace
    from paper_2602_14236_amd import binding
    k16, k8, k4 = counts
    p = params(96, 96, tier_mode=1, k_fp16=k16, k_int8=k8, k_int4=k4, n_layers=1, n_heads=heads, cap_fp16=k16 * frames + 1,
               cap_int8=k8 * frames + 1, cap_int4=k4 * frames + 1, max_frames=frames, tiles_per_frame=tiles)
    ctx = binding.SaliContext(lib_config(p))
    g = torch.Generator(device="cuda").manual_seed(heads + frames)
    rgb = torch.randint(0, 256, (96, 96, 3), generator=g, device="cuda", dtype=torch.uint8)
    for t in range(0, frames, tiles):
        ctx.set_gate_thresholds(*((1e9, 0.0) if (t // tiles) % 5 in (2, 4) else (1.0, 2.0)))       # redundant, or not
        kv = [torch.randn((1, 2, heads, 576, 128), generator=g, device="cuda").to(torch.float16) for _ in range(tiles)]
        ctx.step_batch([rgb] * tiles, kv, t)
    table = ctx.read_frame_table(0, frames)
    assert [r.stored for r in table] == [0 if (t // tiles) % 5 in (2, 4) else 1 for t in range(frames)]
    pools = pool_arrays(ctx)
    cache = SimpleNamespace(rows=dict(enumerate(table)), cfg=SimpleNamespace(n_heads=heads, head_dim=128), pool16=pools["fp16"],
                            codes8=pools["codes8"], scale8=pools["scale8"], codes4=pools["codes4"], scale4=pools["scale4"], zero4=pools["zero4"])
    sm = 128.0 ** -0.5
    for n in (1, 2, 4, 8, 9, 33):
        q = _q(n, heads * n)
        out, lse = torch.empty((heads * n, 128), device="cuda"), torch.empty(heads * n, device="cuda")
        for lo, hi in ((0, frames), (min(2 * tiles, frames - tiles), frames)):
            ctx.attend_decode_gqa(0, q, n, lo, hi, sm, out, lse)
            exp, exp_lse = attend_decode(cache, 0, q.cpu().numpy(), lo, hi, sm, q_per_kv=n)
            err, lse_err = np.abs(out.cpu().numpy() - exp), np.abs(lse.cpu().numpy() - exp_lse)
            bound, lse_bound = (1e-5 * np.abs(exp).max(), 1e-5 * (1 + np.abs(exp_lse))) if n <= 8 else \
                _fp16_operand_bounds(cache, q.cpu().numpy(), lo, hi, sm, n)
            print(f"{heads} heads, {n} queries, frames [{lo}, {hi}): largest error / bound {(err / bound).max():.3f}", flush=True)
            assert np.all(err <= bound) and np.all(lse_err <= lse_bound)
    assert ctx.get_status() == 0
    ctx.close()


@pytest.mark.parametrize("heads,q_per_kv", [(1, 1), (32, 1), (2, 2), (32, 4), (3, 8)])
@pytest.mark.parametrize("rows", [1, 15, 17, 64, 70, 130])
def test_infinite_values_stay_in_their_column(heads, q_per_kv, rows):
    """FP16 rows are used as stored, so an infinity among the values makes that column of the result infinite and no other.  It sits in
    the last row of the frame's run: lane groups without a row of their own ask for that one again and must not add it."""
    from paper_2602_14236_amd import binding
    p = params(96, 96, tier_mode=1, k_fp16=rows, k_int8=0, k_int4=0, n_layers=1, n_heads=heads, cap_fp16=2 * rows, cap_int8=1, cap_int4=1,
               max_frames=2)
    ctx = binding.SaliContext(lib_config(p))
    g = torch.Generator(device="cuda").manual_seed(rows)
    scores = torch.linspace(1.0, 0.0, 576, device="cuda")              # the first tokens are kept, in order
    kept = []
    for t in range(2):
        kv = torch.randn((1, 2, heads, 576, 128), generator=g, device="cuda").to(torch.float16)
        kv[0, 1, :, rows - 1, 5 + t] = float("inf") if t == 0 else float("-inf")
        ctx.kv_compress(kv, scores, t)
        kept.append(kv[0, :, :, :rows].double())
    k, v = (torch.cat([d[i] for d in kept], dim=1) for i in (0, 1))
    n = q_per_kv
    q = torch.randn((heads * n, 128), generator=g, device="cuda").to(torch.float16)
    out, lse = torch.empty((heads * n, 128), device="cuda"), torch.empty(heads * n, device="cuda")
    ctx.attend_decode_gqa(0, q, n, 0, 2, 128.0 ** -0.5, out, lse)
    pr = torch.softmax(torch.bmm(q.double().view(heads, n, 128), k.transpose(1, 2).contiguous()) * 128.0 ** -0.5, dim=-1)
    assert bool((out[:, 5] == float("inf")).all()) and bool((out[:, 6] == float("-inf")).all())
    rest = [d for d in range(128) if d not in (5, 6)]
    v = v[:, :, rest].contiguous()
    err = (out[:, rest].double() - torch.bmm(pr, v).reshape(heads * n, -1)).abs()
    assert bool((err <= 1e-5 * torch.bmm(pr, v.abs()).reshape(heads * n, -1)).all())
    ctx.close()
