"""GPU parity of the DiT block, the denoiser, the cache and the sampler step
against the CPU oracle, through the C ABI, on identical seeded inputs.

Floating-point outputs: max-abs <= 1e-2 and relative RMS <= 1e-3 (the bar of
the task), also for the tensors inside a block.  The integer codes inside a
block are the oracle's (at most 1e-6 of them may differ, by one step)."""
import numpy as np
import pytest

from oracle import dit, quant, sampler
from synthetic import dit_inputs as I
from qc_testlib import (assert_close, code_flip_stats, make_pair, oracle_calibration, rel_rms, max_abs)

pytestmark = pytest.mark.gpu

TINY = I.ModelDesc(depth=2, hidden=32, heads=2, mlp_dim=64, patch=2, latent_c=4, latent_h=8, latent_w=8,
                   num_classes=10)
# ragged everywhere: 35 tokens (not a multiple of the 64-key tile), head dim 20, hidden 80
RAGGED = I.ModelDesc(depth=2, hidden=80, heads=4, mlp_dim=176, patch=1, latent_c=3, latent_h=5, latent_w=7,
                     num_classes=7)
# the limits of the kernels: widest hidden size the row kernels cover (2048) and largest head dimension (80)
WIDEST = I.ModelDesc(depth=1, hidden=2048, heads=32, mlp_dim=2304, patch=1, latent_c=4, latent_h=6, latent_w=7,
                     num_classes=5)
HEAD80 = I.ModelDesc(depth=1, hidden=320, heads=4, mlp_dim=640, patch=2, latent_c=4, latent_h=12, latent_w=10,
                     num_classes=5)
# Every stored tensor is the float32 rounding of an exactly evaluated value and every quantiser decides as the oracle
# does (each fused quantiser is checked alone in tests/test_gpu_quantisers.py; the fc1 epilogue and the attention kernel
# decide again in float64 where their fast arithmetic lands too close to a rounding boundary), so the device's tensors
# and codes are the oracle's bit for bit apart from double-rounding ties.  The tensors inside a block (the cached module
# outputs, Q | K | V) are held to the same bar as the block output, and the codes may differ in at most 1e-6 of the cases.
MAX_FLIP_FRACTION = 1e-6
INNER_MAX_ABS, INNER_REL_RMS = 1e-2, 1e-3


def _cuda(a, dtype=None):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a))
    if dtype is not None:
        t = t.to(dtype)
    return t.cuda()


def _block_case(model, seed, B, std=0.02, wb=8):
    """Single-block parity on random tokens and conditioning."""
    import torch
    import paper_2503_02508_amd as qc
    from dataclasses import replace
    model = replace(I.shrink(model, 1), weight_bits=wb)
    w = I.make_weights(model, seed, std=std)
    tok = I.make_tokens(B, model, seed + 1)
    cond = I.make_cond(B, model, seed + 2, std=0.5)
    qp, _ = sampler.calibrate_block(model, w, I.make_tokens(4, model, seed + 3), I.make_cond(4, model, seed + 4, std=0.5))
    lin, ctx = make_pair(model, w, qp, B)
    ctx.keep_qkv_f32(True)
    lin.taps = {}
    cache, tap = {}, {}
    want = dit.block_full(tok.astype(np.float64), cond.astype(np.float64), 0, model.heads, lin, cache, tap)
    x = _cuda(tok)
    c = _cuda(cond)
    ctx.dit_block(0, qc.QC_FULL, x, c)
    torch.cuda.synchronize()
    got = x.cpu().numpy()
    M, D, R = B * model.tokens, model.hidden, model.mlp_dim
    res = {
        "x": (got, want),
        "A": (ctx.cache_tensor(0, qc.QC_CACHE_ATTN, B).cpu().numpy(), cache[(0, "attn")]),
        "Mo": (ctx.cache_tensor(0, qc.QC_CACHE_MLP, B).cpu().numpy(), cache[(0, "mlp")]),
        "qkv": (ctx.workspace("qkv", (M, 3 * D), torch.float32).cpu().numpy(), tap["qkv"].reshape(M, 3 * D)),
    }
    flips = {
        "attn": code_flip_stats(ctx.workspace("qact_attn", (M, D), torch.int8).cpu().numpy(), lin.taps[(0, "proj")]["codes"]),
        "ln2": code_flip_stats(ctx.workspace("qact_ln", (M, D), torch.int8).cpu().numpy(), lin.taps[(0, "fc1")]["codes"]),
        "gelu": code_flip_stats(ctx.workspace("qact_mlp", (M, R), torch.int8).cpu().numpy(), lin.taps[(0, "fc2")]["codes"]),
    }
    # cached pass on the fresh cache from the same input must reproduce the full pass
    x2 = _cuda(tok)
    ctx.dit_block(0, qc.QC_CACHED, x2, c)
    torch.cuda.synchronize()
    res["x_cached"] = (x2.cpu().numpy(), got)
    want_cached = dit.block_cached(tok.astype(np.float64), cond.astype(np.float64), 0, lin, cache)
    assert np.array_equal(want_cached, want)
    ctx.close()
    return res, flips


@pytest.mark.parametrize("name,model,B,wb", [
    ("cfg0_dit_s2", I.DIT_S2_1BLOCK, 1, 8),
    ("dit_s2_b3", I.DIT_S2_1BLOCK, 3, 8),
    ("xl_256_b2", I.DIT_XL2_256, 2, 8),
    ("xl_256_b2_w4", I.DIT_XL2_256, 2, 4),
    ("tiny", TINY, 2, 8),
    ("ragged", RAGGED, 3, 8),
    ("ragged_w4", RAGGED, 3, 4),
    ("widest_hidden_2048", WIDEST, 2, 8),
    ("head_dim_80", HEAD80, 2, 8),
])
def test_block_full_and_cached_parity(name, model, B, wb):
    std = 0.02 if model.hidden >= 384 else 0.15
    res, flips = _block_case(model, 11, B, std=std, wb=wb)
    report = ["%s: max-abs %.2e rel-RMS %.2e" % (k, max_abs(g, w), rel_rms(g, w)) for k, (g, w) in res.items()]
    report += ["%s flips: %.2e (max dist %d)" % (k, f, d) for k, (f, d) in flips.items()]
    print(name, "; ".join(report))
    for k, (got, want) in res.items():
        if k in ("A", "Mo", "qkv"):
            assert_close(got, want, "%s/%s" % (name, k), INNER_MAX_ABS, INNER_REL_RMS)
        else:
            assert_close(got, want, "%s/%s" % (name, k), 1e-2, 1e-3 if k != "x_cached" else 1e-6)
    for k, (frac, dist) in flips.items():
        assert dist <= 1, "%s/%s codes differ by %d steps" % (name, k, dist)
        assert frac <= MAX_FLIP_FRACTION, "%s/%s: %.2e of the codes differ" % (name, k, frac)


def test_cached_block_needs_a_stored_cache():
    import torch
    import paper_2503_02508_amd as qc
    model = I.shrink(TINY, 1)
    w = I.make_weights(model, 3, std=0.15)
    qp = {(0, s): (np.float32(0.05), 128) for s in dit.SITES}
    _, ctx = make_pair(model, w, qp, 2)
    x = torch.zeros((2, model.tokens, model.hidden), device="cuda")
    c = torch.zeros((2, model.hidden), device="cuda")
    with pytest.raises(qc.QCError) as e:
        ctx.dit_block(0, qc.QC_CACHED, x, c)
    assert e.value.code == -5
    ctx.dit_block(0, qc.QC_FULL, x, c)
    ctx.dit_block(0, qc.QC_CACHED, x, c)
    with pytest.raises(qc.QCError) as e:           # other batch size than the stored one
        ctx.dit_block(0, qc.QC_CACHED, x[:1], c[:1])
    assert e.value.code == -5
    with pytest.raises(qc.QCError) as e:
        ctx.dit_block(0, qc.QC_FULL, torch.zeros((3, model.tokens, model.hidden), device="cuda"),
                      torch.zeros((3, model.hidden), device="cuda"))
    assert e.value.code == -2
    ctx.close()


def test_cache_store_and_reuse_calls():
    import torch
    import paper_2503_02508_amd as qc
    model = I.shrink(TINY, 1)
    w = I.make_weights(model, 3, std=0.15)
    qp = {(0, s): (np.float32(0.05), 128) for s in dit.SITES}
    _, ctx = make_pair(model, w, qp, 2)
    rng = np.random.default_rng(0)
    src = rng.standard_normal((2, model.tokens, model.hidden)).astype(np.float32)
    x = rng.standard_normal(src.shape).astype(np.float32)
    gate = rng.standard_normal((2, 6 * model.hidden)).astype(np.float32)
    ctx.cache_store(0, qc.QC_CACHE_MLP, _cuda(src))
    xd, gd = _cuda(x), _cuda(gate)
    g = gd[:, model.hidden:2 * model.hidden]
    ctx.cache_reuse(0, qc.QC_CACHE_MLP, xd, g)
    torch.cuda.synchronize()
    want = x.astype(np.float64) + gate[:, None, model.hidden:2 * model.hidden].astype(np.float64) * src
    assert np.max(np.abs(xd.cpu().numpy() - want)) < 1e-5
    assert np.array_equal(ctx.cache_tensor(0, qc.QC_CACHE_MLP, 2).cpu().numpy(), src)
    with pytest.raises(qc.QCError) as e:
        ctx.cache_reuse(0, qc.QC_CACHE_ATTN, xd, g)
    assert e.value.code == -5
    ctx.close()


# ------------------------------------------------------------ whole network
def _denoise_case(model, seed, B, t, std, guidance=False, wb=8, stream="fp32"):
    import torch
    import paper_2503_02508_amd as qc
    from dataclasses import replace
    model = replace(model, weight_bits=wb)
    w = I.make_weights(model, seed, std=std)
    clat = np.concatenate([I.make_latents(1, model, 4000 + i) for i in range(4)])
    clab = I.make_labels(4, model, seed + 9)
    qp, _, _ = oracle_calibration(model, w, lat=clat, lab=clab, t=np.full(4, t))
    Beff = 2 * B if guidance else B
    lin, ctx = make_pair(model, w, qp, Beff)
    ctx.set_stream_format(stream)
    lat = I.make_latents(B, model, seed + 1)
    lab = I.make_labels(B, model, seed + 2)
    xin = np.concatenate([lat, lat]) if guidance else lat
    yin = np.concatenate([lab, np.full(B, model.num_classes)]) if guidance else lab
    cache = {}
    with dit.stream_format({"fp32": "f32", "bf16": "bf16"}[stream]):
        want_full = dit.denoiser(xin, np.full(Beff, t), yin, model, w, lin, cache, True)
        want_cached = dit.denoiser(xin, np.full(Beff, t - 7), yin, model, w, lin, cache, False)
    eps = torch.empty((Beff, model.latent_c, model.latent_h, model.latent_w), device="cuda")
    xd, ld = _cuda(lat), _cuda(lab.astype(np.int32))
    ctx.denoise(xd, t, ld, Beff, qc.QC_FULL, eps)
    torch.cuda.synchronize()
    got_full = eps.cpu().numpy()
    got_A = [ctx.cache_tensor(l, qc.QC_CACHE_ATTN, Beff).cpu().numpy() for l in range(model.depth)]
    got_M = [ctx.cache_tensor(l, qc.QC_CACHE_MLP, Beff).cpu().numpy() for l in range(model.depth)]
    ctx.denoise(xd, t - 7, ld, Beff, qc.QC_CACHED, eps)
    torch.cuda.synchronize()
    got_cached = eps.cpu().numpy()
    ctx.close()
    return (got_full, want_full), (got_cached, want_cached), [(got_A[l], cache[(l, "attn")]) for l in range(model.depth)], \
        [(got_M[l], cache[(l, "mlp")]) for l in range(model.depth)]


@pytest.mark.parametrize("name,model,B,std,guidance,wb", [
    ("tiny", TINY, 3, 0.15, False, 8),
    ("tiny_cfg", TINY, 2, 0.15, True, 8),
    ("ragged", RAGGED, 2, 0.15, False, 8),
    ("cfg0_dit_s2", I.DIT_S2_1BLOCK, 1, 0.02, False, 8),
    ("xl_256_depth2", I.shrink(I.DIT_XL2_256, 2), 2, 0.02, False, 8),
    ("xl_256_depth2_w4_cfg", I.shrink(I.DIT_XL2_256, 2), 1, 0.02, True, 4),
])
def test_denoiser_full_and_cached_parity(name, model, B, std, guidance, wb):
    full, cached, As, Ms = _denoise_case(model, 21, B, 500, std, guidance, wb)
    print(name, "eps full max-abs %.2e rel-RMS %.2e; cached max-abs %.2e rel-RMS %.2e" % (
        max_abs(*full), rel_rms(*full), max_abs(*cached), rel_rms(*cached)))
    r = [assert_close(*full, name + "/eps_full"), assert_close(*cached, name + "/eps_cached")]
    for l, (a, m) in enumerate(zip(As, Ms)):
        ra = assert_close(*a, "%s/attn_out[%d]" % (name, l), INNER_MAX_ABS, INNER_REL_RMS)
        rm = assert_close(*m, "%s/mlp_out[%d]" % (name, l), INNER_MAX_ABS, INNER_REL_RMS)
        print("   block %d: attn_out max-abs %.2e rel-RMS %.2e; mlp_out max-abs %.2e rel-RMS %.2e" % ((l,) + ra + rm))
    print(name, "eps full max-abs %.2e rel-RMS %.2e; cached max-abs %.2e rel-RMS %.2e" % (r[0] + r[1]))


def _sampler_case(wl_model, B, steps, interval, n_run, cfg, std, seed=31, wb=8, free_running=False):
    """Teacher-forced (default): at every step the device starts from the
    oracle's sample.  Free-running: the device carries its own sample."""
    import torch
    import paper_2503_02508_amd as qc
    from dataclasses import replace
    model = replace(wl_model, weight_bits=wb)
    w = I.make_weights(model, seed, std=std)
    tt, at, ap = sampler.ddim_schedule(steps)
    idx = np.array([0, steps // 3, 2 * steps // 3, steps - 1])
    clat = np.concatenate([I.make_latents(1, model, 4000 + i) for i in range(4)])
    qp, _, _ = oracle_calibration(model, w, lat=clat, lab=I.make_labels(4, model, seed + 9), t=tt[idx])
    Beff = 2 * B if cfg > 0 else B
    lin, ctx = make_pair(model, w, qp, Beff, interval)
    assert qc.qc_ddim_schedule(steps)[0] == list(tt)
    lat = I.make_latents(B, model, seed + 1)
    lab = I.make_labels(B, model, seed + 2)
    K = I.make_vc_factors(steps, model.latent_c, seed + 3)
    Kd, ld = _cuda(K), _cuda(lab.astype(np.int32))
    x_or = lat.astype(np.float64)
    xd = _cuda(lat)
    cache = {}
    errs = []
    for i in range(n_run):
        if not free_running:
            xd = _cuda(x_or.astype(np.float32))
            x_start = xd.cpu().numpy().astype(np.float64)      # the oracle continues from the fp32 value the device sees
        else:
            x_start = x_or
        x_or, _ = sampler.sample_step(x_start, lab, i, int(tt[i]), at[i], ap[i], model, w, lin, cache, interval, cfg, K[i])
        ctx.sample_step(xd, ld, i, int(tt[i]), float(at[i]), float(ap[i]), cfg, Kd[i])
        torch.cuda.synchronize()
        got = xd.cpu().numpy()
        errs.append((max_abs(got, x_or), rel_rms(got, x_or)))
    ctx.close()
    return errs, got, x_or


@pytest.mark.parametrize("name,model,B,steps,interval,n_run,cfg,std,wb", [
    ("tiny_n2", TINY, 3, 10, 2, 10, 0.0, 0.15, 8),
    ("tiny_n3_cfg", TINY, 2, 10, 3, 7, 1.5, 0.15, 8),
    ("ragged_n2", RAGGED, 2, 8, 2, 5, 0.0, 0.15, 8),
    ("xl_256_depth2_n2", I.shrink(I.DIT_XL2_256, 2), 2, 50, 2, 5, 0.0, 0.02, 8),
    ("xl_256_depth2_n3_cfg", I.shrink(I.DIT_XL2_256, 2), 1, 100, 3, 7, 1.5, 0.02, 8),
    ("xl_256_depth2_n5_w4", I.shrink(I.DIT_XL2_256, 2), 1, 250, 5, 11, 0.0, 0.02, 4),
])
def test_sampler_steps_teacher_forced(name, model, B, steps, interval, n_run, cfg, std, wb):
    errs, _, _ = _sampler_case(model, B, steps, interval, n_run, cfg, std, wb=wb)
    print(name, " ".join("%d:%.1e/%.1e" % (i, ma, rr) for i, (ma, rr) in enumerate(errs)))
    for i, (ma, rr) in enumerate(errs):
        assert ma <= 1e-2 and rr <= 1e-3, "%s step %d: max-abs %.2e rel-RMS %.2e" % (name, i, ma, rr)
    print(name, "worst max-abs %.2e rel-RMS %.2e" % (max(e[0] for e in errs), max(e[1] for e in errs)))


def test_sampler_free_running_whole_loop_via_qc_sample():
    """qc_sample (the whole loop, device carries its own sample) against the oracle loop."""
    import torch
    import paper_2503_02508_amd as qc
    model, steps, interval, B = TINY, 10, 2, 3
    w = I.make_weights(model, 41, std=0.15)
    tt, _, _ = sampler.ddim_schedule(steps)
    clat = np.concatenate([I.make_latents(1, model, 4000 + i) for i in range(4)])
    qp, _, _ = oracle_calibration(model, w, lat=clat, lab=I.make_labels(4, model, 50), t=tt[[0, 3, 6, 9]])
    lin, ctx = make_pair(model, w, qp, B, interval)
    lat, lab = I.make_latents(B, model, 42), I.make_labels(B, model, 43)
    K = I.make_vc_factors(steps, model.latent_c, 44)
    want = sampler.sample(lat, lab, steps, interval, model, w, lin, 0.0, K)
    xd = _cuda(lat)
    ctx.sample(xd, _cuda(lab.astype(np.int32)), steps, 0.0, _cuda(K))
    torch.cuda.synchronize()
    got = xd.cpu().numpy()
    ma, rr = max_abs(got, want), rel_rms(got, want)
    print("free-running tiny: max-abs %.2e rel-RMS %.2e (|x| rms %.2f)" % (ma, rr, np.sqrt(np.mean(want ** 2))))
    assert rr <= 1e-3 and ma <= 1e-2
    ctx.close()


@pytest.mark.parametrize("B,steps,interval,cfg", [(3, 10, 2, 0.0), (8, 150, 3, 0.0), (5, 120, 4, 1.5)])
def test_qc_sample_equals_step_by_step_calls(B, steps, interval, cfg):
    """The whole-loop entry point prepares the conditioning and the adaLN projections of many steps with
    one launch each (several windows at the larger step counts); its samples must be bit-identical to
    the ones the per-step entry point produces."""
    import torch
    import paper_2503_02508_amd as qc
    model = TINY
    w = I.make_weights(model, 61, std=0.15)
    tt, at, ap = sampler.ddim_schedule(steps)
    clat = np.concatenate([I.make_latents(1, model, 4000 + i) for i in range(4)])
    qp, _, _ = oracle_calibration(model, w, lat=clat, lab=I.make_labels(4, model, 62), t=tt[[0, steps // 3, 2 * steps // 3, steps - 1]])
    Beff = 2 * B if cfg > 0 else B
    _, ctx = make_pair(model, w, qp, Beff, interval)
    lat, lab = I.make_latents(B, model, 63), _cuda(I.make_labels(B, model, 64).astype(np.int32))
    K = _cuda(I.make_vc_factors(steps, model.latent_c, 65))
    xa, xb = _cuda(lat), _cuda(lat)
    ctx.sample(xa, lab, steps, cfg, K)
    for i in range(steps):
        ctx.sample_step(xb, lab, i, int(tt[i]), float(at[i]), float(ap[i]), cfg, K[i])
    torch.cuda.synchronize()
    assert torch.isfinite(xa).all()
    assert torch.equal(xa, xb)
    ctx.close()


def _random_mask(steps, depth, seed, p_full=0.5):
    rng = np.random.default_rng(seed)
    m = (rng.random((steps, depth, 2)) < p_full).astype(np.uint8)
    m[0] = 1
    return m


@pytest.mark.parametrize("name,model,B,steps,cfg", [("tiny", TINY, 3, 9, 0.0), ("tiny_cfg", TINY, 2, 8, 1.5),
                                                    ("ragged", RAGGED, 2, 7, 0.0),
                                                    ("xl_256_depth2", I.shrink(I.DIT_XL2_256, 2), 2, 6, 0.0)])
def test_sampler_with_per_module_cache_schedule(name, model, B, steps, cfg):
    """A random per-(step, block, module) schedule: mixed steps recompute some modules and reuse others.
    Teacher-forced against the oracle step by step, then the whole loop through qc_sample."""
    import torch
    std = 0.02 if model.hidden > 256 else 0.15
    w = I.make_weights(model, 71, std=std)
    tt, at, ap = sampler.ddim_schedule(steps)
    clat = np.concatenate([I.make_latents(1, model, 4000 + i) for i in range(4)])
    qp, _, _ = oracle_calibration(model, w, lat=clat, lab=I.make_labels(4, model, 72), t=tt[[0, steps // 3, 2 * steps // 3, steps - 1]])
    Beff = 2 * B if cfg > 0 else B
    lin, ctx = make_pair(model, w, qp, Beff, 2)
    mask = _random_mask(steps, model.depth, 73)
    assert 0 < mask[1:].mean() < 1
    ctx.set_cache_mask(mask)
    lat, lab = I.make_latents(B, model, 74), I.make_labels(B, model, 75)
    K = I.make_vc_factors(steps, model.latent_c, 76)
    Kd, ld = _cuda(K), _cuda(lab.astype(np.int32))
    x_or, cache = lat.astype(np.float64), {}
    worst = (0.0, 0.0)
    for i in range(steps):
        xd = _cuda(x_or.astype(np.float32))
        x_start = xd.cpu().numpy().astype(np.float64)
        x_or, _ = sampler.sample_step(x_start, lab, i, int(tt[i]), at[i], ap[i], model, w, lin, cache, 2, cfg, K[i], mask[i])
        ctx.sample_step(xd, ld, i, int(tt[i]), float(at[i]), float(ap[i]), cfg, Kd[i])
        got = xd.cpu().numpy()
        ma, rr = max_abs(got, x_or), rel_rms(got, x_or)
        assert ma <= 1e-2 and rr <= 1e-3, "%s step %d: max-abs %.2e rel-RMS %.2e" % (name, i, ma, rr)
        worst = (max(worst[0], ma), max(worst[1], rr))
    print(name, "per-module schedule, teacher-forced: worst max-abs %.2e rel-RMS %.2e" % worst)
    # whole loop: qc_sample under the schedule equals the per-step calls bit for bit
    xa, xb = _cuda(lat), _cuda(lat)
    ctx.sample(xa, ld, steps, cfg, Kd)
    for i in range(steps):
        ctx.sample_step(xb, ld, i, int(tt[i]), float(at[i]), float(ap[i]), cfg, Kd[i])
    torch.cuda.synchronize()
    assert torch.equal(xa, xb)
    # more steps than the schedule holds is an error, and so is reusing a module that was never stored
    with pytest.raises(Exception):
        ctx.sample(xa, ld, steps + 1, cfg, Kd)
    ctx.close()


def test_schedule_written_from_the_interval_rule_is_the_interval_sampler():
    import torch
    model, B, steps, N = TINY, 3, 10, 3
    w = I.make_weights(model, 81, std=0.15)
    tt, _, _ = sampler.ddim_schedule(steps)
    clat = np.concatenate([I.make_latents(1, model, 4000 + i) for i in range(4)])
    qp, _, _ = oracle_calibration(model, w, lat=clat, lab=I.make_labels(4, model, 82), t=tt[[0, 3, 6, 9]])
    _, ctx = make_pair(model, w, qp, B, N)
    lat, lab = _cuda(I.make_latents(B, model, 83)), _cuda(I.make_labels(B, model, 84).astype(np.int32))
    K = _cuda(I.make_vc_factors(steps, model.latent_c, 85))
    xa, xb = lat.clone(), lat.clone()
    ctx.sample(xa, lab, steps, 0.0, K)
    mask = np.zeros((steps, model.depth, 2), np.uint8)
    mask[::N] = 1
    ctx.set_cache_mask(mask)
    ctx.sample(xb, lab, steps, 0.0, K)
    torch.cuda.synchronize()
    assert torch.equal(xa, xb)
    ctx.set_cache_mask(None)
    ctx.close()


@pytest.mark.parametrize("name,model,B,steps,interval,cfg", [
    ("tiny_n2", TINY, 3, 8, 2, 0.0), ("ragged_n3_cfg", RAGGED, 2, 7, 3, 1.5),
    ("xl_256_depth2_n2", I.shrink(I.DIT_XL2_256, 2), 2, 50, 2, 0.0)])
def test_sampler_with_bf16_cache(name, model, B, steps, interval, cfg):
    """Reduced-precision cache storage: the stored tensors are the bfloat16 rounding of the fp32 ones (bit for bit,
    up to values the two sides computed differently within fp32 rounding), and the sampler stays inside the bar
    against the oracle run with the same storage."""
    import torch
    n_run = min(steps, 2 * interval + 1)
    std = 0.02 if model.hidden > 256 else 0.15
    w = I.make_weights(model, 91, std=std)
    tt, at, ap = sampler.ddim_schedule(steps)
    clat = np.concatenate([I.make_latents(1, model, 4000 + i) for i in range(4)])
    qp, _, _ = oracle_calibration(model, w, lat=clat, lab=I.make_labels(4, model, 92), t=tt[[0, steps // 3, 2 * steps // 3, steps - 1]])
    Beff = 2 * B if cfg > 0 else B
    lin, ctx = make_pair(model, w, qp, Beff, interval)
    ctx.set_cache_format("bf16")
    lat, lab = I.make_latents(B, model, 93), I.make_labels(B, model, 94)
    K = I.make_vc_factors(steps, model.latent_c, 95)
    Kd, ld = _cuda(K), _cuda(lab.astype(np.int32))
    x_or, cache = lat.astype(np.float64), {}
    worst = (0.0, 0.0)
    for i in range(n_run):
        xd = _cuda(x_or.astype(np.float32))
        x_start = xd.cpu().numpy().astype(np.float64)
        x_or, _ = sampler.sample_step(x_start, lab, i, int(tt[i]), at[i], ap[i], model, w, lin, cache, interval, cfg, K[i],
                                      cache_bf16=True)
        ctx.sample_step(xd, ld, i, int(tt[i]), float(at[i]), float(ap[i]), cfg, Kd[i])
        got = xd.cpu().numpy()
        ma, rr = max_abs(got, x_or), rel_rms(got, x_or)
        assert ma <= 1e-2 and rr <= 1e-3, "%s step %d: max-abs %.2e rel-RMS %.2e" % (name, i, ma, rr)
        worst = (max(worst[0], ma), max(worst[1], rr))
        if i == 0:
            # what the refresh step stored: bfloat16 values, equal to the oracle's rounding wherever the two
            # fp32 values agree to well below a bfloat16 step
            for which, key in ((0, "attn"), (1, "mlp")):
                dev = ctx.cache_tensor(0, which, Beff).float().cpu().numpy().astype(np.float64)
                ref = cache[(0, key)]
                # the stored tensor against the oracle's: the floating-point bar (flipped activation codes move the
                # fp32 value before rounding) plus one bfloat16 step; what is stored must be bfloat16 values.  The
                # rounding itself is checked bit for bit in test_bf16_cache_store_and_reuse_calls.
                excess = np.abs(dev - ref) - (np.abs(ref) * 2.0 ** -7 + 1e-2)
                assert excess.max() <= 0, "%s cache %s differs by more than one bf16 step (%.2e)" % (name, key, excess.max())
                assert rel_rms(dev, ref) <= 1e-3 + 2.0 ** -8
                assert np.array_equal(quant.bf16_round(dev), dev), "%s cache %s holds values that are not bfloat16" % (name, key)
    print(name, "bf16 cache: worst max-abs %.2e rel-RMS %.2e" % worst)
    # switching the format discards the cache: a cached step must now be refused
    ctx.set_cache_format("fp32")
    with pytest.raises(Exception):
        ctx.sample_step(xd, ld, 1, int(tt[1]), float(at[1]), float(ap[1]), cfg, Kd[1], 1)
    ctx.close()


def test_bf16_cache_store_and_reuse_calls():
    import torch
    import paper_2503_02508_amd as qc
    from oracle import quant
    model, B = TINY, 2
    w = I.make_weights(model, 96, std=0.15)
    qp = {(b, s): quant.act_qparams(-4, 4) for b in range(model.depth) for s in dit.SITES}
    _, ctx = make_pair(model, w, qp, B, 2)
    ctx.set_cache_format("bf16")
    rng = np.random.default_rng(97)
    src = rng.standard_normal((B, model.tokens, model.hidden)).astype(np.float32)
    x = rng.standard_normal((B, model.tokens, model.hidden)).astype(np.float32)
    gate = rng.standard_normal((B, model.hidden)).astype(np.float32)
    ctx.cache_store(1, qc.QC_CACHE_MLP, _cuda(src))
    stored = ctx.cache_tensor(1, qc.QC_CACHE_MLP, B).float().cpu().numpy()
    assert np.array_equal(stored.astype(np.float64), quant.bf16_round(src))
    xd = _cuda(x)
    ctx.cache_reuse(1, qc.QC_CACHE_MLP, xd, _cuda(gate))
    want = x.astype(np.float64) + gate[:, None, :].astype(np.float64) * quant.bf16_round(src)
    assert max_abs(xd.cpu().numpy(), want) <= 1e-5
    ctx.close()


def test_a_refused_calibration_leaves_the_parameters_alone():
    """The range of one site is infinite: none of the others is installed."""
    import torch
    import paper_2503_02508_amd as qc
    model = I.shrink(TINY, 1)
    w = I.make_weights(model, 5)
    w["blocks"][0]["fc1_b"][0] = np.inf                       # the input of fc2
    ctx = qc.Context(model, 1, 1)
    ctx.load_weights(w, keep_fp32=True)
    for site in range(5):
        ctx.set_act_qparams(0, site, 0.5 + site, 100 + site)
    with pytest.raises(qc.QCError) as e:
        ctx.calibrate(_cuda(I.make_latents(1, model, 6)), [500], [3])
    assert e.value.code == -4
    assert [ctx.get_act_qparams(0, site) for site in range(5)] == [(0.5 + site, 100 + site) for site in range(5)]
    ctx.close()


def test_calibration_matches_oracle():
    """qc_calibrate_minmax (fp32 un-quantised forward on the device) against the oracle's calibration."""
    import torch
    import paper_2503_02508_amd as qc
    for model, std in [(TINY, 0.15), (I.DIT_S2_1BLOCK, 0.02), (I.shrink(I.DIT_XL2_256, 2), 0.02)]:
        w = I.make_weights(model, 51, std=std)
        clat = np.concatenate([I.make_latents(1, model, 4000 + i) for i in range(4)])
        clab = I.make_labels(4, model, 52)
        t = np.array([980, 660, 320, 0])
        qp, ranges, _ = oracle_calibration(model, w, lat=clat, lab=clab, t=t)
        ctx = qc.Context(model, 1, 1)
        ctx.load_weights(w, keep_fp32=True)
        ctx.calibrate(_cuda(clat), t, clab)
        for (blk, site), (s, z) in qp.items():
            gs, gz = ctx.get_act_qparams(blk, dit.SITES.index(site))
            assert abs(gs - float(s)) <= 2e-5 * float(s), (blk, site, gs, s)
            assert abs(gz - z) <= 1, (blk, site, gz, z)
        ctx.close()


def test_out_of_range_label_is_clamped_and_reported():
    """Labels live on the device: a label outside [0, num_classes] is clamped by the conditioning kernel, the run
    completes with the clamped label's result, and qc_check reports QC_ERR_RANGE once."""
    import torch
    import paper_2503_02508_amd as qc
    model = TINY
    w = I.make_weights(model, 5, std=0.15)
    ctx = qc.Context(model, 2, 1)
    ctx.load_weights(w)
    for blk in range(model.depth):
        for site in range(5):
            ctx.set_act_qparams(blk, site, 0.05, 128)
    x = _cuda(I.make_latents(2, model, 6))
    eps_bad, eps_ok = torch.empty_like(x), torch.empty_like(x)
    ctx.check()                                                       # nothing flagged yet
    ctx.denoise(x, 300, _cuda(np.array([1, model.num_classes + 7], dtype=np.int32)), 2, qc.QC_FULL, eps_bad)
    with pytest.raises(qc.QCError) as e:
        ctx.check()
    assert e.value.code == -4
    ctx.check()                                                       # reported once, then cleared
    ctx.denoise(x, 300, _cuda(np.array([1, model.num_classes], dtype=np.int32)), 2, qc.QC_FULL, eps_ok)
    ctx.check()
    assert torch.equal(eps_bad, eps_ok)
    ctx.close()


@pytest.mark.parametrize("name,model,B,std,guidance,wb", [
    ("tiny", TINY, 3, 0.15, False, 8),
    ("ragged_cfg", RAGGED, 2, 0.15, True, 8),
    ("xl_256_depth2", I.shrink(I.DIT_XL2_256, 2), 2, 0.02, False, 8),
    ("xl_256_depth2_large_m_w4", I.shrink(I.DIT_XL2_256, 2), 40, 0.02, False, 4),     # M = 10240: the large-M GEMM's epilogues
])
def test_denoiser_with_bf16_residual_stream(name, model, B, std, guidance, wb):
    """Reduced-precision variant: the token tensor is stored as bfloat16 (embedding output and the stream after every
    gated add) on both sides; everything else as in the float32-stream test, to the same bar."""
    full, cached, As, Ms = _denoise_case(model, 23, B, 500, std, guidance, wb, stream="bf16")
    r = [assert_close(*full, name + "/eps_full"), assert_close(*cached, name + "/eps_cached")]
    for l, (a, m) in enumerate(zip(As, Ms)):
        assert_close(*a, "%s/attn_out[%d]" % (name, l), INNER_MAX_ABS, INNER_REL_RMS)
        assert_close(*m, "%s/mlp_out[%d]" % (name, l), INNER_MAX_ABS, INNER_REL_RMS)
    print(name, "bf16 stream: eps full max-abs %.2e rel-RMS %.2e; cached max-abs %.2e rel-RMS %.2e" % (r[0] + r[1]))
    # and it is a different computation from the float32-stream one
    full32, _, _, _ = _denoise_case(model, 23, min(B, 2), 500, std, guidance, wb) if B <= 3 else (None, None, None, None)
    if full32 is not None:
        assert not np.array_equal(full32[0], full[0][:full32[0].shape[0]])


@pytest.mark.parametrize("name,model,B,steps,interval,cfg", [
    ("tiny_n2", TINY, 3, 8, 2, 0.0), ("ragged_n3_cfg", RAGGED, 2, 7, 3, 1.5),
    ("xl_256_depth2_n2", I.shrink(I.DIT_XL2_256, 2), 2, 50, 2, 0.0)])
def test_sampler_with_bf16_stream_and_bf16_cache(name, model, B, steps, interval, cfg):
    """Both reduced-precision storage variants together, through the whole free-running loop (qc_sample): bfloat16
    residual stream and bfloat16 cache on both sides, final latents to the bar."""
    import torch
    std = 0.02 if model.hidden > 256 else 0.15
    w = I.make_weights(model, 191, std=std)
    tt, at, ap = sampler.ddim_schedule(steps)
    clat = np.concatenate([I.make_latents(1, model, 4000 + i) for i in range(4)])
    qp, _, _ = oracle_calibration(model, w, lat=clat, lab=I.make_labels(4, model, 192), t=tt[[0, steps // 3, 2 * steps // 3, steps - 1]])
    Beff = 2 * B if cfg > 0 else B
    lin, ctx = make_pair(model, w, qp, Beff, interval)
    ctx.set_cache_format("bf16")
    ctx.set_stream_format("bf16")
    lat, lab = I.make_latents(B, model, 193), I.make_labels(B, model, 194)
    n_run = min(steps, 3 * interval + 1)
    K = I.make_vc_factors(steps, model.latent_c, 195)
    xd = _cuda(lat)
    x_or, cache = lat.astype(np.float64), {}
    with dit.stream_format("bf16"):
        for i in range(n_run):
            x_or, _ = sampler.sample_step(x_or, lab, i, int(tt[i]), at[i], ap[i], model, w, lin, cache, interval, cfg, K[i],
                                          cache_bf16=True)
    Kd, ld = _cuda(K), _cuda(lab.astype(np.int32))
    for i in range(n_run):
        ctx.sample_step(xd, ld, i, int(tt[i]), float(at[i]), float(ap[i]), cfg, Kd[i])
    torch.cuda.synchronize()
    got = xd.cpu().numpy()
    ma, rr = max_abs(got, x_or), rel_rms(got, x_or)
    print(name, "bf16 stream + cache, %d free-running steps: max-abs %.2e rel-RMS %.2e" % (n_run, ma, rr))
    assert ma <= 1e-2 and rr <= 1e-3
    tok = ctx.workspace("tokens", (Beff, model.tokens, model.hidden), torch.bfloat16)
    assert torch.isfinite(tok.float()).all()
    ctx.close()
