"""Kernel variants that a launch size picks: each against the other variant, bit for bit, or against the oracle, at the
sizes where the choice changes and where tiles have remainders."""
from dataclasses import replace

import numpy as np
import pytest

from synthetic import dit_inputs as I

pytestmark = pytest.mark.gpu


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("hidden,heads,mlp,hw,B", [(1152, 16, 4608, (32, 32), 3),      # both tile sizes of the float32 linear
                                                   (80, 4, 176, (10, 14), 5),          # remainders in rows, columns and k
                                                   (48, 4, 112, (64, 64), 2)])         # a whole group is one sample
def test_reference_forward_does_not_depend_on_the_batch(hidden, heads, mlp, hw, B):
    """The un-quantised forward of a batch (samples in groups, larger tiles) equals that of each latent alone."""
    import torch
    import paper_2503_02508_amd as qc
    m = I.ModelDesc(depth=1, hidden=hidden, heads=heads, mlp_dim=mlp, patch=2, latent_c=4, latent_h=hw[0], latent_w=hw[1])
    w = I.make_weights(m, 11)
    ctx = qc.Context(m, B, 1)
    ctx.load_weights(w, keep_fp32=True)
    x, lab = _cuda(I.make_latents(B, m, 12)), _cuda(I.make_labels(B, m, 13))
    eps, one = torch.empty_like(x), torch.empty_like(x)
    ctx.denoise_f32(x, 345, lab, B, eps)
    for b in range(B):
        ctx.denoise_f32(x[b:b + 1], 345, lab[b:b + 1], 1, one[b:b + 1])
    assert torch.equal(eps, one)
    assert float(eps.abs().max()) > 0


def _net(hidden, heads, mlp, h, w, patch=2):
    return I.ModelDesc(depth=1, hidden=hidden, heads=heads, mlp_dim=mlp, patch=patch, latent_c=4, latent_h=h, latent_w=w)


@pytest.mark.parametrize("name,model,B,wb", [
    ("attention: 36 features a head (packed tail, two chunks), 70 tokens", _net(144, 4, 576, 20, 14), 3, 8),
    ("attention: 72 features a head, 1 key past a tile", _net(288, 4, 512, 10, 26), 2, 8),
    ("attention: two query blocks a wavefront, 575 tokens", _net(256, 4, 512, 46, 50), 33, 8),
    ("attention: 16 features a head", _net(64, 4, 128, 16, 22), 2, 8),
    # keys in LDS: two tiles there, or one (76 and 80 features); one, two, three and more tiles of keys, the last one full, ragged or with a
    # single key; a packed tail of four features, padded feature chunks
    ("attention, one query block: 72 features, 64 tokens", _net(1152, 16, 1152, 16, 16), 9, 8),
    ("attention, one query block: 72 features, 128 tokens", _net(1152, 16, 1152, 16, 32), 5, 8),
    ("attention, one query block: 64 features, 192 tokens", _net(384, 6, 512, 24, 32), 9, 8),
    ("attention, one query block: 80 features, 260 tokens", _net(320, 4, 512, 20, 52), 9, 8),
    ("attention, one query block: 76 features, 35 tokens", _net(304, 4, 512, 10, 14), 36, 8),
    ("attention, two query blocks: 68 features, 193 tokens", _net(272, 4, 512, 2, 386), 34, 8),
    ("attention, two query blocks: 44 features, 256 tokens", _net(176, 4, 512, 32, 32), 33, 8),
    ("attention, two query blocks: 20 features, 129 tokens", _net(80, 4, 512, 6, 86), 34, 8),
    ("attention, two query blocks: 80 features, 200 tokens", _net(320, 4, 512, 20, 40), 33, 8),
    ("attention, two query blocks: 12 features, 320 tokens", _net(48, 4, 512, 32, 40), 22, 8),
    # keys shared by the wavefronts: two rounds of tiles, the second of three wavefronts (the last one's ragged); one tile for three
    # wavefronts and a half of queries; fewer keys than a tile, padded feature chunk; 80 features a head
    ("attention, shared keys: 425 tokens, 32 queries a workgroup", _net(1152, 16, 1152, 50, 34), 1, 8),
    ("attention, shared keys: 133 tokens, 64 features", _net(384, 6, 512, 14, 38), 1, 8),
    ("attention, shared keys: 35 tokens, 48 features", _net(192, 4, 512, 10, 14), 2, 8),
    ("attention, shared keys: 100 tokens, 80 features", _net(320, 4, 512, 20, 20), 3, 8),
    ("attention, shared keys: 260 tokens, 40 features", _net(160, 4, 512, 20, 52), 2, 8),
    ("split-K: one row past a 32-row tile, 4-bit", _net(128, 2, 512, 6, 22), 1, 4),
    ("split-K: 64 x 64 tiles with remainders", _net(384, 6, 1536, 30, 26), 2, 8),
    # more than 150 tiles of 128 x 256 that do not all lie inside one batch element: 425 tokens (no unit of four tokens is
    # whole), 252 tokens (units of four are), the last tile has 2 or 48 rows
    ("large-M, 425 tokens", _net(1152, 16, 4608, 50, 34), 10, 8),
    ("large-M, 252 tokens, 4-bit", _net(1152, 16, 4608, 36, 28), 20, 4),
    # 100 - 300 tiles of 64 x 256: 100 and 77 tokens (tiles that span batch elements, with and without whole units of four tokens; the
    # last tile has 52 and 31 rows), 64 tokens (one batch element a tile), residuals of 425 tokens (the last tile has 13 rows)
    ("64-row tiles, 100 tokens", _net(384, 6, 1536, 20, 20), 21, 8),
    ("64-row tiles, 77 tokens, 4-bit", _net(384, 6, 1536, 14, 22), 27, 4),
    ("64-row tiles, 64 tokens", _net(384, 6, 1536, 16, 16), 40, 8),
    # V^T of tiles whose tokens start anywhere in a unit of four: 2, 3, 1 tokens more than whole units; the last two in tiles of 128 rows
    ("64-row tiles, 78 tokens", _net(384, 6, 1536, 12, 26), 27, 8),
    ("64-row tiles, 91 tokens", _net(384, 6, 1536, 14, 26), 23, 8),
    ("large-M, 255 tokens, 64 features a head", _net(384, 6, 1536, 30, 34), 16, 8),
    ("large-M, 133 tokens, 64 features a head", _net(384, 6, 1536, 14, 38), 31, 8),
    ("64-row tiles, residuals, 425 tokens", _net(1152, 16, 4608, 50, 34), 5, 8),
    ("64-row tiles, residuals, 256 tokens, 4-bit", _net(1152, 16, 4608, 32, 32), 9, 4),
    ("split-K: 32 x 64 tiles in place of 252 of 64 x 64, 425 tokens", _net(1152, 16, 4608, 50, 34), 2, 8),
    ("split-K: 32 x 64 tiles in place of 288 of 64 x 64, 4-bit", _net(1152, 16, 4608, 32, 32), 1, 4),
    ("split-K: 64 x 96 tiles", _net(1152, 16, 4608, 32, 32), 4, 8),
    # chunks of K a wavefront of the MLP's second product walks, three of them in flight: 4 and 3, 5, 4
    ("split-K: 13 chunks", _net(512, 8, 1664, 20, 28), 2, 8),
    ("split-K: 20 chunks", _net(512, 8, 2560, 20, 28), 2, 8),
    ("split-K: 16 chunks, 4-bit", _net(512, 8, 2048, 20, 28), 2, 4),
])
def test_quantisers_of_small_and_ragged_launches(name, model, B, wb):
    from test_gpu_quantisers import test_each_fused_quantiser_alone as check
    check(name, model, B, wb, 0.02 if model.hidden > 1000 else 0.05)


@pytest.mark.parametrize("hw,B,wb", [((36, 28), 20, 4), ((36, 28), 20, 8), ((50, 34), 10, 4), ((50, 34), 10, 8)])
def test_large_m_ragged_block_repeats_itself(hw, B, wb):
    """Every run of a block whose large-M tiles span batch elements gives the same stored tensors from the same input, bit for bit."""
    import torch
    import paper_2503_02508_amd as qc
    from oracle import sampler
    from qc_testlib import make_pair, qkv_difference, qkv_rows_from_heads
    model = replace(_net(1152, 16, 4608, *hw), weight_bits=wb)
    w = I.make_weights(model, 77, std=0.02)
    D, T = model.hidden, model.tokens
    M = B * T
    tok, cond = _cuda(I.make_tokens(B, model, 78)), _cuda(I.make_cond(B, model, 79, std=0.5))
    qp, _ = sampler.calibrate_block(model, w, I.make_tokens(4, model, 80), I.make_cond(4, model, 81, std=0.5))
    _, ctx = make_pair(model, w, qp, B)

    def run():
        x = tok.clone()
        ctx.dit_block(0, qc.QC_FULL, x, cond)
        torch.cuda.synchronize()
        return dict(mod=ctx.workspace("mod", (512, 6 * D), torch.float32)[:B].clone(), qkv=qkv_rows_from_heads(ctx, model, B, B),
                    c_attn=ctx.workspace("qact_attn", (M, D), torch.int8).clone(), c_ln2=ctx.workspace("qact_ln", (M, D), torch.int8).clone(),
                    c_gelu=ctx.workspace("qact_mlp", (M, model.mlp_dim), torch.int8).clone(), x=x.reshape(M, D))

    first = run()
    for rep in range(7):
        again = run()
        for k in first:
            if not torch.equal(first[k], again[k]):
                where = qkv_difference(again[k].cpu().numpy(), first[k].cpu().numpy(), D) if k == "qkv" else "rows %s" % (
                    torch.nonzero((first[k] != again[k]).any(dim=1)).flatten()[:64].tolist())
                raise AssertionError("run %d: %s differs from the first run's: %s" % (rep + 2, k, where))
    ctx.close()


@pytest.mark.parametrize("cache,stream", [("fp32", "fp32"), ("bf16", "bf16")])
def test_large_m_ragged_denoiser(cache, stream):
    """Full and cached denoiser calls whose large-M tiles span batch elements, against the oracle with the same storage."""
    import torch
    import paper_2503_02508_amd as qc
    from oracle import dit
    from qc_testlib import assert_close, make_pair, oracle_calibration
    m = _net(1152, 16, 4608, 50, 34)
    B, n = 10, 5
    w = I.make_weights(m, 21)
    lat, lab = I.make_latents(n, m, 22), I.make_labels(n, m, 23)
    qp, _, _ = oracle_calibration(m, w, lat=lat[:2], lab=lab[:2], t=np.array([900, 100]))
    lin, ctx = make_pair(m, w, qp, B, 2)
    ctx.set_cache_format(cache)
    ctx.set_stream_format(stream)
    xd, ld = _cuda(lat), _cuda(lab)
    eps = torch.empty((B,) + lat.shape[1:], device="cuda")
    got = []
    for mode, t in ((qc.QC_FULL, 500), (qc.QC_CACHED, 480)):
        ctx.denoise(xd, t, ld, B, mode, eps)
        got.append(eps.cpu().numpy())
    ctx.close()
    # the oracle on three of the ten batch elements (they are independent): the first, one in the middle, the last
    for b in (0, 4, 9):
        cache_or = {}
        yb = np.array([lab[b % n] if b < n else m.num_classes])
        with dit.stream_format({"fp32": "f32", "bf16": "bf16"}[stream]):
            for k, (full, t) in enumerate(((True, 500), (False, 480))):
                want = dit.denoiser(lat[b % n][None].astype(np.float64), np.array([t]), yb, m, w, lin, cache_or, full, cache_bf16=cache == "bf16")
                assert_close(got[k][b], want[0], "batch element %d, call %d" % (b, k))


@pytest.mark.parametrize("cache,stream", [("fp32", "bf16"), ("bf16", "fp32"), ("bf16", "bf16")])
@pytest.mark.parametrize("hw,B", [((50, 34), 5), ((32, 32), 8)])
def test_64_row_tiles_equal_the_small_launches(hw, B, cache, stream):
    """Residual linears on 64-row tiles (a batch) against the small tiles of each latent alone, bit for bit, in every storage format."""
    import torch
    import paper_2503_02508_amd as qc
    from qc_testlib import make_pair, oracle_calibration
    m = _net(1152, 16, 4608, *hw)
    w = I.make_weights(m, 21)
    lat, lab = I.make_latents(B, m, 22), I.make_labels(B, m, 23)
    qp, _, _ = oracle_calibration(m, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    _, ctx = make_pair(m, w, qp, B, 2)
    ctx.set_cache_format(cache)
    ctx.set_stream_format(stream)
    xd, ld = _cuda(lat), _cuda(lab)
    got = [torch.empty(lat.shape, device="cuda") for _ in range(2)]
    for eps, mode, t in zip(got, (qc.QC_FULL, qc.QC_CACHED), (500, 480)):
        ctx.denoise(xd, t, ld, B, mode, eps)
    for b in range(B):
        one = torch.empty_like(xd[:1])
        for eps, mode, t in zip(got, (qc.QC_FULL, qc.QC_CACHED), (500, 480)):
            ctx.denoise(xd[b:b + 1], t, ld[b:b + 1], 1, mode, one)
            assert torch.equal(one, eps[b:b + 1]), (b, mode)
    ctx.close()


@pytest.mark.parametrize("model,B", [(_net(1152, 16, 4608, 32, 32), 2 * 16 + 1),        # halves of 17 and 16 latents
                                     (_net(384, 6, 1536, 64, 64), 5), (_net(384, 6, 1536, 50, 34), 41),
                                     # groups of eight tile rows, the last one of six and of three
                                     (_net(1152, 16, 4608, 50, 34), 41),
                                     # Q | K | V of both halves above 128 MiB: streaming stores, whole tiles and ragged ones
                                     (_net(384, 6, 1536, 32, 32), 115), (_net(384, 12, 1536, 50, 34), 69),
                                     # above 448 MiB, heads that are no whole lines
                                     (_net(1152, 16, 4608, 32, 32), 133), (_net(1152, 16, 4608, 50, 34), 81)])
def test_halves_of_a_large_batch(model, B):
    """More than 4096 rows in two concurrent halves: each latent as it comes out alone, eager and in a replayed graph."""
    import torch
    import paper_2503_02508_amd as qc
    from qc_testlib import make_pair, oracle_calibration
    m = replace(model, depth=2)
    w = I.make_weights(m, 21)
    lat, lab = I.make_latents(B, m, 22), I.make_labels(B, m, 23)
    qp, _, _ = oracle_calibration(m, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    _, ctx = make_pair(m, w, qp, B, 2)
    xd, ld = _cuda(lat), _cuda(lab)
    calls = list(zip((qc.QC_FULL, qc.QC_CACHED), (500, 480)))

    def run(x, l, outs):
        for eps, (mode, t) in zip(outs, calls):
            ctx.denoise(x, t, l, x.shape[0], mode, eps)

    want = [torch.empty_like(xd) for _ in calls]
    for b in range(B):
        one = [torch.empty_like(xd[:1]) for _ in calls]
        run(xd[b:b + 1], ld[b:b + 1], one)
        for k in range(2):
            want[k][b:b + 1] = one[k]
    got = [torch.empty_like(xd) for _ in calls]
    run(xd, ld, got)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(xd, ld, got)
    for _ in range(3):
        for g in got:
            g.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        run(xd, ld, got)
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    ctx.close()


@pytest.mark.parametrize("hw,B,steps,cfg,mask", [
    ((20, 20), 13, 45, 0.0, False),             # two windows of steps, halves of 7 and 6 latents on the caller's and one internal stream
    ((20, 20), 13, 7, 0.0, True),               # a schedule per block and module
    ((36, 28), 17, 5, 0.0, False),              # both halves on internal streams
    ((20, 20), 7, 5, 1.5, False)])              # guidance: the halves meet at every step
def test_halves_of_a_sampling_run(hw, B, steps, cfg, mask):
    """A run whose halves go through a window of steps on their own equals the same steps called one by one, and latents run alone."""
    import torch
    from oracle import sampler
    from qc_testlib import make_pair, oracle_calibration
    m = replace(_net(1152, 16, 1152, *hw), depth=2)
    w = I.make_weights(m, 61)
    lat, lab = I.make_latents(B, m, 62), I.make_labels(B, m, 63)
    qp, _, _ = oracle_calibration(m, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    _, ctx = make_pair(m, w, qp, 2 * B if cfg else B, 3)
    xd, ld = _cuda(lat), _cuda(lab)
    K = _cuda(np.linspace(0.9, 1.1, steps * 4, dtype=np.float32).reshape(steps, 4))
    if mask:
        rng = np.random.default_rng(5)
        sched = (rng.random((steps, 2, 2)) < 0.5).astype(np.uint8)
        sched[0] = 1
        sched[2] = 1
        sched[3] = 0
        ctx.set_cache_mask(sched)
    want = xd.clone()
    for i, (t, at, ap) in enumerate(zip(*sampler.ddim_schedule(steps))):
        ctx.sample_step(want, ld, i, int(t), float(at), float(ap), cfg, K[i])
    for _ in range(3):
        got = xd.clone()
        ctx.sample(got, ld, steps, cfg, K)
        assert torch.equal(got, want)
    for b in (0, B // 2, B // 2 + 1, B - 1):
        one = xd[b:b + 1].clone()
        ctx.sample(one, ld[b:b + 1], steps, cfg, K)
        assert torch.equal(one, want[b:b + 1]), b
    ctx.close()


def test_contexts_share_the_internal_streams():
    """Three contexts of one device in threads and on streams of their own, one captured while the others run, and contexts made after
    all earlier ones were closed: every result as it comes out alone."""
    import threading
    import torch
    import paper_2503_02508_amd as qc
    from qc_testlib import make_pair, oracle_calibration
    m = replace(_net(768, 12, 768, 20, 20), depth=2)            # 1700 rows: two halves
    w, B, n = I.make_weights(m, 51), 17, 3
    lat, lab = I.make_latents(B, m, 52), I.make_labels(B, m, 53)
    qp, _, _ = oracle_calibration(m, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    xd, ld = _cuda(lat), _cuda(lab)

    def make():
        return make_pair(m, w, qp, B, 2)[1]

    ctx = make()
    want = xd.clone()
    ctx.sample(want, ld, 4)
    torch.cuda.synchronize()
    ctx.close()
    for _ in range(2):                                   # the second time the streams are made anew
        ctxs, outs, bad = [make() for _ in range(n)], [[] for _ in range(n)], []

        def run(i):
            try:
                s = torch.cuda.Stream()
                with torch.cuda.stream(s):
                    for k in range(8):
                        x = xd.clone()
                        if i == 0 and k == 4:
                            g = torch.cuda.CUDAGraph()
                            with torch.cuda.graph(g, stream=s, capture_error_mode="thread_local"):
                                ctxs[i].sample(x, ld, 4)
                            x.copy_(xd)
                            g.replay()
                        else:
                            ctxs[i].sample(x, ld, 4)
                        outs[i].append(x)
                    s.synchronize()
            except Exception as e:                       # seen by the main thread
                bad.append(e)

        torch.cuda.synchronize()
        threads = [threading.Thread(target=run, args=(i,)) for i in range(n)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert not bad, bad
        assert all(torch.equal(x, want) for o in outs for x in o) and all(len(o) == 8 for o in outs)
        for c in ctxs:
            c.close()


def test_a_stream_that_is_held_up_holds_up_no_other_context():
    """A call on a stream behind a kernel of half a second, then calls of other contexts on other streams: one of theirs is done long before
    it.  (Not all: a stream that shares its hardware queue, one of four, with one that waits does wait, and in some rounds all do.
    Every round has contexts and streams that lie on other queues.)"""
    import time
    import torch
    from qc_testlib import make_pair, oracle_calibration
    m = replace(_net(768, 12, 768, 20, 20), depth=2)            # 1700 rows: two halves
    w, B = I.make_weights(m, 51), 17
    lat, lab = I.make_latents(B, m, 52), I.make_labels(B, m, 53)
    qp, _, _ = oracle_calibration(m, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    xd, ld = _cuda(lat), _cuda(lab)
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)                              # (the kernel is loaded when it is first used)
    begin.record()
    torch.cuda._sleep(1000000)
    end.record()
    torch.cuda.synchronize()
    cycles = int(1000000 * 500 / begin.elapsed_time(end))
    want, keep, early = None, [], 0
    for _ in range(16):
        ctxs, streams = [make_pair(m, w, qp, B, 2)[1] for _ in range(5)], [torch.cuda.Stream() for _ in range(5)]
        keep.append(torch.cuda.Stream())
        outs, done = [xd.clone() for _ in ctxs], [torch.cuda.Event() for _ in ctxs]
        if want is None:
            want = xd.clone()
            ctxs[0].sample(want, ld, 4)
        torch.cuda.synchronize()
        for i, (ctx, s) in enumerate(zip(ctxs, streams)):
            with torch.cuda.stream(s):
                if i == 0:
                    torch.cuda._sleep(cycles)
                ctx.sample(outs[i], ld, 4)
                done[i].record()
        stop = time.monotonic() + 0.2
        while time.monotonic() < stop and not all(e.query() for e in done[1:]):
            time.sleep(0.005)
        finished = [e.query() for e in done]
        torch.cuda.synchronize()
        early += 0 if finished[0] else sum(finished[1:])
        assert all(torch.equal(x, want) for x in outs)
        for c in ctxs:
            c.close()
        if early:
            break
    assert early >= 1


@pytest.mark.parametrize("model,B", [
    (_net(64, 2, 128, 10, 14), 1),              # 35 tokens: the last group of 16 tokens has 3
    (_net(400, 10, 800, 6, 10), 3),             # groups of 16 tokens span batch elements; features end inside a chunk
    (_net(1152, 16, 1152, 18, 14), 5),
    (_net(2048, 32, 2048, 6, 6), 9),            # widest row; more rows of conditioning than one group
    (_net(96, 3, 192, 24, 24, patch=4), 2),     # 64 features a patch: four groups of output features
    (_net(64, 2, 128, 5, 7, patch=1), 4),       # 4 features a patch
    (_net(32, 2, 64, 130, 128), 8)])            # 32 tokens a workgroup of the embedding, 8 of them in the last
def test_conditioning_embedding_and_final_layer(model, B):
    import torch
    from oracle import dit
    from qc_testlib import assert_close, make_pair, oracle_calibration
    w = I.make_weights(model, 31)
    lat, lab = I.make_latents(B, model, 32), I.make_labels(B, model, 33)
    qp, _, _ = oracle_calibration(model, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    lin, ctx = make_pair(model, w, qp, B, 1)
    eps = torch.empty(lat.shape, device="cuda")
    ctx.denoise(_cuda(lat), 333, _cuda(lab), B, 0, eps)
    want = dit.denoiser(lat.astype(np.float64), np.full(B, 333), lab, model, w, lin, {}, True)
    assert_close(eps.cpu().numpy(), want, "eps")
    ctx.close()


@pytest.mark.parametrize("model,wb,B,cfg", [
    (replace(_net(2048, 32, 2048, 6, 6), depth=2), 8, 4, 1.5),        # widest row, 8 rows of conditioning
    (replace(_net(272, 4, 544, 6, 10), depth=3), 4, 3, 0.0),          # 272 = 2 * 128 + 16: the last load of a weight row is 16 bytes
    (replace(_net(16, 1, 32, 4, 4), depth=9), 8, 5, 0.0),             # one group of 16 features; more codes than threads
    (replace(_net(384, 6, 512, 66, 62), depth=1), 4, 1, 1.5),         # 2046 tokens: two to a workgroup of the embedding
    (replace(_net(1152, 16, 1152, 10, 14), depth=2), 8, 1, 0.0)])
def test_single_steps_equal_a_window_of_steps(model, wb, B, cfg):
    """The conditioning of one step (three launches with several parts each) against that of all steps at once."""
    import torch
    import paper_2503_02508_amd as qc
    from qc_testlib import make_pair, oracle_calibration
    model = replace(model, weight_bits=wb)
    w = I.make_weights(model, 41)
    lat, lab = I.make_latents(B, model, 42), I.make_labels(B, model, 43)
    qp, _, _ = oracle_calibration(model, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    _, ctx = make_pair(model, w, qp, 2 * B if cfg else B, 2)
    K = _cuda(I.make_vc_factors(4, model.latent_c, 44))
    labels = _cuda(lab.astype(np.int32))
    for stream in ("fp32", "bf16"):
        ctx.set_stream_format(stream)
        whole, single = _cuda(lat), _cuda(lat)
        ctx.sample(whole, labels, 4, cfg, K)
        for i, (t, at, ap) in enumerate(zip(*qc.qc_ddim_schedule(4))):
            ctx.sample_step(single, labels, i, t, at, ap, cfg, K[i])
        assert torch.equal(whole, single), stream
        assert float((whole - _cuda(lat)).abs().max()) > 0
    ctx.close()


@pytest.mark.parametrize("model,B,steps,cfg", [
    (replace(_net(48, 4, 112, 10, 14), depth=34), 3, 5, 0.0),         # more blocks than a launch takes; two steps' projections at once
    (replace(_net(32, 2, 64, 64, 64), depth=2), 5, 2, 1.5),           # ten rows of conditioning, samples one at a time
    (replace(_net(64, 4, 128, 4, 4), depth=34), 21, 2, 1.5),          # 42 rows together: the projections of six blocks at a time
    (replace(_net(32, 2, 64, 4, 4), depth=2), 19, 2, 0.0),            # 19 rows, more than eight a block: one block at a time
    (replace(_net(2048, 32, 2048, 4, 4), depth=1), 5, 3, 0.0)])       # widest row
def test_reference_trajectory_of_a_fit_does_not_depend_on_the_batch(model, B, steps, cfg):
    """The un-quantised trajectory beside the quantised one: adaLN projections of several steps at once against one latent's."""
    import torch
    from qc_testlib import make_pair, oracle_calibration
    w = I.make_weights(model, 51)
    lat, lab = I.make_latents(B, model, 52), I.make_labels(B, model, 53).astype(np.int32)
    qp, _, _ = oracle_calibration(model, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    _, ctx = make_pair(model, w, qp, 2 * B if cfg else B, 2)
    ctx.load_weights(w, keep_fp32=True)

    def fit(b0, b1):
        x, ref, K = _cuda(lat[b0:b1]), _cuda(lat[b0:b1]), torch.empty(steps, model.latent_c, device="cuda")
        ctx.vc_fit_sampler(x, ref, _cuda(lab[b0:b1]), steps, cfg, 1e-3, K)
        return ref
    whole = fit(0, B)
    assert float((whole - _cuda(lat)).abs().max()) > 0
    for b in range(B):
        assert torch.equal(whole[b:b + 1], fit(b, b + 1))
    ctx.close()


@pytest.mark.parametrize("hidden,hw,B", [(64, (14, 10), 32), (272, (14, 10), 60), (576, (18, 14), 17), (1008, (14, 10), 61),
                                         (1152, (14, 10), 236), (1280, (50, 34), 3), (1152, (6, 6), 456),
                                         (1152, (6, 6), 73), (768, (6, 6), 73), (1536, (14, 10), 235), (2048, (14, 10), 20)])
def test_layer_norm_codes_of_many_rows(hidden, hw, B):
    """A wavefront a row (1, 2 or 4 rows in turn, batch elements that end between them), which decides most codes in float32,
    against a workgroup a row, which forms every value in float64, each thread the statistics or one for all (wider rows: a workgroup for
    4 rows or for one): means far off, outliers, constant rows, ranges beyond float32's squares, values that are not finite."""
    import torch
    import paper_2503_02508_amd as qc
    from qc_testlib import make_pair, oracle_calibration
    model = _net(hidden, hidden // 16, 64, *hw)
    w = I.make_weights(model, 61)
    T, D = model.tokens, model.hidden
    lat, lab = I.make_latents(1, model, 62), I.make_labels(1, model, 63)
    qp, _, _ = oracle_calibration(model, w, lat=lat, lab=lab, t=np.array([400]))
    _, ctx = make_pair(model, w, qp, B, 1)
    rng = np.random.default_rng(64)
    x = rng.standard_normal((B * T, D)).astype(np.float32)
    kind = np.arange(B * T) % 64
    x[kind == 1] += 300.0
    x[kind == 2] *= 1e-3
    x[kind == 3, 5] *= 1e3
    x[kind == 4] = 0.0
    x[kind == 5] = 1.5
    x[kind == 6] *= 1e25
    x[kind == 7, 0] = np.inf
    x[kind == 8, D - 1] = np.nan
    x[kind == 9, 1] = -3e38
    x[kind == 10] *= 1e-25
    cond = rng.standard_normal((B, D)).astype(np.float32)

    def codes(b0, b1):
        ctx.dit_block(0, qc.QC_FULL, _cuda(x[b0 * T:b1 * T].reshape(b1 - b0, T, D)), _cuda(cond[b0:b1]))
        return ctx.workspace("qact_ln", ((b1 - b0) * T, D), torch.int8).clone()
    whole = codes(0, B)
    assert B * T >= 640 and int(whole.unique().numel()) > 100
    for step in (639 // T, 2400 // -(-D // 256) // T):
        for b0 in range(0, B, max(1, step)):
            b1 = min(B, b0 + max(1, step))
            assert torch.equal(whole[b0 * T:b1 * T], codes(b0, b1))
    ctx.close()


@pytest.mark.parametrize("hidden,B", [(64, 480), (272, 40), (272, 240), (576, 480), (1008, 40), (1152, 240)])
def test_layer_norm_of_many_bfloat16_rows(hidden, B):
    """The same with a bfloat16 stream (launches of 700 to 16800 rows, 1, 2 or 4 to a wavefront, against 630): every module output of a block
    and the noise estimate, for tokens of all sizes, equal ones, and ones that are not finite."""
    import torch
    import paper_2503_02508_amd as qc
    from qc_testlib import make_pair, oracle_calibration
    model = _net(hidden, hidden // 16, 64, 14, 10)
    w = I.make_weights(model, 71)
    lat, lab = I.make_latents(B, model, 72), I.make_labels(B, model, 73).astype(np.int32)
    qp, _, _ = oracle_calibration(model, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    _, ctx = make_pair(model, w, qp, B, 2)
    ctx.set_stream_format("bf16")
    kind = np.arange(B) % 16
    lat[kind == 1] *= 1e4
    lat[kind == 2] = 0.0
    lat[kind == 3] += 300.0
    lat[kind == 4] *= 1e25
    lat[kind == 5, 0, 3, 3] = np.inf
    lat[kind == 6, 1, 0, 9] = np.nan
    lat[kind == 7, 2, 5, 5] = 3e4
    lat[kind == 8] *= 1e-25
    x, y = _cuda(lat), _cuda(lab)

    def run(b0, b1):
        eps = torch.empty_like(x[b0:b1])
        ctx.denoise(x[b0:b1], 500, y[b0:b1], b1 - b0, qc.QC_FULL, eps)
        return eps, *(ctx.cache_tensor(0, m, b1 - b0).clone() for m in (qc.QC_CACHE_ATTN, qc.QC_CACHE_MLP))
    whole = run(0, B)
    fine = torch.from_numpy((kind < 4) | (kind > 6)).cuda()
    assert bool(whole[0][fine].isfinite().all()) and float(whole[0][fine].abs().max()) > 0
    for b0 in range(0, B, 18):
        b1 = min(B, b0 + 18)
        for name, a, b in zip(("eps", "attention", "mlp"), whole, run(b0, b1)):
            assert torch.allclose(a[b0:b1], b, rtol=0, atol=0, equal_nan=True), (name, b0)
    ctx.close()
