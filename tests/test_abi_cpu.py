"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every symbol the header declares, and rejects bad arguments before touching a
device."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from oracle import sampler as OS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def qc():
    import paper_2503_02508_amd as m
    return m


def _declared():
    names = set()
    inc = os.path.join(ROOT, "include")
    for h in sorted(os.listdir(inc)):
        if h.endswith(".h"):
            text = open(os.path.join(inc, h)).read()
            text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
            names |= set(re.findall(r"\b(qc_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol(qc):
    names = _declared()
    assert len(names) >= 27 and "qc_sample_step" in names and "qc_w8a8_linear" in names and "qc_tap_cluster" in names
    for n in names:
        assert hasattr(qc.lib, n), n


def _desc(qc, **kw):
    d = dict(depth=2, hidden=64, heads=4, mlp_dim=128, patch=2, latent_c=4, latent_h=8, latent_w=8, num_classes=10,
             freq_dim=256, weight_bits=8, cache_interval=2)
    d.update(kw)
    return qc.ModelDesc(**d)


def test_arena_bytes_and_bad_descriptions(qc):
    n = C.c_size_t()
    assert qc.lib.qc_arena_bytes(C.byref(_desc(qc)), 4, C.byref(n)) == 0 and n.value > 0
    small = n.value
    assert qc.lib.qc_arena_bytes(C.byref(_desc(qc)), 8, C.byref(n)) == 0 and n.value > small
    for kw, code in [(dict(hidden=62), -2), (dict(hidden=72), -7), (dict(depth=0), -2), (dict(latent_h=7), -2), (dict(weight_bits=3), -7),
                     (dict(cache_interval=0), -4), (dict(hidden=4096, heads=64), -7), (dict(heads=1, hidden=128), -7),
                     (dict(freq_dim=255), -2)]:
        assert qc.lib.qc_arena_bytes(C.byref(_desc(qc, **kw)), 4, C.byref(n)) == code, kw
        assert qc.last_error()
    assert qc.lib.qc_arena_bytes(C.byref(_desc(qc)), 0, C.byref(n)) == -2
    assert qc.lib.qc_arena_bytes(None, 4, C.byref(n)) == -1
    assert qc.lib.qc_arena_bytes(C.byref(_desc(qc)), 4, None) == -1


def test_arena_of_large_batches_of_small_latents(qc):
    """What a block adds to the arena grows with the batch by its two cached outputs; the un-quantised forward's projections do not grow with both."""
    def size(depth, batch):
        n = C.c_size_t()
        assert qc.lib.qc_arena_bytes(C.byref(_desc(qc, depth=depth, latent_h=4, latent_w=4, patch=2)), batch, C.byref(n)) == 0
        return n.value
    D = _desc(qc).hidden
    grown = (size(28, 256) - size(20, 256)) - (size(28, 8) - size(20, 8))
    assert grown <= 8 * 2 * (256 - 8) * 4 * D * 4 + 64 * 256, grown              # 4 tokens a sample; 256-byte steps


def test_create_rejects_bad_arenas_without_a_device(qc):
    h = C.c_void_p()
    d = _desc(qc)
    assert qc.lib.qc_create(C.byref(d), None, 1 << 30, 4, C.byref(h)) == -1
    assert qc.lib.qc_create(C.byref(d), C.c_void_p(0x1000 + 8), 1 << 30, 4, C.byref(h)) == -3
    assert qc.lib.qc_create(C.byref(d), C.c_void_p(0x1000), 1024, 4, C.byref(h)) == -6
    assert "needed" in qc.last_error()
    assert qc.lib.qc_create(C.byref(d), C.c_void_p(0x1000), 1 << 30, 4, None) == -1
    assert qc.lib.qc_destroy(None) == -1


def test_context_state_checks_without_a_device(qc):
    """A context over a fake (never dereferenced) arena: every call must fail on its checks."""
    d = _desc(qc)
    n = C.c_size_t()
    qc.lib.qc_arena_bytes(C.byref(d), 2, C.byref(n))
    h = C.c_void_p()
    assert qc.lib.qc_create(C.byref(d), C.c_void_p(0x100000), n.value, 2, C.byref(h)) == 0
    fake = C.c_void_p(0x200000)
    assert qc.lib.qc_set_act_qparams(h, 5, 0, 1.0, 0) == -4
    assert qc.lib.qc_set_act_qparams(h, 0, 7, 1.0, 0) == -4
    assert qc.lib.qc_set_act_qparams(h, 0, 0, 0.0, 0) == -4
    assert qc.lib.qc_set_act_qparams(h, 0, 0, 1.0, 300) == -4
    s, z = C.c_float(), C.c_int()
    assert qc.lib.qc_get_act_qparams(h, 0, 0, C.byref(s), C.byref(z)) == -5
    # weights not loaded / parameters not set -> state error before any launch
    assert qc.lib.qc_dit_block(h, 0, 0, fake, fake, 1, None) == -5
    assert qc.lib.qc_dit_block(h, 0, 0, fake, fake, 3, None) == -2          # batch above max_batch
    assert qc.lib.qc_denoise(h, fake, 10, fake, 1, 1, 0, fake, None) == -5
    assert qc.lib.qc_sample_step(h, fake, fake, 1, 0, 10, 0.5, 0.6, 0.0, None, -1, None) == -5
    assert qc.lib.qc_sample_step(h, fake, fake, 1, 0, 10, 0.0, 0.6, 0.0, None, -1, None) == -4
    assert qc.lib.qc_sample_step(h, fake, fake, 1, -1, 10, 0.5, 0.6, 0.0, None, -1, None) == -4
    assert qc.lib.qc_sample_step(h, fake, fake, 1, 0, 10, 0.5, 0.6, 0.0, None, 3, None) == -4
    assert qc.lib.qc_cache_store(h, 0, 2, fake, 1, None) == -4
    assert qc.lib.qc_cache_store(h, 9, 0, fake, 1, None) == -4
    assert qc.lib.qc_cache_reuse(h, 0, 0, fake, fake, 64, 1, None) == -5        # nothing stored
    assert qc.lib.qc_cache_reuse(h, 0, 0, fake, fake, 10, 1, None) == -2
    # cache schedule: host array [steps][depth][2]; row 0 must be all ones, entries 0/1
    L = d.depth
    ok = (C.c_ubyte * (3 * L * 2))(*([1] * (L * 2) + [0, 1] * L + [0] * (L * 2)))
    assert qc.lib.qc_set_cache_mask(h, ok, 3) == 0
    assert qc.lib.qc_sample_step(h, fake, fake, 1, 3, 10, 0.5, 0.6, 0.0, None, -1, None) == -4     # step beyond the schedule
    bad0 = (C.c_ubyte * (L * 2))(*([1] * (L * 2 - 1) + [0]))
    assert qc.lib.qc_set_cache_mask(h, bad0, 1) == -4
    bad2 = (C.c_ubyte * (2 * L * 2))(*([1] * (L * 2) + [2] * (L * 2)))
    assert qc.lib.qc_set_cache_mask(h, bad2, 2) == -4
    assert qc.lib.qc_set_cache_mask(h, ok, 0) == -2
    assert qc.lib.qc_set_cache_mask(None, ok, 3) == -1
    assert qc.lib.qc_set_cache_mask(h, None, 0) == 0                                               # back to the interval rule
    # the fitting entry points check the weight table and the context state first
    assert qc.lib.qc_denoise_f32(h, None, fake, 10, fake, 1, 1, fake, None) != 0
    assert qc.lib.qc_vc_fit_sampler(h, None, fake, C.c_void_p(0x300000), fake, 1, 4, 0.0, 1e-3, fake, None) != 0
    assert qc.lib.qc_denoise_f32(None, None, fake, 10, fake, 1, 1, fake, None) == -1
    assert qc.lib.qc_vc_fit_sampler(None, None, fake, fake, fake, 1, 4, 0.0, 1e-3, fake, None) == -1
    p = C.c_void_p()
    assert qc.lib.qc_cache_ptr(h, 1, 1, C.byref(p)) == 0 and p.value >= 0x100000
    assert qc.lib.qc_workspace_ptr(h, 99, C.byref(p), None) == -4
    # cache storage format: unknown formats refused, a switch leaves the context usable
    assert qc.lib.qc_set_cache_format(None, 0) == -1
    assert qc.lib.qc_set_cache_format(h, 2) == -4 and qc.lib.qc_set_cache_format(h, -1) == -4
    assert qc.lib.qc_set_cache_format(h, 1) == 0 and qc.lib.qc_set_cache_format(h, 0) == 0
    assert qc.lib.qc_destroy(h) == 0


def test_single_op_argument_checks_without_a_device(qc):
    f = C.c_void_p(0x1000)
    assert qc.lib.qc_quantize_act(None, f, 4, 1.0, 0, None) == -1
    assert qc.lib.qc_quantize_act(C.c_void_p(0x1004), f, 4, 1.0, 0, None) == -3
    assert qc.lib.qc_quantize_act(f, f, 4, -1.0, 0, None) == -4
    assert qc.lib.qc_quantize_act(f, f, 0, 1.0, 0, None) == 0                   # empty input: nothing to do
    assert qc.lib.qc_w8a8_linear(f, f, f, f, None, 1.0, 0, 4, 4, 24, 8, f, None, None) == -2
    assert qc.lib.qc_w8a8_linear(f, f, f, f, None, 1.0, 0, 0, 4, 32, 8, f, None, None) == 0   # M = 0
    assert qc.lib.qc_w8a8_linear(f, f, f, f, None, 1.0, 0, -1, 4, 32, 8, f, None, None) == -2
    assert qc.lib.qc_w8a8_linear(f, C.c_void_p(0x1001), f, f, None, 1.0, 0, 4, 4, 32, 8, f, None, None) == -3
    assert qc.lib.qc_quantize_weight(f, 4, 20, 8, f, f, f, None) == -2
    assert qc.lib.qc_quantize_weight(f, 4, 32, 2, f, f, f, None) == -7
    assert qc.lib.qc_vc_correct(None, f, None, 1, 4, 8, 8, None) == -1
    assert qc.lib.qc_vc_correct(f, f, None, 0, 4, 8, 8, None) == 0
    assert qc.lib.qc_vc_correct(f, f, None, 1, 0, 8, 8, None) == -2
    assert qc.lib.qc_vc_fit(None, f, 1, 4, 8, 8, 1e-3, f, f, None) == -1
    assert qc.lib.qc_vc_fit(f, f, 1, 4, 8, 8, 1e-3, None, f, None) == -1
    assert qc.lib.qc_vc_fit(f, f, 0, 4, 8, 8, 1e-3, f, f, None) == -2
    assert qc.lib.qc_vc_fit(f, f, 1, 4, 8, 8, -1.0, f, f, None) == -4
    assert qc.lib.qc_vc_fit(f, f, 1, 4, 8, 8, float("nan"), f, f, None) == -4
    assert qc.lib.qc_vc_fit(f, f, 1, 4, 8, 8, 1e-3, C.c_void_p(0x1004), f, None) == -3


def test_clustering_argument_checks_without_a_device(qc):
    f, n = C.c_void_p(0x1000), C.c_size_t()
    L = qc.lib
    assert L.qc_tap_workspace_bytes(1024, 64, 128, 8, 16, C.byref(n)) == 0 and n.value > 1024 * 128 * 4
    small = n.value
    assert L.qc_tap_workspace_bytes(2048, 64, 128, 8, 16, C.byref(n)) == 0 and n.value > small
    assert L.qc_tap_workspace_bytes(1024, 64, 128, 8, 16, None) == -1
    for args, code in [((0, 64, 128, 8, 16), -2), ((1024, 64, 128, 8, 12), -7), ((1024, 64, 128, 8, 136), -7),
                       ((1024, 64, 128, 24, 16), -2), ((1024, 64, 8, 8, 16), -2), ((100, 64, 128, 8, 16), -2),
                       ((1 << 20, 4096, 128, 8, 16), -7)]:
        assert L.qc_tap_workspace_bytes(*args, C.byref(n)) == code, args
        assert qc.last_error()
    big = C.c_size_t(1 << 40)
    assert L.qc_tap_similarity(None, f, 64, 8, f, 16, 0.5, f, f, f, f, big, None) == -1
    assert L.qc_tap_similarity(f, f, 64, 8, f, 16, 1.5, f, f, f, f, big, None) == -4
    assert L.qc_tap_similarity(f, f, 64, 8, f, 16, float("nan"), f, f, f, f, big, None) == -4
    assert L.qc_tap_similarity(f, f, 64, 8, f, 65, 0.5, f, f, f, f, big, None) == -2
    assert L.qc_tap_similarity(C.c_void_p(0x1004), f, 64, 8, f, 16, 0.5, f, f, f, f, big, None) == -3
    assert L.qc_tap_similarity(f, f, 64, 8, f, 16, 0.5, f, f, f, f, C.c_size_t(16), None) == -6
    assert L.qc_tap_similarity(f, f, 64, 8, f, 16, 0.5, f, f, f, None, big, None) == -1
    assert L.qc_tap_normalise(None, f, f, 64, 16, f, big, None) == -1
    assert L.qc_tap_normalise(f, f, f, 0, 16, f, big, None) == -2
    assert L.qc_tap_embed(f, 64, 16, 4, 8, 5, f, f, None, f, big, None) == -1
    assert L.qc_tap_embed(f, 64, 16, 4, 12, 5, f, f, f, f, big, None) == -7
    assert L.qc_tap_embed(f, 64, 16, 9, 8, 5, f, f, f, f, big, None) == -2
    assert L.qc_tap_embed(f, 64, 16, 4, 8, -1, f, f, f, f, big, None) == -4
    assert L.qc_tap_embed(f, 64, 16, 4, 8, 5, f, f, f, f, C.c_size_t(64), None) == -6
    assert L.qc_tap_kmeans(f, 64, 200, 4, f, 10, f, f, None, f, big, None) == -7
    assert L.qc_tap_kmeans(f, 64, 8, 4, f, 0, f, f, None, f, big, None) == -4
    assert L.qc_tap_kmeans(f, 64, 8, 4, None, 10, f, f, None, f, big, None) == -1
    assert L.qc_tap_aggregate(f, 9, 64, 4, f, None, f, big, None) == -7
    assert L.qc_tap_aggregate(f, 0, 64, 4, f, None, f, big, None) == -2
    assert L.qc_tap_aggregate(None, 3, 64, 4, f, None, f, big, None) == -1
    assert L.qc_tap_cluster(f, f, 64, 8, f, 3, 16, 0.5, 4, 8, 5, f, f, 10, f, None, f, big, None) == -1
    assert L.qc_tap_cluster(f, f, 64, 8, f, 9, 16, 0.5, 4, 8, 5, f, f, 10, f, f, f, big, None) == -7
    assert L.qc_tap_cluster(f, f, 64, 8, f, 3, 16, 0.5, 4, 8, 5, f, f, 10, f, f, f, C.c_size_t(1000), None) == -6
    ms, cnt = C.c_float(), C.c_int()
    assert L.qc_tap_profile_end(C.byref(ms), C.byref(cnt)) == -5           # no _begin
    assert L.qc_tap_profile_end(None, C.byref(cnt)) == -1
    assert L.qc_tap_profile_begin() == 0
    assert L.qc_tap_profile_end(C.byref(ms), C.byref(cnt)) == 0 and cnt.value == 0 and ms.value == 0.0


@pytest.mark.parametrize("steps", [50, 100, 250, 7, 1])
def test_ddim_schedule_matches_oracle(qc, steps):
    t, a, b = qc.qc_ddim_schedule(steps)
    tt, at, ap = OS.ddim_schedule(steps)
    assert t == list(tt)
    assert np.allclose(a, at, rtol=1e-13) and np.allclose(b, ap, rtol=1e-13)
    with pytest.raises(qc.QCError):
        qc.qc_ddim_schedule(0)
