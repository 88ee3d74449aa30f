"""CPU-only checks of the HIP library's host side: exported symbols, host helpers, argument validation.

No kernel is launched here: every call below either is a host helper or is rejected by validation before
any HIP call.
"""
import ctypes as C
import math
import os
import re

import numpy as np
import pytest

from paper_2101_01321_amd import binding as B, synth
import oracle
from oracle import params as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RNG = np.random.default_rng(7)


def _declared_symbols():
    names = set()
    for header in ("ibert.h", "ibert_testing.h"):
        text = open(os.path.join(ROOT, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(ibert_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    L = B.lib()
    names = _declared_symbols()
    assert len(names) >= 18
    for n in names:
        assert hasattr(L, n), n
        assert n in B.SIGNATURES, "binding lacks a signature for " + n
    assert L.ibert_version() >= 100
    assert B.lib().ibert_status_string(0) == b"ok"
    assert b"precondition" in B.lib().ibert_status_string(-3)


def test_struct_sizes_match_the_header_layout():
    # natural alignment, no packing pragmas: sizes follow from the field lists in include/ibert.h
    assert C.sizeof(B.Dyadic) == 8
    assert C.sizeof(B.GemmDesc) == 5 * 4 + 4 + 12 * 8 + 2 * 4 + 8 + 2 * 4 + 8
    assert C.sizeof(B.SoftmaxParams) == 20
    assert C.sizeof(B.GeluParams) == 24
    assert C.sizeof(B.LayerWeights) == 20 * 8
    assert C.sizeof(B.LayerQuant) == 8 + 20 + 8 + 8 + 4 + 24 + 8 + 4 + 4
    assert C.sizeof(B.WorkspaceLayout) == 10 * 8


def test_dyadic_helper_agrees_with_the_oracle_derivation():
    vals = [1.0, 0.5, -0.75, 2.0 ** -31, 2.0 ** -40, 0.0, math.nextafter(1.0, 0.0), 1234.5678, -3e-7]
    vals += list(np.exp(RNG.uniform(math.log(1e-9), math.log(1e3), size=2000)) * RNG.choice([-1, 1], size=2000))
    for M in vals:
        d = B.ibert_dyadic_from_double(float(M))
        assert d.tuple() == P.dyadic_from_double(float(M)), M
    with pytest.raises(B.IbertError):
        B.ibert_dyadic_from_double(2.0 ** 31)
    with pytest.raises(B.IbertError):
        B.ibert_dyadic_from_double(float("nan"))


def test_softmax_gelu_layernorm_helpers_agree_with_the_oracle_derivation():
    scales = [2.0 ** -e for e in range(3, 11)] + list(np.exp(RNG.uniform(math.log(2e-3), math.log(0.2), size=300)))
    for S in scales:
        want = P.softmax_params(float(S))
        if oracle.lib().orc_softmax_check(want, 128) == 0:
            got = B.ibert_softmax_params_from_scale(float(S), 128)
            assert (got.q_ln2, got.q_b, got.q_c, got.out_frac_bits, got.out_dtype) == \
                   (want.q_ln2, want.q_b, want.q_c, want.out_frac_bits, want.out_dtype)
        else:
            with pytest.raises(B.IbertError):
                B.ibert_softmax_params_from_scale(float(S), 128)
        S_out = float(np.exp(RNG.uniform(math.log(0.01), math.log(1.0))))
        w = P.gelu_params(float(S), S_out)
        g = B.ibert_gelu_params_from_scale(float(S), S_out)
        assert (g.q_b, g.q_c, g.q_1, g.q_max, g.out.m, g.out.s) == (w.q_b, w.q_c, w.q_1, w.q_max, w.out_m, w.out_s)
        hw = P.hgelu_params(float(S), S_out)
        hg = B.ibert_hgelu_params_from_scale(float(S), S_out)
        assert (hg.slope.m, hg.slope.s, hg.q_3, hg.q_6, hg.q_max, hg.out.m, hg.out.s) == \
               (hw.slope_m, hw.slope_s, hw.q_3, hw.q_6, hw.q_max, hw.out_m, hw.out_s)
    for C_ in (1, 7, 256, 768, 1024):
        gamma = RNG.normal(1.0, 0.1, size=C_)
        beta = RNG.normal(0.0, 0.1, size=C_)
        for S_out in (5.0 / 127, 0.013, 0.4):
            gq, bq, s = B.ibert_layernorm_params_from_float(gamma, beta, S_out)
            wq, wb, ws = P.layernorm_params(gamma, beta, S_out)
            assert s == ws and np.array_equal(gq, wq) and np.array_equal(bq, wb)
            assert np.abs(gq).max() < 2 ** 14 and np.abs(bq).max() < 2 ** 29


@pytest.mark.parametrize("name", ["tiny", "base_b1", "large_b32", "base512_b64"])
def test_layer_constants_agree_with_the_oracle_derivation(name):
    cfg = synth.CONFIGS[name]
    sc = synth.static_scales(cfg, 0.0371)
    q = B.ibert_layer_quant_from_scales(sc, cfg.seq, cfg.hidden // cfg.heads)
    raw = {k: v for k, v in synth.layer_raw(synth.EncoderConfig("t", cfg.hidden, cfg.heads, 64, 8, 1, 1), 0).items()}
    raw_small = dict(raw)
    w, oq = P.layer_params(raw_small, sc, cfg.hidden, cfg.heads)
    assert q.scores_dy.tuple() == (oq.scores_m, oq.scores_s)
    assert q.ctx_dy.tuple() == (oq.ctx_m, oq.ctx_s)
    assert q.res1_dy.tuple() == (oq.res1_m, oq.res1_s)
    assert q.res2_dy.tuple() == (oq.res2_m, oq.res2_s)
    assert (q.softmax.q_ln2, q.softmax.q_b, q.softmax.q_c, q.softmax.out_frac_bits) == \
           (oq.softmax.q_ln2, oq.softmax.q_b, oq.softmax.q_c, oq.softmax.out_frac_bits)
    assert (q.gelu.q_b, q.gelu.q_c, q.gelu.q_1, q.gelu.q_max, q.gelu.out.m, q.gelu.out.s) == \
           (oq.gelu.q_b, oq.gelu.q_c, oq.gelu.q_1, oq.gelu.q_max, oq.gelu.out_m, oq.gelu.out_s)
    m, s = B.ibert_channel_dyadics_from_scales(sc["S_h1"], raw["sw_1"], sc["S_g_in"])
    assert np.array_equal(m, w["m_1"]) and np.array_equal(s, w["s_1"])


def test_workspace_layout_is_aligned_and_disjoint():
    lo = B.ibert_encoder_layer_workspace_layout(32, 128, 768, 12, 3072)
    T, H, F, BH, L = 4096, 768, 3072, 384, 128
    sizes = {"qkv": T * 3 * H, "scores": BH * L * L * 4, "probs": BH * L * L, "ctx": T * H, "r1": T * H * 4,
             "h1": T * H, "f1": T * F * 4, "g": T * F, "r2": T * H * 4}
    spans = sorted((getattr(lo, k), getattr(lo, k) + v) for k, v in sizes.items())
    for (a0, a1), (b0, _) in zip(spans, spans[1:]):
        assert a1 <= b0
    assert all(a % 256 == 0 for a, _ in spans) and spans[-1][1] <= lo.total
    assert B.ibert_encoder_layer_workspace_bytes(32, 128, 768, 12, 3072) == lo.total
    assert B.ibert_encoder_workspace_bytes(32, 128, 768, 12, 3072) >= lo.total + 2 * T * H
    assert B.ibert_encoder_layer_workspace_bytes(1, 128, 768, 5, 3072) == 0     # heads must divide hidden


def test_entry_points_reject_bad_arguments_before_touching_the_gpu():
    L = B.lib()
    sp = B.ibert_softmax_params_from_scale(2.0 ** -6, 128)
    gp = B.ibert_gelu_params_from_scale(2.0 ** -7, 0.05)
    dummy = 256  # a non-NULL fake address: validation must fail before it is ever dereferenced
    # NULL / shape
    assert L.ibert_softmax_i(None, None, 4, 128, 128, 128, None, None) == -1
    assert L.ibert_softmax_i(dummy, dummy, -1, 128, 128, 128, C.byref(sp), None) == -2
    assert L.ibert_softmax_i(dummy, dummy, 4, 128, 64, 128, C.byref(sp), None) == -2
    assert L.ibert_softmax_i(None, dummy, 4, 128, 128, 128, C.byref(sp), None) == -1
    assert L.ibert_softmax_i(None, None, 0, 128, 128, 128, C.byref(sp), None) == 0      # empty: no-op
    bad = B.SoftmaxParams(44, 86, 3930, 9, B.I8)
    assert L.ibert_softmax_i(dummy, dummy, 4, 128, 128, 128, C.byref(bad), None) == -3
    bad = B.SoftmaxParams(100, 86, 3930, 7, B.I8)                                       # q_ln2 > q_b
    assert L.ibert_softmax_i(dummy, dummy, 4, 128, 128, 128, C.byref(bad), None) == -3
    bad = B.SoftmaxParams(2839, 5541, 16099000, 7, B.I8)                                # row sum could pass 2^31
    assert L.ibert_softmax_i(dummy, dummy, 4, 128, 128, 128, C.byref(bad), None) == -3
    assert L.ibert_gelu_i(dummy, dummy, -5, C.byref(gp), None) == -2
    assert L.ibert_gelu_i(None, None, 0, C.byref(gp), None) == 0
    bad = B.GeluParams(-161, -28366, -28366, 10 ** 6, B.Dyadic(-5, 3))                  # |t| could pass 2^31
    assert L.ibert_gelu_i(dummy, dummy, 5, C.byref(bad), None) == -3
    bad = B.GeluParams(-161, -28366, -28366, 100, B.Dyadic(-5, 63))
    assert L.ibert_gelu_i(dummy, dummy, 5, C.byref(bad), None) == -3
    assert L.ibert_layernorm_i(dummy, dummy, 4, 2048, 2048, 2048, dummy, dummy, 18, None) == -3
    assert L.ibert_layernorm_i(dummy, dummy, 4, 768, 768, 768, dummy, dummy, 0, None) == -3
    assert L.ibert_layernorm_i(dummy, dummy, 4, 768, 768, 768, None, dummy, 18, None) == -1
    assert L.ibert_layernorm_i(None, None, 0, 768, 768, 768, None, None, 18, None) == 0
    assert L.ibert_layernorm_i16(dummy, dummy, 4, 2048, 2048, 2048, dummy, dummy, 18, None) == -3
    assert L.ibert_layernorm_i16(dummy, dummy, 4, 768, 700, 768, dummy, dummy, 18, None) == -2
    assert L.ibert_layernorm_i16(dummy, dummy, 4, 768, 768, 768, None, dummy, 18, None) == -1
    assert L.ibert_layernorm_i16(None, None, 0, 768, 768, 768, None, None, 18, None) == 0
    d = B.GemmDesc()
    d.M, d.N, d.K, d.batch_outer, d.batch_inner = 4, 4, 4, 1, 1
    d.lda = d.ldw = d.ldc = 4
    d.per_channel, d.requant, d.out_dtype, d.out_clamp = 0, B.Dyadic(1, 0), B.I8, 127
    assert L.ibert_gemm_i8_requant(C.byref(d), None, dummy, None, None, None, None, dummy, None) == -1
    d.out_clamp = 128
    assert L.ibert_gemm_i8_requant(C.byref(d), dummy, dummy, None, None, None, None, dummy, None) == -3
    d.out_dtype, d.out_clamp = B.I16, 32768                      # a 16-bit output cannot hold a wider clamp
    assert L.ibert_gemm_i8_requant(C.byref(d), dummy, dummy, None, None, None, None, dummy, None) == -3
    d.out_dtype = 3                                              # no such type
    assert L.ibert_gemm_i8_requant(C.byref(d), dummy, dummy, None, None, None, None, dummy, None) == -3
    d.out_dtype = B.I8
    d.out_clamp, d.requant = 127, B.Dyadic(1, 63)
    assert L.ibert_gemm_i8_requant(C.byref(d), dummy, dummy, None, None, None, None, dummy, None) == -3
    d.requant, d.lda = B.Dyadic(1, 0), 3
    assert L.ibert_gemm_i8_requant(C.byref(d), dummy, dummy, None, None, None, None, dummy, None) == -2
    d.lda, d.per_channel = 4, 1
    assert L.ibert_gemm_i8_requant(C.byref(d), dummy, dummy, None, None, None, None, dummy, None) == -1
    d.M = 0
    assert L.ibert_gemm_i8_requant(C.byref(d), None, None, None, None, None, None, None, None) == 0
    # layer: workspace too small / NULL
    w, q = B.LayerWeights(), B.LayerQuant()
    assert L.ibert_encoder_layer_i(C.byref(w), C.byref(q), dummy, 512, 1, 128, 256, 4, 1024, dummy * 1, 16, None) == -5
    assert L.ibert_encoder_layer_i(None, C.byref(q), dummy, 512, 1, 128, 256, 4, 1024, dummy, 1 << 30, None) == -1
    assert L.ibert_encoder_layer_i(C.byref(w), C.byref(q), dummy, 512, 1, 128, 256, 4, 1024, 256, 1 << 30, None) == -1


def test_fused_entry_points_reject_bad_arguments_before_touching_the_gpu():
    L = B.lib()
    sp = B.ibert_softmax_params_from_scale(2.0 ** -6, 128)
    gp = B.ibert_gelu_params_from_scale(2.0 ** -7, 0.05)
    dy = B.Dyadic(1518500250, 36)
    dummy = 256
    att = lambda qkv, ctx, b, l, h, nh, s_dy, smp, c_dy, scr, nbytes: L.ibert_attention_i(qkv, ctx, b, l, h, nh, s_dy, smp, c_dy, scr, nbytes, None)
    assert att(dummy, dummy, 1, 128, 768, 12, None, C.byref(sp), C.byref(dy), None, 0) == -1
    assert att(dummy, dummy, 1, 128, 768, 5, C.byref(dy), C.byref(sp), C.byref(dy), None, 0) == -2          # heads must divide hidden
    assert att(dummy, dummy, -1, 128, 768, 12, C.byref(dy), C.byref(sp), C.byref(dy), None, 0) == -2
    assert att(dummy, dummy, 1, 128, 768, 12, C.byref(B.Dyadic(1, 63)), C.byref(sp), C.byref(dy), None, 0) == -3
    sp32 = B.ibert_softmax_params_from_scale(2.0 ** -6, 128, 24, B.I32)
    assert att(dummy, dummy, 1, 128, 768, 12, C.byref(dy), C.byref(sp32), C.byref(dy), None, 0) == -3       # probabilities must be INT8
    assert att(None, None, 0, 128, 768, 12, C.byref(dy), C.byref(sp), C.byref(dy), None, 0) == 0            # empty batch
    assert att(None, dummy, 1, 128, 768, 12, C.byref(dy), C.byref(sp), C.byref(dy), None, 0) == -1
    # a length the one-kernel form does not cover needs the scratch buffer, big enough and 256-byte aligned
    need = L.ibert_attention_scratch_bytes(1, 72, 12)
    assert need >= 5 * 12 * 72 * 72 and need % 256 == 0
    sp72 = B.ibert_softmax_params_from_scale(2.0 ** -6, 72)
    assert att(dummy, dummy, 1, 72, 768, 12, C.byref(dy), C.byref(sp72), C.byref(dy), None, 0) == -5
    assert att(dummy, dummy, 1, 72, 768, 12, C.byref(dy), C.byref(sp72), C.byref(dy), 512, need - 1) == -5
    assert att(dummy, dummy, 1, 72, 768, 12, C.byref(dy), C.byref(sp72), C.byref(dy), 512 + 16, need) == -5
    # MatMul + GELU
    d = B.GemmDesc()
    d.M, d.N, d.K, d.batch_outer, d.batch_inner = 4, 4, 4, 1, 1
    d.lda = d.ldw = d.ldc = 4
    d.per_channel, d.requant, d.out_dtype = 0, B.Dyadic(1, 0), B.I8
    gg = lambda desc, A, W, gelu, Cc, scr: L.ibert_gemm_i8_gelu(desc, A, W, None, None, None, gelu, Cc, scr, None)
    assert gg(None, dummy, dummy, C.byref(gp), dummy, None) == -1
    assert gg(C.byref(d), dummy, dummy, None, dummy, None) == -1
    assert gg(C.byref(d), None, dummy, C.byref(gp), dummy, None) == -1
    bad = B.GeluParams(-161, -28366, -28366, 10 ** 6, B.Dyadic(-5, 3))
    assert gg(C.byref(d), dummy, dummy, C.byref(bad), dummy, None) == -3
    d.lda = 3
    assert gg(C.byref(d), dummy, dummy, C.byref(gp), dummy, None) == -2
    d.lda, d.M = 4, 0
    assert gg(C.byref(d), None, None, C.byref(gp), None, None) == 0                                        # empty problem
    # the integer square root
    assert L.ibert_isqrt_i(dummy, dummy, -1, 0, None) == -2 and L.ibert_isqrt_i(dummy, dummy, 8, 4, None) == -3
    assert L.ibert_isqrt_i(dummy, dummy, 8, -1, None) == -3 and L.ibert_isqrt_i(None, dummy, 8, 0, None) == -1
    assert L.ibert_isqrt_i(None, None, 0, 1, None) == 0
    # a layer's route flags start at zero (every fusion) when the quantization constants come from the helper
    assert B.ibert_layer_quant_from_scales(synth.static_scales(synth.CONFIGS["tiny"], 0.03), 128, 64).route == 0


def _matmul_desc(M, N, K, **kw):
    d = B.GemmDesc()
    d.M, d.N, d.K, d.batch_outer, d.batch_inner = M, N, K, 1, 1
    d.lda, d.ldw, d.ldc, d.ldr = K, K, N, N
    d.per_channel, d.out_dtype, d.out_clamp = 1, B.I8, 127
    for k, v in kw.items():
        setattr(d, k, v)
    return d


def _needs_no_gpu():
    import torch
    if torch.cuda.is_available():
        pytest.skip("made-up pointers: only where nothing can be launched")


@pytest.mark.parametrize("cfg", [23, 24, 25, 26, 27, 28, 29, 30])
def test_a_hip_error_of_the_chosen_matmul_kernel_reaches_the_caller(cfg):
    # (without a device every HIP call fails: the error to come back is that of the kernel the configuration names, not the
    # one of another kernel tried in its place)
    _needs_no_gpu()
    L = B.lib()
    d = _matmul_desc(256, 768, 256)
    L.ibert_gemm_config_override(cfg)
    try:
        assert L.ibert_gemm_i8_requant(C.byref(d), 4096, 4096, 4096, 4096, 4096, None, 4096, None) == -6
    finally:
        L.ibert_gemm_config_override(-1)
    assert b"MaxDynamicSharedMemorySize, 163840)" in L.ibert_last_hip_error(), L.ibert_last_hip_error()


@pytest.mark.parametrize("M,N,K,asks", [
    (130, 128, 256, True), (128, 1024, 256, True), (4095, 3072, 384, True),        # a short K and few whole tiles
    (2741, 3072, 768, True), (15311, 3072, 768, True),                             # many tiles, the last row of them cut
    (4096, 768, 2048, True), (2048, 1024, 2048, True),                             # a long K and one tile for every unit
    (4096, 3072, 768, False), (2048, 3072, 128, False), (4096, 768, 1920, False), (4096, 1536, 2048, False),
    (2048, 1024, 1920, False), (128, 3072, 768, False), (200, 72, 512, False), (1, 16, 512, False),
    (4096, 3072, 784, True), (128, 768, 528, True)])                               # K no multiple of 128
def test_matmul_gelu_asks_for_scratch_and_dense_outputs_by_the_documented_rule(M, N, K, asks):
    # what is refused without them does not depend on which problems a later kernel has come to serve in one launch
    _needs_no_gpu()
    gp = B.ibert_gelu_params_from_scale(2.0 ** -7, 8.0 / 127)
    call = lambda d, scr: B.lib().ibert_gemm_i8_gelu(C.byref(d), 4096, 4096, 4096, 4096, 4096, C.byref(gp), 4096, scr, None)
    assert call(_matmul_desc(M, N, K), None) == (-5 if asks else -6)               # -6: no device to launch it on
    assert call(_matmul_desc(M, N, K, ldc=N + 16), 4096) == (-7 if asks else -6)
    assert call(_matmul_desc(M, N, K, ldc=N + 16), None) == (-7 if asks else -6)
    assert call(_matmul_desc(M, N, K), 4096) == -6


def test_embedding_and_masked_entry_points_reject_bad_arguments_before_touching_the_gpu():
    L = B.lib()
    dy = B.Dyadic(1518500250, 36)
    dummy = 256
    emb = lambda ids, tok, pos, T, seq, H, V, mp, tdy, pdy, g, b, sh, y, ldy: L.ibert_embedding_i(
        ids, tok, pos, T, seq, H, V, mp, tdy, pdy, g, b, sh, y, ldy, None)
    ok = (dummy, dummy, dummy, 10, 4, 64, 100, 8, C.byref(dy), C.byref(dy), dummy, dummy, 12, dummy, 64)
    def but(**kw):
        names = ("ids", "tok", "pos", "T", "seq", "H", "V", "mp", "tdy", "pdy", "g", "b", "sh", "y", "ldy")
        a = dict(zip(names, ok))
        a.update(kw)
        return emb(*[a[n] for n in names])
    assert but(tdy=None) == -1 and but(pdy=None) == -1
    assert but(T=-1) == -2 and but(seq=0) == -2 and but(V=0) == -2 and but(mp=3) == -2 and but(ldy=63) == -2
    assert but(tdy=C.byref(B.Dyadic(1, 63))) == -3 and but(H=1025, ldy=1025) == -3 and but(sh=0) == -3 and but(sh=31) == -3
    assert but(T=0, ids=None, y=None) == 0                                     # no tokens: nothing to do
    assert but(ids=None) == -1 and but(tok=None) == -1 and but(y=None) == -1 and but(g=None) == -1
    # h-GELU
    hp = B.ibert_hgelu_params_from_scale(2.0 ** -6, 0.05)
    assert L.ibert_hgelu_i(dummy, dummy, 8, None, None) == -1 and L.ibert_hgelu_i(dummy, dummy, -1, C.byref(hp), None) == -2
    assert L.ibert_hgelu_i(None, None, 0, C.byref(hp), None) == 0 and L.ibert_hgelu_i(None, dummy, 8, C.byref(hp), None) == -1
    for field, val in (("q_max", 2 ** 31 - 1), ("q_3", -1), ("q_6", 5)):
        bad = B.ibert_hgelu_params_from_scale(2.0 ** -6, 0.05)
        setattr(bad, field, val)
        assert L.ibert_hgelu_i(dummy, dummy, 8, C.byref(bad), None) == -3
    # masked Softmax
    sp = B.ibert_softmax_params_from_scale(2.0 ** -6, 128)
    sm = lambda x, y, rows, cols, ldx, ldy, p, kl, rpl: L.ibert_softmax_masked_i(x, y, rows, cols, ldx, ldy, p, kl, rpl, None)
    assert sm(dummy, dummy, 4, 128, 128, 128, None, dummy, 2) == -1
    assert sm(dummy, dummy, 4, 128, 128, 128, C.byref(sp), dummy, 0) == -2
    assert sm(dummy, dummy, 4, 128, 100, 128, C.byref(sp), dummy, 2) == -2
    assert sm(dummy, dummy, 4, 128, 128, 128, C.byref(sp), None, 2) == -1
    assert sm(None, None, 0, 128, 128, 128, C.byref(sp), None, 2) == 0
    # the masked layer validates like the plain one (the lengths live on the device and are not looked at)
    assert L.ibert_encoder_layer_masked_i(None, None, dummy, dummy, 1, 128, 768, 12, 3072, dummy, dummy, 1 << 30, None) == -1
    assert L.ibert_encoder_masked_i(None, None, 1, dummy, dummy, 1, 128, 768, 12, 3072, dummy, dummy, 1 << 30, None) == -1
    assert L.ibert_attention_masked_i(dummy, dummy, 1, 128, 768, 5, C.byref(dy), C.byref(sp), C.byref(dy), dummy, None, 0, None) == -2


def _isqrt_inputs():
    k = np.arange(1, 65536, dtype=np.uint64)
    n = np.unique(np.concatenate([k * k - 1, k * k, k * k + 1, np.array([0, 1, 2, 3, 17413928, 2 ** 32 - 1], np.uint64),
                                  np.random.default_rng(4).integers(0, 2 ** 32, size=1_000_000, dtype=np.uint64)]))
    return n[n < 2 ** 32]


def _check_floor_sqrt(n, x):
    assert np.all(x * x <= n) and np.all((x + 1) * (x + 1) > n)            # the defining property, on all of them
    assert np.array_equal(x[::97], np.array([math.isqrt(int(v)) for v in n[::97]], np.uint64))


@pytest.mark.parametrize("lanes,shifts", [(64, (10, 4, 0)), (32, (11, 6, 1, 0)), (16, (12, 8, 4, 0))])
def test_lane_parallel_square_root_recipe_is_exact(lanes, shifts):
    # the LayerNorm kernel's square root: in each round the lanes of a row test r + (lane + 1) << s, those whose square
    # does not exceed n are counted, r grows by count << s.  Replayed here with 32-bit wrap-around products, as on the
    # device, on every n next to a perfect square and on 10^6 random n.
    n = _isqrt_inputs()
    r = np.zeros_like(n)
    for s in shifts:
        cnt = np.zeros_like(n)
        for lane in range(lanes):
            c = r + (np.uint64(lane + 1) << np.uint64(s))
            ok = (c <= 65535) & (((c * c) & np.uint64(0xffffffff)) <= n)
            cnt += ok.astype(np.uint64)
        r = r + (cnt << np.uint64(s))
    _check_floor_sqrt(n, r)


def test_shift_and_subtract_square_root_recipe_is_exact():
    # the per-lane form: sixteen steps of an add, a compare and a conditional subtract
    n0 = _isqrt_inputs()
    n, res = n0.copy(), np.zeros_like(n0)
    bit = np.uint64(1 << 30)
    while bit:
        t = res + bit
        ge = n >= t
        n = np.where(ge, n - t, n)
        res = np.where(ge, (res >> np.uint64(1)) + bit, res >> np.uint64(1))
        bit >>= np.uint64(2)
    _check_floor_sqrt(n0, res)


# ------------------------------------------------------------------------------------------- weights read ahead
def _weight_plan(M, N, K, kind, gelu=None):
    d = B.GemmDesc()
    for k, v in dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=1,
                     out_dtype=B.I16 if kind == "i16res" else B.I8, out_clamp=127).items():
        setattr(d, k, v)
    plan, readers, ahead = (C.c_int32 * 3)(), np.zeros(N, np.uint8), np.zeros((8, N * K // 1024), np.uint8)
    if gelu is None:
        rc = B.lib().ibert_gemm_weight_plan(C.byref(d), kind == "gelu", plan, readers.ctypes.data, ahead.ctypes.data)
    else:
        rc = B.lib().ibert_gemm_gelu_weight_plan(C.byref(d), C.byref(gelu), plan, readers.ctypes.data, ahead.ctypes.data)
    assert rc == 0, (M, N, K, kind, rc)                       # (a read past the end of W is an error)
    return list(plan), readers, ahead


def _check_weight_plan(M, N, K, kind, gelu=None):
    (config, rows, xs), readers, ahead = _weight_plan(M, N, K, kind, gelu)
    case = (M, N, K, kind, config, rows, xs)
    assert readers.all() and N % rows == 0, case
    assert ahead.max() == 1 and ahead.any(axis=0).all(), case            # all of W, nothing twice by one XCD
    by_kb = np.bitwise_or.reduce(ahead << np.arange(8, dtype=np.uint8)[:, None], axis=0)
    if xs < 2:
        assert (ahead.sum(axis=0) == 1).all(), case                      # once, by any XCD
        return config
    # every XCD that multiplies a row has read each KB of it ahead, and no more XCDs than share it
    assert (ahead.sum(axis=0) == 8 >> xs).all(), case
    at = np.arange(N * K // 1024, dtype=np.int64) * 1024
    for row in (at // K, (at + 1023) // K):
        assert not (readers[row] & ~by_kb).any(), case
    return config


@pytest.mark.parametrize("H,F", [(128, 640), (256, 1024), (384, 640), (512, 2048), (768, 3072), (1024, 4096), (1024, 1152)])
def test_weights_read_ahead_are_those_the_kernels_read(H, F):
    # the plan an encoder makes before the attention against the dealing of tiles of the kernels themselves, and what the attention reads
    # by it, over token counts from one to the largest
    seen = set()
    for M in [1, 2, 16, 17, 61, 128, 129, 300, 488, 777, 1000, 1024, 2048, 2741, 4096, 4100, 8192, 15311, 16384, 32768]:
        for N, K, kind in ((3 * H, H, "i8"), (H, H, "i16res"), (F, H, "gelu"), (H, F, "i16res")):
            seen.add(_check_weight_plan(M, N, K, kind))
    assert len(seen) > 4, seen


# (the same parameters as in the test of the table's room on the device: what is planned is what is launched)
@pytest.mark.parametrize("bn,S,S_out,fits", [(256, 2.0 ** -6, 0.7, 1), (256, 2.0 ** -6, 3.2685, 1), (256, 2.0 ** -6, 3.2688, 0),
                                             (192, 2.0 ** -6, 2.5, 1), (192, 2.0 ** -5, 10.9846, 1), (192, 2.0 ** -5, 10.9848, 0),
                                             (256, 2.0 ** -9, 0.06, 0), (192, 2.0 ** -9, 0.06, 0)])                   # no table at all
def test_weights_read_ahead_follow_the_gelu_table(bn, S, S_out, fits):
    # a table that finds no room beside the persistent tiles sends the MatMul to another tile, which shares its weights in another way
    gp = B.ibert_gelu_params_from_scale(S, S_out)
    config = _check_weight_plan(256 * 90 - 7, 4 * bn, 128, "gelu", gp)
    assert (config in (23, 24)) == bool(fits), config


@pytest.mark.parametrize("N,K,kind,read", [(32768, 1024, "gelu", 1), (32768 + 128, 1024, "gelu", 0), (1024, 32768, "i16res", 1),
                                           (1024, 32768 + 128, "i16res", 0), (1024, 131072, "i16res", 0)])
def test_weights_read_ahead_are_bounded(N, K, kind, read):
    # matrices of up to 32 MB are read ahead, larger ones are not
    for M in (1, 128, 4096):
        _, _, ahead = _weight_plan(M, N, K, kind)
        assert ahead.any(axis=0).all() if read else not ahead.any(), (M, N, K)


def test_weights_read_ahead_for_every_tile():
    # the same for tiles that the choice takes rarely, forced
    try:
        for config, bn in [(25, 16), (26, 32), (27, 32), (28, 64), (29, 96), (30, 64), (15, 32), (3, 64), (17, 96), (18, 96), (19, 128), (21, 96),
                           (22, 128), (7, 128), (9, 96), (13, 192), (14, 128), (23, 256), (24, 192)]:
            B.lib().ibert_gemm_config_override(config)
            for M in [1, 100, 256, 512, 1025, 4096, 9000]:
                for tiles in (1, 2, 4, 7, 8, 12, 16):
                    if tiles * bn * 256 % 1024 == 0:
                        assert _check_weight_plan(M, tiles * bn, 256, "i8") == config
    finally:
        B.lib().ibert_gemm_config_override(-1)


@pytest.mark.parametrize("M,N,K,config", [
    (5248, 3968, 2304, 14), (7114, 3968, 2048, 14), (20736, 1408, 2944, 14), (6431, 1664, 384, 14), (2264, 3968, 256, 14),     # 256x128
    (588, 2880, 128, 9), (4009, 768, 128, 9), (10591, 192, 128, 9), (1060, 2592, 256, 9), (3603, 1152, 256, 9),              # 128x96
    (2048, 3072, 128, 9), (2048, 3072, 256, 9), (801, 3712, 128, 7), (896, 2432, 128, 7),                                    # 128x128
    (3072, 3072, 128, 13), (12288, 768, 128, 13), (6144, 1536, 128, 13),                                                     # 256x192
    (488, 3072, 768, 21), (1024, 4096, 1024, 22), (1274, 1024, 1664, 22), (2048, 1024, 1280, 22)])                           # with loaders
def test_gelu_tile_chosen_is_the_fastest_measured(M, N, K, config):
    # problems at which the configuration named was the fastest of all on the device, most by 4 to 17 % before the next
    assert _weight_plan(M, N, K, "gelu")[0][0] == config


# ------------------------------------------------------------------------------------------- QKV projection and attention as one kernel
def _qkv_plan(batch, seq, heads):
    H = 64 * heads
    tile, places, readers, ahead = C.c_int32(), np.zeros((batch, heads), np.uint8), np.zeros((3, heads), np.uint8), np.zeros((8, 3 * H * H // 1024), np.uint8)
    rc = B.lib().ibert_qkv_attention_plan(batch, seq, heads, C.byref(tile), places.ctypes.data, readers.ctypes.data, ahead.ctypes.data)
    return rc, tile.value, places, readers, ahead


@pytest.mark.parametrize("heads", [2, 4, 6, 10, 12, 14, 16, 24])
def test_qkv_attention_deals_every_head_once_and_reads_its_weights_ahead(heads):
    H, tiles = 64 * heads, set()
    try:
        for forced in (None, 8112, 8222, 8442, 8422, 8414, 16313, 16412):
            for batch in (1, 2, 3, 5, 8, 11, 16, 21, 32, 43, 61, 64, 97, 128, 250):
                for seq in (1, 17, 32, 33, 61, 64, 90, 100, 128, 129, 192, 193, 256):
                    B.lib().ibert_qkv_attention_override(-1 if forced is None else forced)
                    rc, tile, places, readers, ahead = _qkv_plan(batch, seq, heads)
                    case = (batch, seq, heads, tile, rc)
                    if rc == -7:
                        assert forced is None, case
                        continue
                    assert rc == 0, case                                   # (a place or a read outside is an error)
                    tiles.add(tile)
                    assert (places == 1).all() and readers.all(), case
                    assert ahead.max() == 1 and ahead.any(axis=0).all(), case
                    copies = ahead.sum(axis=0)
                    if (copies == 1).all():
                        continue                                           # once, by any XCD
                    by_kb = np.bitwise_or.reduce(ahead << np.arange(8, dtype=np.uint8)[:, None], axis=0)
                    kb_of_head = by_kb.reshape(3, heads, H * 64 // 1024)   # (64 rows of H bytes)
                    assert not (readers[:, :, None] & ~kb_of_head).any(), case
    finally:
        B.lib().ibert_qkv_attention_override(-1)
    assert len(tiles) >= 7, tiles


@pytest.mark.parametrize("batch,seq,heads,tile", [(8, 61, 12, 8214), (32, 128, 12, 8412), (32, 128, 16, 8412), (1, 128, 4, 8414), (1, 128, 12, 0), (3, 59, 12, 0), (8, 128, 12, 0), (256, 128, 16, 0),
                                                  (4, 256, 16, 0), (16, 256, 16, 16412), (16, 150, 12, 16313), (61, 251, 12, 0), (128, 64, 12, 8422), (43, 32, 12, 8222), (128, 32, 12, 8442),
                                                  (512, 40, 16, 0), (1024, 16, 12, 0), (33, 128, 16, 0), (43, 128, 16, 0), (44, 128, 16, 8412), (43, 128, 12, 8412), (33, 64, 16, 8422)])
def test_qkv_attention_is_chosen_where_it_was_the_faster_way(batch, seq, heads, tile):
    rc, got, *_ = _qkv_plan(batch, seq, heads)
    assert (got if rc == 0 else 0) == tile


@pytest.mark.parametrize("kind", ["tall", "fast", "slow", "bias", "mixed"])
def test_qkv_constants_show_a_wrong_requantization(kind):
    # what the GPU tests of the joined kernel feed it: results vary in every channel that is meant to, and each of the mistakes that a requantization may
    # have (rounding left out, half a unit too much, a clamp at -128, no clamp, a wrapped sum) changes some
    import qkv_constants as QC
    heads, B_, L = 4, 2, 128
    cfg, x, _, w, q = QC.layer(heads, B_, L)
    vary = QC.deal(w, cfg.hidden, kind)
    _, inter = oracle.encoder_layer(w, q, x, B_, L, cfg.hidden, heads, cfg.ffn, dump=True)
    qkv = inter["qkv"]
    assert (qkv.min(axis=0) < qkv.max(axis=0))[vary].all()
    acc = x.reshape(B_ * L, -1).astype(np.int64) @ w["w_qkv"].astype(np.int64).T.reshape(cfg.hidden, -1)
    assert np.abs(acc).max() < 1 << 23
    total, m, sh = acc + w["b_qkv"].astype(np.int64), w["m_qkv"].astype(np.int64), w["s_qkv"].astype(np.int64)
    half = np.where(sh > 0, np.int64(1) << np.maximum(sh - 1, 0), 0)

    def requantized(t=total, add=half, lo=-127, hi=127):
        return np.clip((t * m + add) >> sh, lo, hi)
    assert np.array_equal(requantized(), qkv)
    for name, wrong in (("rounding left out", requantized(add=0 * half)), ("one more", requantized(add=half + (np.int64(1) << np.maximum(sh - 8, 0)))), ("clamp", requantized(lo=-128)),
                        ("wrapped byte", requantized(lo=-(1 << 62), hi=1 << 62).astype(np.int8)), ("wrapped sum", requantized(t=((total + (1 << 30)) % (1 << 31)) - (1 << 30)))):
        if name != "wrapped sum" or kind == "bias":
            assert (wrong != qkv).any(), name


# few heads: a layer by itself anywhere; in a forward of several, up to eight sequences only where rows and K steps are few
@pytest.mark.parametrize("batch,seq,heads,tile", [(1, 96, 2, 8314), (1, 97, 2, 0), (8, 128, 2, 0), (9, 128, 2, 8414), (1, 64, 4, 8214), (1, 65, 4, 0), (1, 128, 4, 0), (8, 128, 4, 0), (9, 65, 4, 8314),
                                                  (1, 32, 6, 8114), (1, 33, 6, 0), (8, 64, 6, 0), (9, 33, 6, 8214), (8, 61, 12, 8214), (32, 128, 12, 8412), (1, 128, 12, 0), (1, 257, 2, 0), (8, 200, 2, 0)])
def test_qkv_attention_of_few_heads_in_a_forward_of_several_layers(batch, seq, heads, tile):
    got = C.c_int32()
    for layers in (2, 12):
        assert B.lib().ibert_qkv_attention_chosen(batch, seq, heads, layers, C.byref(got)) == 0
        assert got.value == tile, layers
    assert B.lib().ibert_qkv_attention_chosen(batch, seq, heads, 1, C.byref(got)) == 0
    rc, alone, *_ = _qkv_plan(batch, min(seq, 256), heads)
    assert got.value == (alone if rc == 0 and seq <= 256 else 0)
    assert not (heads <= 6 and seq <= 128) or got.value


# rows to a wavefront: 16 rows make a workgroup of four, 256 of these a round
@pytest.mark.parametrize("C_,rows,want", [(768, 1, 1), (768, 3568, 1), (768, 3569, 4), (768, 4096, 4), (768, 4097, 1), (768, 7152, 1), (768, 7153, 4), (768, 8191, 4), (768, 8192, 0),
                                          (768, 32768, 0), (512, 2544, 1), (512, 2545, 4), (512, 4097, 1), (512, 5104, 1), (512, 5105, 4), (512, 8192, 4), (512, 8193, 4), (512, 32768, 4),
                                          (1024, 4096, 1), (1024, 8192, 1), (1024, 8193, 0), (1024, 10736, 0), (1024, 10737, 4), (1024, 12288, 4), (1024, 12289, 0), (1024, 32768, 4),
                                          (256, 4096, 0), (770, 4096, 0), (640, 4096, 0)])
def test_layernorm_rows_of_a_wavefront(C_, rows, want):
    got = C.c_int32(-1)
    for shift, expect in ((14, want), (8, want), (7, 0)):
        assert B.lib().ibert_layernorm_i16_plan(rows, C_, shift, C.byref(got)) == 0
        assert got.value == expect, shift


# ------------------------------------------------------------------------------------------- buffers that end with the last row
def test_rows_of_the_persistent_tiles_are_checked_whole_against_the_buffers_end(tmp_path):
    # Output and residual are buffers that end with the last row, so that lanes past it neither load nor store.  The range check takes the
    # lane's offset alone: with a part of the row in the scalar offset, lanes past M would pass it.  Looked up in the built code: all that
    # moves between such a buffer and registers has no scalar offset.  (Operands go to LDS, with the K step as the scalar offset:
    # their rows past M fail on the lane's offset.)
    import os
    import re
    import shutil
    import subprocess
    from paper_2101_01321_amd import build
    tool = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(tool):
        pytest.skip("no disassembler")
    so = shutil.copy(build.LIB, tmp_path)
    subprocess.run([tool, "--offloading", so], check=True, capture_output=True, cwd=tmp_path)
    seen = {"buffer_load": 0, "buffer_store": 0}
    for part in sorted(tmp_path.glob("*gfx950")):
        text = subprocess.run([tool, "-d", "--no-show-raw-insn", str(part)], check=True, capture_output=True, text=True).stdout
        for line in re.findall(r"^\s+(buffer_(?:load|store)_dword.*)$", text, re.M):
            if " lds" in line:
                continue
            seen[line[:line.index("_dword")]] += 1
            assert re.match(r"buffer_\w+ v\S+, v\d+, s\[[0-9:]+\], 0 offen", line), line
    assert seen["buffer_load"] >= 8 and seen["buffer_store"] >= 32, seen
