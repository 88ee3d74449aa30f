"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, bit for bit, on the same seeded inputs.

Bar: every integer output equal.  Dequantised outputs vs their float counterparts are covered by the
oracle pins (the GPU equals the oracle exactly, so the same tolerances hold); one end-to-end float check
is repeated here on GPU outputs for the record.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from oracle import params as P, GemmSpec, I8, I32

I16 = 2     # the library's 16-bit MatMul output type (same values as I32)
from paper_2101_01321_amd import synth


@pytest.fixture(scope="module")
def G(gpu):
    import gpu_util
    from paper_2101_01321_amd import binding
    binding.lib()                      # fail loudly if the HIP library is missing
    return gpu_util


def _eq(got, want, what):
    if not np.array_equal(got, want):
        bad = np.argwhere(np.asarray(got) != np.asarray(want))
        first = tuple(bad[0])
        raise AssertionError("%s: %d of %d differ; first at %s: got %s want %s" % (
            what, len(bad), np.asarray(want).size, first, np.asarray(got)[first], np.asarray(want)[first]))


# ------------------------------------------------------------------------------------------- GELU
@pytest.mark.parametrize("S_in,S_out", [(2.0 ** -7, 8.0 / 127), (2.0 ** -6, 0.406), (2.0 ** -4, 0.1), (0.011, 0.02)])
def test_gelu_matches_oracle(G, S_in, S_out):
    from paper_2101_01321_amd import binding as B
    gp = B.ibert_gelu_params_from_scale(S_in, S_out)
    op = P.gelu_params(S_in, S_out)
    x, _ = synth.gelu_inputs(517, 3072, scale=S_in)
    x = x.reshape(-1)
    x[:8] = [0, 1, -1, 2 ** 31 - 1, -2 ** 31, gp.q_max, -gp.q_max, gp.q_max + 1]
    x[8:4008] = np.arange(-2000, 2000)
    G.say("gelu S_in=%g n=%d" % (S_in, x.size))
    _eq(G.gelu(x, gp), oracle.gelu(x, op), "gelu")
    for n, xo, yo in [(0, 0, 0), (1, 0, 0), (3, 0, 0), (4, 0, 0), (4097, 0, 0), (5000, 1, 0), (5000, 0, 3), (16385, 3, 1)]:
        G.say("gelu ragged n=%d x_off=%d y_off=%d" % (n, xo, yo))
        if n == 0:
            assert G.gelu(x[:0], gp).size == 0
        else:
            _eq(G.gelu(x[:n], gp, x_off=xo, y_off=yo), oracle.gelu(x[:n], op), "gelu n=%d" % n)


@pytest.mark.parametrize("S_in,S_out", [(2.0 ** -7, 8.0 / 127), (2.0 ** -6, 0.406), (2.0 ** -4, 0.1), (0.011, 0.02),
                                        (2.0 ** -13, 0.05), (0.9, 0.3)])
def test_hgelu_matches_oracle(G, S_in, S_out):
    # Eq. 6 in integers; scales of 2^-4 and above leave the 24-bit forms (q_max reaches 2^23), 2^-13 has a large q_6
    from paper_2101_01321_amd import binding as B
    hp, op = B.ibert_hgelu_params_from_scale(S_in, S_out), P.hgelu_params(S_in, S_out)
    x, _ = synth.gelu_inputs(517, 3072, scale=S_in)
    x = x.reshape(-1)
    x[:8] = [0, 1, -1, 2 ** 31 - 1, -2 ** 31, hp.q_max, -hp.q_max, hp.q_max + 1]
    x[8:4008] = np.arange(-2000, 2000)
    want = oracle.hgelu(x, op)
    assert len(np.unique(want)) > 3
    G.say("h-GELU S_in=%g n=%d" % (S_in, x.size))
    _eq(G.hgelu(x, hp), want, "h-GELU")
    for n, xo, yo in [(1, 0, 0), (3, 0, 0), (4097, 0, 0), (5000, 1, 0), (5000, 0, 3), (16385, 3, 1)]:
        G.say("h-GELU ragged n=%d x_off=%d y_off=%d" % (n, xo, yo))
        _eq(G.hgelu(x[:n], hp, x_off=xo, y_off=yo), want[:n], "h-GELU n=%d" % n)
    # hand-made constants outside what the helper produces: negative slope, shifts at the ends of the range
    for slope, out in (((-1827387392, 30), (1518500250, 40)), ((1827387392, 0), (1518500250, 62)), ((3, 1), (5, 2)),
                       ((1827387392, 31), (1518500250, 33)), ((1827387392, 32), (-1518500250, 36))):
        hp2, op2 = B.ibert_hgelu_params_from_scale(S_in, S_out), P.hgelu_params(S_in, S_out)
        hp2.slope.m, hp2.slope.s, hp2.out.m, hp2.out.s = slope[0], slope[1], out[0], out[1]
        op2.slope_m, op2.slope_s, op2.out_m, op2.out_s = slope[0], slope[1], out[0], out[1]
        if slope[1] == 0:
            hp2.q_max = op2.q_max = min(hp2.q_max, 1)        # slope 2^30.8: keep DY(q; slope) inside 64 bits either way
        G.say("h-GELU constants slope=%s out=%s" % (slope, out))
        _eq(G.hgelu(x[:20000], hp2), oracle.hgelu(x[:20000], op2), "h-GELU slope=%s out=%s" % (slope, out))


def test_hgelu_full_shape(G):
    from paper_2101_01321_amd import binding as B
    x, S = synth.gelu_inputs(4096, 3072)                     # the FFN activation of Base, batch 32
    hp, op = B.ibert_hgelu_params_from_scale(S, 8.0 / 127), P.hgelu_params(S, 8.0 / 127)
    G.say("h-GELU full [4096,3072]")
    _eq(G.hgelu(x, hp), oracle.hgelu(x, op).reshape(-1), "h-GELU full")


def test_gelu_full_shape(G):
    from paper_2101_01321_amd import binding as B
    x, S = synth.gelu_inputs(4096, 3072)                     # configs[1]: N(0,2) at scale 2^-7
    gp, op = B.ibert_gelu_params_from_scale(S, 8.0 / 127), P.gelu_params(S, 8.0 / 127)
    G.say("gelu full [4096,3072]")
    _eq(G.gelu(x, gp), oracle.gelu(x, op).reshape(-1), "gelu full")


# ------------------------------------------------------------------------------------------- Softmax
@pytest.mark.parametrize("cols", [1, 2, 3, 5, 63, 64, 65, 100, 127, 128, 129, 200, 256, 300, 511, 512, 513, 1000,
                                  1024, 1500, 2048, 2500])
def test_softmax_matches_oracle_over_widths(G, cols):
    from paper_2101_01321_amd import binding as B
    rows = 67
    x, S = synth.softmax_logits(rows, cols)
    x[0, :] = 5                                              # all equal
    x[1, :] = -2 ** 31
    x[1, cols // 2] = 2 ** 31 - 1                            # extreme spread
    x[2, :] = -2 ** 31                                       # all at the minimum
    if oracle.lib().orc_softmax_check(P.softmax_params(S), cols) != 0:
        S = 2.0 ** -4
    sp, op = B.ibert_softmax_params_from_scale(S, cols), P.softmax_params(S)
    G.say("softmax cols=%d" % cols)
    _eq(G.softmax(x, sp), oracle.softmax(x, op), "softmax cols=%d" % cols)
    if cols in (5, 127, 300, 513, 2500):
        G.say("softmax cols=%d unaligned rows" % cols)
        got = G.softmax(x, sp, ldx=cols + 3, ldy=cols + 1, x_off=1, y_off=3)
        _eq(got[:, :cols], oracle.softmax(x, op), "softmax unaligned cols=%d" % cols)
        assert np.all(got[:, cols:] == 77)                  # padding untouched


@pytest.mark.parametrize("S", [2.0 ** -4, 2.0 ** -5, 2.0 ** -7, 0.0123, 2.0 ** -8])
def test_softmax_other_scales_and_spreads(G, S):
    from paper_2101_01321_amd import binding as B
    cols = 128
    sp, op = B.ibert_softmax_params_from_scale(S, cols), P.softmax_params(S)
    for std in (0.5, 4.0, 40.0, 4000.0):
        x, _ = synth.softmax_logits(513, cols, std=std, scale=S)
        G.say("softmax S=%g std=%g" % (S, std))
        _eq(G.softmax(x, sp), oracle.softmax(x, op), "softmax S=%g std=%g" % (S, std))
    sp32, op32 = B.ibert_softmax_params_from_scale(S, cols, 24, B.I32), P.softmax_params(S, 24, I32)
    x, _ = synth.softmax_logits(200, cols, scale=S)
    G.say("softmax i32 out S=%g" % S)
    _eq(G.softmax(x, sp32), oracle.softmax(x, op32), "softmax i32")


def test_softmax_full_shape(G):
    from paper_2101_01321_amd import binding as B
    x, S = synth.softmax_logits(32 * 12 * 128, 128)         # configs[1]
    sp, op = B.ibert_softmax_params_from_scale(S, 128), P.softmax_params(S)
    G.say("softmax full [49152,128]")
    _eq(G.softmax(x, sp), oracle.softmax(x, op), "softmax full")
    x, S = synth.softmax_logits(3 * 512, 512)
    sp = B.ibert_softmax_params_from_scale(S, 512)
    G.say("softmax [1536,512]")
    _eq(G.softmax(x, sp), oracle.softmax(x, op), "softmax 512")


# ------------------------------------------------------------------------------------------- LayerNorm
@pytest.mark.parametrize("C", [1, 3, 100, 255, 256, 257, 512, 640, 768, 1000, 1024])
@pytest.mark.parametrize("rows", [5, 2051])
def test_layernorm_matches_oracle(G, C, rows):
    from paper_2101_01321_amd import binding as B
    x, S, gamma, beta = synth.layernorm_inputs(rows, C)
    x[0, :] = 123                                            # constant row: sigma clamps to 1
    x[1, :] = 32767 * (-1) ** np.arange(C)
    x[2, :] = 0
    x[2, 0] = 2 ** 31 - 1                                    # clamped on load
    x[3, :] = -2 ** 31
    gq, bq, s = B.ibert_layernorm_params_from_float(gamma, beta, 5.0 / 127)
    G.say("layernorm C=%d rows=%d" % (C, rows))
    _eq(G.layernorm(x, gq, bq, s), oracle.layernorm(x, gq, bq, s), "layernorm C=%d rows=%d" % (C, rows))
    # the same rows stored as int16 (clamped first: that is all 16 bits can hold, and what the kernel's own clamp makes of them)
    xc = np.clip(x, -32767, 32767)
    G.say("layernorm int16 C=%d rows=%d" % (C, rows))
    _eq(G.layernorm(xc, gq, bq, s, half=True), oracle.layernorm(x, gq, bq, s), "layernorm int16 C=%d rows=%d" % (C, rows))
    if C in (3, 257, 1000):
        G.say("layernorm int16 C=%d rows=%d unaligned" % (C, rows))
        got = G.layernorm(xc, gq, bq, s, ldx=C + 1, ldy=C + 3, x_off=3, y_off=1, half=True)
        _eq(got[:, :C], oracle.layernorm(x, gq, bq, s), "layernorm int16 unaligned")
        assert np.all(got[:, C:] == 77)
    if C in (3, 257, 1000):
        G.say("layernorm C=%d rows=%d unaligned" % (C, rows))
        got = G.layernorm(x, gq, bq, s, ldx=C + 1, ldy=C + 3, x_off=3, y_off=1)
        _eq(got[:, :C], oracle.layernorm(x, gq, bq, s), "layernorm unaligned")
        assert np.all(got[:, C:] == 77)


@pytest.mark.parametrize("C", [512, 768, 1024])
@pytest.mark.parametrize("rows", [6, 7, 129, 2544, 2545, 3568, 3569, 4095, 4096, 4097, 4111, 8191, 8192, 8193, 10736, 10737, 12288, 12289])
def test_layernorm_many_int16_rows(G, C, rows):
    # one row and four to a wavefront: both sides of the switch, rows that leave a group or a workgroup unfilled, the least shift it takes and the one before, and what
    # 16 bits hold that the clamp does not
    from paper_2101_01321_amd import binding as B
    x, S, gamma, beta = synth.layernorm_inputs(rows, C, seed=rows + C)
    x[::5] *= 40
    x = np.clip(x, -32767, 32767)
    x[0], x[1], x[2], x[-1] = 123, 0, -32768, -32768
    x[3] = np.where(np.arange(C) % 2, 32767, -32768)
    x[4] = np.where(np.arange(C) == C - 1, 1, 0)
    x[-2] = 32767
    gq, bq, s = B.ibert_layernorm_params_from_float(gamma, beta, 5.0 / 127)
    for shift in (s, 8, 7):
        G.say("layernorm int16 [%d,%d] shift %d" % (rows, C, shift))
        got = G.layernorm(x, gq, bq, shift, ldx=C + 8, ldy=C + 16, half=True)
        _eq(got[:, :C], oracle.layernorm(x, gq, bq, shift), "layernorm int16 [%d,%d] shift %d" % (rows, C, shift))
        assert np.all(got[:, C:] == 77)
        if shift == s:
            # (rounds of 256 workgroups of 16 rows: three from 8193 rows on, 7/8 of them filled from 10737 on; four from 12289 on)
            many = C == 512 or rows < 8192 or (C == 1024 and rows in (8192, 10737, 12288))
            want = b"layernorm_many_kernel" if many else b"layernorm_rows_kernel"
            assert B.lib().ibert_last_kernel() == want


def test_layernorm_full_shape_and_small_sigma(G):
    from paper_2101_01321_amd import binding as B
    x, S, gamma, beta = synth.layernorm_inputs(4096, 768)   # configs[1]
    gq, bq, s = B.ibert_layernorm_params_from_float(gamma, beta, 5.0 / 127)
    G.say("layernorm full [4096,768]")
    _eq(G.layernorm(x, gq, bq, s), oracle.layernorm(x, gq, bq, s), "layernorm full")
    _eq(G.layernorm(np.clip(x, -32767, 32767), gq, bq, s, half=True), oracle.layernorm(x, gq, bq, s), "layernorm full, int16 rows")
    # int16 rows, many of them: the wide-chunk form of the kernel (whole rows, and rows that end inside a lane's reach)
    for rows, C in ((8200, 768), (8197, 1024), (9000, 512), (8300, 256), (8200, 640), (8192, 1000), (8200, 8)):
        x, S, gamma, beta = synth.layernorm_inputs(rows, C, seed=rows + C)
        x[::5] *= 40                                                     # rows that saturate the 16-bit clamp
        xc = np.clip(x, -32767, 32767)
        gq2, bq2, s2 = B.ibert_layernorm_params_from_float(gamma, beta, 5.0 / 127)
        G.say("layernorm int16 [%d,%d]" % (rows, C))
        _eq(G.layernorm(xc, gq2, bq2, s2, half=True), oracle.layernorm(x, gq2, bq2, s2), "layernorm int16 [%d,%d]" % (rows, C))
        G.say("layernorm int16 [%d,%d], padded rows" % (rows, C))
        got = G.layernorm(xc, gq2, bq2, s2, ldx=C + 8, ldy=C + 16, half=True)
        _eq(got[:, :C], oracle.layernorm(x, gq2, bq2, s2), "layernorm int16 padded [%d,%d]" % (rows, C))
        assert np.all(got[:, C:] == 77)
    rng = np.random.default_rng(5)
    x = rng.integers(-3, 4, size=(3000, 768)).astype(np.int32)       # tiny variances: sqrt of small numbers
    x[::7] *= 9000
    G.say("layernorm small/large sigma")
    _eq(G.layernorm(x, gq, bq, s), oracle.layernorm(x, gq, bq, s), "layernorm sigma sweep")


@pytest.mark.parametrize("method", [0, 1, 2, 3])
def test_isqrt_matches_oracle(G, method):
    # Alg. 4's result on the device, by both routines the LayerNorm kernels use: every perfect square and its two
    # neighbours, powers of two and their neighbours, the ends of the range, the paper's six-pass example, random values
    k = np.arange(65536, dtype=np.uint64)
    sq = k * k
    p2 = np.uint64(1) << np.arange(33, dtype=np.uint64)
    n = np.concatenate([sq, sq + 1, np.maximum(sq, 1) - 1, p2, p2 + 1, p2 - 1, [0, 1, 2, 3, 17413928, 2 ** 32 - 1, 2 ** 32 - 2],
                        np.random.default_rng(4).integers(0, 2 ** 32, size=1_000_000, dtype=np.uint64)])
    n = n[n < 2 ** 32].astype(np.uint32)
    want, _ = oracle.isqrt_array(n)
    G.say("isqrt method %d on %d values" % (method, n.size))
    _eq(G.isqrt(n, method), np.asarray(want, np.uint32), "isqrt method %d" % method)


# ------------------------------------------------------------------------------------------- GEMM
def _gemm_case(G, M, N, K, out_dtype, per_channel, bias, residual, seed, clamp=None):
    from paper_2101_01321_amd import binding as B
    A, W, sw, b = synth.gemm_operands(M, N, K, layer=seed)
    mult, shift = B.ibert_channel_dyadics_from_scales(0.03, sw, 0.4 if out_dtype == I8 else 0.002)
    clamp = clamp if clamp is not None else (127 if out_dtype == I8 else 32767)
    R = np.random.default_rng(seed).integers(-127, 128, size=(M, N), dtype=np.int8) if residual else None
    dy = (int(mult[0]), int(shift[0])) if N else (1, 0)
    res_dy = (1717986918, 29)
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=per_channel,
              requant=dy, out_dtype=out_dtype, out_clamp=clamp, residual_dy=res_dy)
    got = G.gemm(kw, A, W, b if bias else None, mult if per_channel else None, shift if per_channel else None, R,
                 out_elems=M * N)
    # (the 16-bit output holds the values of the 32-bit one: the oracle has no type of its own for it)
    spec = GemmSpec(M, N, K, per_channel=per_channel, dy=dy, out_dtype=I32 if out_dtype == I16 else out_dtype,
                    out_clamp=clamp, res_dy=res_dy)
    want = oracle.gemm_requant(spec, A, W, b if bias else None, mult if per_channel else None,
                               shift if per_channel else None, R)
    if out_dtype == I16:
        assert got.dtype == np.int16 and np.abs(want).max() > 300       # not a case that would fit 8 bits
    _eq(got, want, "gemm %dx%dx%d" % (M, N, K))


@pytest.mark.parametrize("M,N,K", [(128, 128, 64), (128, 128, 128), (256, 384, 192), (200, 136, 80), (1, 16, 16),
                                   (77, 50, 48), (130, 250, 1024), (64, 64, 32), (300, 48, 160), (5, 5, 16)])
def test_gemm_mfma_path_matches_oracle(G, M, N, K):
    for out_dtype, pc, bias, res in [(I8, 1, True, False), (I32, 1, True, True), (I32, 0, False, False), (I8, 0, True, True),
                                     (I16, 1, True, True)]:
        G.say("gemm M=%d N=%d K=%d out=%d pc=%d bias=%d res=%d" % (M, N, K, out_dtype, pc, bias, res))
        _gemm_case(G, M, N, K, out_dtype, pc, bias, res, seed=M + N + K)


@pytest.mark.parametrize("M,N,K", [(33, 21, 70), (64, 64, 17), (9, 130, 5), (16, 16, 0)])
def test_gemm_generic_path_matches_oracle(G, M, N, K):
    # K not a multiple of 16 -> row stride unaligned -> the byte-load kernel
    for out_dtype, pc, bias, res in [(I8, 1, True, True), (I32, 0, True, False), (I16, 1, True, True)]:
        G.say("gemm generic M=%d N=%d K=%d out=%d" % (M, N, K, out_dtype))
        _gemm_case(G, M, N, K, out_dtype, pc, bias, res, seed=7 * M + K)


def test_gemm_k_tail_inside_aligned_rows(G):
    # lda/ldw are multiples of 16 but K is not: the MFMA path must zero-fill the tail of the last K step
    from paper_2101_01321_amd import binding as B
    M, N, K, ld = 70, 90, 100, 112
    rng = np.random.default_rng(3)
    A = rng.integers(-127, 128, size=(M, ld), dtype=np.int8)
    W = rng.integers(-127, 128, size=(N, ld), dtype=np.int8)
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=ld, ldw=ld, ldc=N, per_channel=0, requant=(2 ** 30, 30),
              out_dtype=I32, out_clamp=2 ** 31 - 1)
    G.say("gemm K tail")
    got = G.gemm(kw, A, W, out_elems=M * N).reshape(M, N)
    _eq(got, A[:, :K].astype(np.int64) @ W[:, :K].astype(np.int64).T, "gemm K tail")


def test_gemm_attention_shapes(G):
    # scores (batched, strided views of the packed QKV buffer) and context (W given as [K,N]) as the layer issues them
    B_, nh, L, dh = 2, 3, 72, 64
    H = nh * dh
    rng = np.random.default_rng(11)
    qkv = rng.integers(-127, 128, size=(B_ * L, 3 * H), dtype=np.int8)
    dy = (1518500250, 33)
    kw = dict(M=L, N=L, K=dh, batch_outer=B_, batch_inner=nh, lda=3 * H, ldw=3 * H, ldc=L,
              strideA_outer=L * 3 * H, strideA_inner=dh, strideW_outer=L * 3 * H, strideW_inner=dh,
              strideC_outer=nh * L * L, strideC_inner=L * L, per_channel=0, requant=dy, out_dtype=I32,
              out_clamp=2 ** 31 - 1)
    G.say("gemm scores-shaped")
    got = G.gemm(kw, qkv, qkv, out_elems=B_ * nh * L * L, offsets={"W": H})
    spec = GemmSpec(L, L, dh, lda=3 * H, ldw=3 * H, ldc=L, batch_outer=B_, batch_inner=nh, sA=(L * 3 * H, dh),
                    sW=(L * 3 * H, dh), sC=(nh * L * L, L * L), per_channel=0, dy=dy, out_dtype=I32, out_clamp=2 ** 31 - 1)
    flat = qkv.reshape(-1)
    _eq(got, oracle.gemm_requant(spec, flat, flat[H:], out_elems=B_ * nh * L * L), "scores")
    Pm = rng.integers(0, 128, size=(B_ * nh, L, L), dtype=np.int8)
    dy = (1073741824, 37)
    kw = dict(M=L, N=dh, K=L, batch_outer=B_, batch_inner=nh, lda=L, ldw=3 * H, ldc=H, trans_w=1,
              strideA_outer=nh * L * L, strideA_inner=L * L, strideW_outer=L * 3 * H, strideW_inner=dh,
              strideC_outer=L * H, strideC_inner=dh, per_channel=0, requant=dy, out_dtype=I8, out_clamp=127)
    G.say("gemm context-shaped")
    got = G.gemm(kw, Pm, qkv, out_elems=B_ * L * H, offsets={"W": 2 * H})
    spec = GemmSpec(L, dh, L, lda=L, ldw=3 * H, ldc=H, batch_outer=B_, batch_inner=nh, trans_w=1, sA=(nh * L * L, L * L),
                    sW=(L * 3 * H, dh), sC=(L * H, dh), per_channel=0, dy=dy, out_dtype=I8, out_clamp=127)
    _eq(got, oracle.gemm_requant(spec, Pm.reshape(-1), flat[2 * H:], out_elems=B_ * L * H), "context")


def _attention_oracle(qkv, B_, L, H, nh, scores_dy, op, ctx_dy):
    dh = H // nh
    flat = qkv.reshape(-1)
    spec = GemmSpec(L, L, dh, lda=3 * H, ldw=3 * H, ldc=L, batch_outer=B_, batch_inner=nh, sA=(L * 3 * H, dh),
                    sW=(L * 3 * H, dh), sC=(nh * L * L, L * L), per_channel=0, dy=scores_dy, out_dtype=I32, out_clamp=2 ** 31 - 1)
    scores = oracle.gemm_requant(spec, flat, flat[H:], out_elems=B_ * nh * L * L)
    probs = oracle.softmax(scores.reshape(-1, L), op)
    spec = GemmSpec(L, dh, L, lda=L, ldw=3 * H, ldc=H, batch_outer=B_, batch_inner=nh, trans_w=1, sA=(nh * L * L, L * L),
                    sW=(L * 3 * H, dh), sC=(L * H, dh), per_channel=0, dy=ctx_dy, out_dtype=I8, out_clamp=127)
    return oracle.gemm_requant(spec, probs.reshape(-1), flat[2 * H:], out_elems=B_ * L * H).reshape(B_ * L, H)


@pytest.mark.parametrize("B_,nh,L,S,sdy,cdy", [
    (2, 3, 128, 2.0 ** -6, (1518500250, 36), (1073741824, 37)),       # the one-kernel shape, 24-bit Softmax path
    (1, 12, 128, 2.0 ** -6, (1920459399, 38), (1518500250, 36)),
    (2, 2, 128, 2.0 ** -6, (1187698534, 28), (1073741824, 37)),        # a multiplier above one: funnel-shift form
    (1, 3, 128, 2.0 ** -6, (1187698534, 32), (2800, 21)),        # shifts at the edges of the two forms
    (2, 2, 128, 2.0 ** -6, (1187698534, 28), (700000, 25)),             # both shifts below 32, and each side of 32 in turn
    (1, 3, 128, 2.0 ** -6, (1187698534, 32), (1400000, 26)),
    (1, 2, 256, 2.0 ** -6, (1187698534, 31), (1073741824, 37)),
    (1, 2, 128, 2.0 ** -5, (1187698534, 20), (1518500250, 33)),        # below the fast range: general form
    (3, 2, 128, 2.0 ** -2, (1518500250, 41), (1073741824, 37)),       # q_ln2 = 2: the general Softmax path
    (2, 2, 128, 2.0 ** -9, (1518500250, 30), (1073741824, 35)),       # wide logits, context clamps at 127
    (1, 2, 256, 2.0 ** -6, (1518500250, 36), (1073741824, 37)),       # longer rows, still one kernel
    (1, 3, 384, 2.0 ** -6, (1187698534, 28), (1073741824, 37)),
    (2, 2, 512, 2.0 ** -6, (1187698534, 28), (1518500250, 38)),
    (1, 1, 512, 2.0 ** -2, (1518500250, 41), (60000, 22)),       # general Softmax and requantization forms at L = 512
    (2, 3, 72, 2.0 ** -6, (1518500250, 36), (1073741824, 37)),        # other lengths: three kernels through scratch
    (1, 2, 192, 2.0 ** -6, (1518500250, 36), (1073741824, 37)),
])
def test_attention_equals_scores_softmax_context(G, B_, nh, L, S, sdy, cdy):
    from paper_2101_01321_amd import binding as B
    dh, H = 64, nh * 64
    rng = np.random.default_rng(B_ * 100 + nh * 10 + L)
    qkv = np.clip(np.rint(rng.normal(0, 40, size=(B_ * L, 3 * H))), -127, 127).astype(np.int8)
    qkv[0, :] = 127                                          # a saturated query/key/value row
    qkv[1, :H] = 0                                           # a query with all-equal scores
    qkv[L - 1, H:2 * H] = -127
    sp, op = B.ibert_softmax_params_from_scale(S, L), P.softmax_params(S)
    want = _attention_oracle(qkv, B_, L, H, nh, sdy, op, cdy)
    assert len(np.unique(want)) > 10
    G.say("attention B=%d heads=%d L=%d S=%g" % (B_, nh, L, S))
    _eq(G.attention(qkv, B_, L, H, nh, sdy, sp, cdy), want, "attention")
    if L in (128, 256, 384, 512):
        G.say("attention, one-kernel form without scratch")
        _eq(G.attention(qkv, B_, L, H, nh, sdy, sp, cdy, with_scratch=False), want, "attention (no scratch)")
    else:
        with pytest.raises(B.IbertError):
            G.attention(qkv, B_, L, H, nh, sdy, sp, cdy, with_scratch=False)


@pytest.mark.parametrize("M,N,K,ldw", [(128, 64, 128, 192), (100, 64, 64, 64), (130, 128, 96, 256), (64, 20, 48, 36),
                                        (256, 192, 272, 192), (37, 4, 16, 8), (512, 64, 512, 2304)])
def test_gemm_trans_w_mfma_path(G, M, N, K, ldw):
    # W given as [K,N] with aligned rows: the transposing loader of the MFMA kernel
    rng = np.random.default_rng(M * 7 + N)
    nb = 3
    A = rng.integers(0, 128, size=(nb, M, K), dtype=np.int8)
    W = rng.integers(-127, 128, size=(nb, K, ldw), dtype=np.int8)
    for od, dy in ((I8, (1073741824, 37)), (I32, (1518500250, 30))):
        kw = dict(M=M, N=N, K=K, batch_outer=nb, batch_inner=1, lda=K, ldw=ldw, ldc=N, trans_w=1,
                  strideA_outer=M * K, strideW_outer=K * ldw, strideC_outer=M * N, per_channel=0, requant=dy,
                  out_dtype=od, out_clamp=127 if od == I8 else 2 ** 31 - 1)
        G.say("gemm trans_w M=%d N=%d K=%d ldw=%d out=%d" % (M, N, K, ldw, od))
        got = G.gemm(kw, A, W, out_elems=nb * M * N)
        spec = GemmSpec(M, N, K, lda=K, ldw=ldw, ldc=N, batch_outer=nb, batch_inner=1, trans_w=1, sA=(M * K, 0),
                        sW=(K * ldw, 0), sC=(M * N, 0), per_channel=0, dy=dy, out_dtype=od,
                        out_clamp=127 if od == I8 else 2 ** 31 - 1)
        _eq(got, oracle.gemm_requant(spec, A.reshape(-1), W.reshape(-1), out_elems=nb * M * N), "trans_w gemm")


@pytest.mark.parametrize("cfg,M,N,K", [(6, 512, 384, 128), (6, 256, 576, 256), (6, 768, 192, 768), (7, 128, 128, 128),
                                       (7, 384, 256, 384), (7, 256, 640, 1152), (8, 512, 256, 256), (8, 256, 768, 640),
                                       (9, 256, 288, 384), (10, 512, 384, 512),
                                       # three LDS stages: every step count around the ring depth
                                       (11, 128, 96, 128), (11, 256, 96, 256), (11, 128, 192, 384), (11, 128, 96, 512),
                                       (11, 256, 192, 1280), (12, 128, 128, 128), (12, 128, 128, 256), (12, 256, 128, 384),
                                       (12, 128, 256, 512), (12, 128, 256, 1024),
                                       # 256x192 with eight wavefronts
                                       (13, 256, 192, 128), (13, 512, 384, 256), (13, 256, 576, 640), (13, 768, 192, 1152),
                                       (14, 256, 128, 128), (14, 512, 384, 256), (14, 256, 256, 896),
                                       # 256x256 with eight wavefronts
                                       (16, 256, 256, 128), (16, 512, 256, 256), (16, 256, 768, 384), (16, 512, 512, 1024),
                                       # 64x96, three and two LDS stages
                                       (17, 64, 96, 128), (17, 128, 192, 256), (17, 192, 96, 384), (17, 256, 288, 1024),
                                       (18, 64, 96, 128), (18, 128, 192, 256), (18, 64, 96, 512), (18, 128, 96, 640),
                                       # 64x128
                                       (19, 64, 128, 128), (19, 128, 256, 256), (19, 192, 128, 384), (19, 256, 384, 1024),
                                       # 128x96 with eight wavefronts in four rows of two, three stages
                                       (20, 128, 96, 128), (20, 256, 192, 256), (20, 128, 288, 640), (20, 384, 96, 1024),
                                       # ... and with four loader wavefronts beside them
                                       (21, 128, 96, 128), (21, 256, 192, 256), (21, 128, 288, 640), (21, 384, 96, 1024),
                                       (22, 128, 128, 128), (22, 256, 256, 256), (22, 128, 384, 640), (22, 384, 128, 1024)])
def test_gemm_direct_to_lds_tiles(G, cfg, M, N, K):
    # the tile configurations whose loader writes LDS straight from global memory (whole tiles only), forced
    # through the configuration override; 1, 2, odd and even numbers of K steps
    from paper_2101_01321_amd import binding as B
    assert B.lib().ibert_gemm_config_override(cfg) > cfg
    try:
        for out_dtype, pc, bias, res in [(I8, 1, True, False), (I32, 1, True, True), (I8, 0, False, True), (I16, 1, True, True)]:
            G.say("gemm direct-to-LDS cfg=%d M=%d N=%d K=%d out=%d" % (cfg, M, N, K, out_dtype))
            _gemm_case(G, M, N, K, out_dtype, pc, bias, res, seed=cfg + M + N + K)
            # (the persistent kernel takes 8-bit outputs without a residual and 16-bit ones; the ring tile serves the others)
            ring = cfg in (8, 16) and not (out_dtype == I16 or (out_dtype == I8 and not res))
            name = B.lib().ibert_last_kernel().decode()
            assert name.startswith("gemm_nt_mfma_kernel<128, 128, 64, 2, " if ring else G.kernel_of(cfg)), name
    finally:
        B.lib().ibert_gemm_config_override(-1)


@pytest.mark.parametrize("cfg", [20, 21, 22])
@pytest.mark.parametrize("shift,form", [(40, "direct"), (30, "staged")])
@pytest.mark.parametrize("out_dtype,res", [(I8, False), (I8, True), (I16, True), (I32, True), (I32, False)])
def test_gemm_four_rows_of_wavefronts_epilogue_forms(G, cfg, out_dtype, res, shift, form):
    # The 128x96 tile whose eight wavefronts stand in four rows of two (20), the same with four loader wavefronts that end
    # before the epilogue (21), and the 128x128 tile with loaders (22): both epilogue forms -- the register-direct one
    # (shifts of 40) and the staged general one (shifts of 30), whose staging tile is laid out by wavefront row and whose
    # barriers the loaders no longer join -- for every output type, and the kernel's record must name the form.
    from paper_2101_01321_amd import binding as B
    import torch
    M, N, K = 384, 384 if cfg == 22 else 192, 768
    rng = np.random.default_rng(shift + out_dtype)
    A = rng.integers(-127, 128, size=(M, K), dtype=np.int8)
    W = rng.integers(-127, 128, size=(N, K), dtype=np.int8)
    bias = rng.integers(-50000, 50000, size=N, dtype=np.int32)
    mult = rng.integers(2 ** 29, 2 ** 30, size=N, dtype=np.int64).astype(np.int32)
    shifts = np.full(N, shift, np.int32)
    R = rng.integers(-127, 128, size=(M, N), dtype=np.int8) if res else None
    clamp = 127 if out_dtype == I8 else (32767 if out_dtype == I16 else 2 ** 31 - 1)
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=1,
              out_dtype=out_dtype, out_clamp=clamp, residual_dy=(1717986918, 29))
    word = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    assert B.lib().ibert_gemm_config_override(cfg) > cfg
    B.ibert_gemm_epilogue_record(word)
    try:
        G.say("gemm cfg %d out=%d res=%s shift=%d" % (cfg, out_dtype, res, shift))
        got = G.gemm(kw, A, W, bias, mult, shifts, R, out_elems=M * N)
    finally:
        B.ibert_gemm_epilogue_record(None)
        B.lib().ibert_gemm_config_override(-1)
    assert int(word.item()) == (B.EPILOGUE_DIRECT if form == "direct" else B.EPILOGUE_STAGED)
    spec = GemmSpec(M, N, K, per_channel=1, dy=(1, 0), out_dtype=I32 if out_dtype == I16 else out_dtype, out_clamp=clamp,
                    res_dy=(1717986918, 29))
    want = oracle.gemm_requant(spec, A, W, bias, mult, shifts, R)
    _eq(got, want, "gemm four rows of wavefronts")


@pytest.mark.parametrize("cfg", [15, -1])
@pytest.mark.parametrize("M,N,K", [(128, 768, 3072), (32, 32, 128), (33, 65, 144), (100, 200, 512), (7, 40, 16), (160, 96, 1000)])
def test_gemm_small_tiles(G, cfg, M, N, K):
    # the 32-row tiles of the small-batch regime, forced through the configuration override and by the launcher's
    # own choice: whole and ragged tiles, one to many K steps, a K tail
    from paper_2101_01321_amd import binding as B
    assert B.lib().ibert_gemm_config_override(cfg) > 15
    try:
        for out_dtype, pc, bias, res in [(I8, 1, True, False), (I32, 1, True, True), (I8, 0, False, True), (I16, 0, True, True)]:
            G.say("gemm small tiles cfg=%d M=%d N=%d K=%d out=%d" % (cfg, M, N, K, out_dtype))
            _gemm_case(G, M, N, K, out_dtype, pc, bias, res, seed=cfg + M + N + K)
    finally:
        B.lib().ibert_gemm_config_override(-1)


@pytest.mark.parametrize("cfg,M,N,K", [(-1, 4096, 3072, 768), (6, 512, 384, 256), (7, 256, 384, 128), (10, 256, 384, 384),
                                       (13, 512, 384, 256), (13, 256, 576, 640), (14, 512, 256, 384),
                                       (9, 384, 288, 256), (10, 512, 256, 128), (-1, 100, 72, 48), (-1, 130, 64, 128),
                                       # the small tiles of the few-sequence regime carry it too, ragged edges included
                                       (3, 200, 136, 256), (15, 100, 72, 640), (15, 32, 32, 128), (-1, 128, 3072, 768)])
@pytest.mark.parametrize("S_in,S_out", [(2.0 ** -7, 8.0 / 127), (0.011, 0.02)])
def test_gemm_gelu_equals_matmul_then_gelu(G, cfg, M, N, K, S_in, S_out):
    # steps 7+8 in one call: every tile configuration that carries the GELU epilogue, the built-in choice at the
    # full Base shape, and two shapes that fall back to the two-kernel route through the scratch buffer
    from paper_2101_01321_amd import binding as B
    if (M, S_in) == (4096, 0.011):
        pytest.skip("full shape is run once")
    gp, op = B.ibert_gelu_params_from_scale(S_in, S_out), P.gelu_params(S_in, S_out)
    A, W, sw, b = synth.gemm_operands(M, N, K, layer=M + K)
    mult, shift = B.ibert_channel_dyadics_from_scales(0.03, sw, S_in)     # accumulators land on the GELU input scale
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, per_channel=1, out_dtype=I8, out_clamp=5)
    spec = GemmSpec(M, N, K, per_channel=1, dy=(1, 0), out_dtype=I32, out_clamp=gp.q_max)
    f = oracle.gemm_requant(spec, A, W, b, mult, shift, None)
    want = oracle.gelu(f.reshape(-1), op)
    assert want.min() < 0 < want.max() and len(np.unique(want)) > 20     # not a degenerate case
    B.lib().ibert_gemm_config_override(cfg)
    try:
        G.say("gemm+gelu cfg=%d M=%d N=%d K=%d S_in=%g" % (cfg, M, N, K, S_in))
        got, scratch = G.gemm_gelu(kw, A, W, b, mult, shift, gp, M * N)
    finally:
        B.lib().ibert_gemm_config_override(-1)
    _eq(got, want, "gemm+gelu")
    one_kernel = K % 128 == 0 and (M % 128 == 0 or cfg in (3, 15))
    assert np.all(scratch == -5) == one_kernel                              # scratch untouched iff GELU ran in the epilogue
    if not one_kernel:
        _eq(scratch, f.reshape(-1), "scratch holds the MatMul result")
        with pytest.raises(B.IbertError):
            G.gemm_gelu(kw, A, W, b, mult, shift, gp, M * N, with_scratch=False)


@pytest.mark.parametrize("cfg,M,N,K", [(6, 256, 192, 256), (9, 128, 192, 384), (7, 128, 128, 128), (11, 128, 96, 640),
                                       (20, 128, 192, 384), (21, 128, 192, 384), (21, 256, 96, 128), (22, 128, 256, 640)])
def test_gemm_direct_to_lds_tiles_batched(G, cfg, M, N, K):
    # whole-tile configurations on a batched problem: 2 x 3 batch elements, W shared along the outer batch axis,
    # odd workgroup counts (no XCD run) and even ones
    from paper_2101_01321_amd import binding as B
    rng = np.random.default_rng(cfg * 1000 + M + K)
    bo, bi = 2, 3
    A = rng.integers(-127, 128, size=(bo * bi, M, K), dtype=np.int8)
    W = rng.integers(-127, 128, size=(bi, N, K), dtype=np.int8)
    R = rng.integers(-127, 128, size=(bo * bi, M, N), dtype=np.int8)
    B.lib().ibert_gemm_config_override(cfg)
    try:
        for od, dy, res in ((I8, (1518500250, 44), None), (I32, (1518500250, 38), R)):
            kw = dict(M=M, N=N, K=K, batch_outer=bo, batch_inner=bi, lda=K, ldw=K, ldc=N, ldr=N,
                      strideA_outer=bi * M * K, strideA_inner=M * K, strideW_outer=0, strideW_inner=N * K,
                      strideC_outer=bi * M * N, strideC_inner=M * N, strideR_outer=bi * M * N, strideR_inner=M * N,
                      per_channel=0, requant=dy, out_dtype=od, out_clamp=127 if od == I8 else 32767, residual_dy=(1717986918, 33))
            G.say("gemm direct-to-LDS batched cfg=%d M=%d N=%d K=%d out=%d" % (cfg, M, N, K, od))
            got = G.gemm(kw, A, W, residual=res, out_elems=bo * bi * M * N)
            spec = GemmSpec(M, N, K, lda=K, ldw=K, ldc=N, ldr=N, batch_outer=bo, batch_inner=bi, sA=(bi * M * K, M * K),
                            sW=(0, N * K), sC=(bi * M * N, M * N), sR=(bi * M * N, M * N), per_channel=0, dy=dy, out_dtype=od,
                            out_clamp=127 if od == I8 else 32767, res_dy=(1717986918, 33))
            want = oracle.gemm_requant(spec, A.reshape(-1), W.reshape(-1), None, None, None,
                                       None if res is None else res.reshape(-1), out_elems=bo * bi * M * N)
            _eq(got, want, "batched direct-to-LDS gemm")
    finally:
        B.lib().ibert_gemm_config_override(-1)


@pytest.mark.parametrize("cfg", [6, 9, 13])
@pytest.mark.parametrize("table", [True, False])
@pytest.mark.parametrize("S_in,S_out", [(2.0 ** -7, 8.0 / 127), (2.0 ** -6, 0.748), (0.011, 0.02)])
def test_gemm_gelu_every_gelu_input_value(G, cfg, table, S_in, S_out):
    # Drive the MatMul so that its requantized outputs walk through every integer from below -q_max to above +q_max.
    # table=True: shifts of 33 (the register-direct epilogue), where the fused kernel reads GELU from its table in LDS,
    # outside of which the function is constant -- the kernel's label must say that the table was used;
    # table=False: shifts of 30, which take the general requantization and the arithmetic form of GELU.
    from paper_2101_01321_amd import binding as B
    gp, op = B.ibert_gelu_params_from_scale(S_in, S_out), P.gelu_params(S_in, S_out)
    M, N, K = 768, 384, 128
    f_mul = 8 if table else 1                               # accumulators are f_mul times the value they requantize to
    A = np.zeros((M, K), np.int8)
    W = np.zeros((N, K), np.int8)
    a0 = np.arange(M) % 255 - 127
    c = np.where(np.arange(M) < 765, np.arange(M) // 255 - 1, 0)
    W[:, :2 * f_mul] = 127
    A[:, :f_mul] = a0[:, None]                              # acc = f_mul (127 a0 + 16129 c + bias'), c in {-1, 0, 1}
    A[:, f_mul:2 * f_mul] = (127 * c)[:, None]
    bias = (f_mul * (np.arange(N) % 128 - 64)).astype(np.int32)   # fills the gaps of 127 between products
    mult = np.full(N, 2 ** 30, np.int32)
    shift = np.full(N, 33 if table else 30, np.int32)       # DY(acc; 2^30, 33) = acc / 8 exactly; DY(acc; 2^30, 30) = acc
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, per_channel=1, out_dtype=I8, out_clamp=5)
    f = oracle.gemm_requant(GemmSpec(M, N, K, per_channel=1, dy=(1, 0), out_dtype=I32, out_clamp=gp.q_max), A, W, bias, mult, shift, None)
    hit = np.unique(f)
    span = min(gp.q_max, 32000)
    assert hit.min() <= -span and hit.max() >= span and np.all(np.diff(hit) == 1)      # every integer in between
    want = oracle.gelu(f.reshape(-1), op)
    import torch
    word = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    B.lib().ibert_gemm_config_override(cfg)
    B.ibert_gemm_epilogue_record(word)
    try:
        G.say("gemm+gelu sweep cfg=%d S_in=%g table=%s" % (cfg, S_in, table))
        got, scratch = G.gemm_gelu(kw, A, W, bias, mult, shift, gp, M * N)
    finally:
        B.ibert_gemm_epilogue_record(None)
        B.lib().ibert_gemm_config_override(-1)
    assert np.all(scratch == -5)                             # one kernel
    assert int(word.item()) == (B.EPILOGUE_DIRECT_GELU_TABLE if table else B.EPILOGUE_STAGED)
    _eq(got, want, "gemm+gelu sweep")


@pytest.mark.parametrize("cfg", [21, 22])
@pytest.mark.parametrize("table", [True, False])
def test_gemm_gelu_every_gelu_input_value_on_tiles_with_loaders(G, cfg, table):
    test_gemm_gelu_every_gelu_input_value(G, cfg, table, 2.0 ** -6, 0.748)


def test_gemm_base_shapes_full(G):
    # the four projection GEMMs of RoBERTa-Base at batch 32 (T = 4096), full outputs
    for M, N, K, od, res in [(4096, 2304, 768, I8, False), (4096, 768, 768, I32, True), (4096, 3072, 768, I32, False),
                             (4096, 768, 3072, I32, True)]:
        G.say("gemm base M=%d N=%d K=%d" % (M, N, K))
        _gemm_case(G, M, N, K, od, 1, True, res, seed=N + K)


@pytest.mark.parametrize("H,F", [(1024, 4096), (768, 3072)])
def test_gemm_projection_shapes_at_32768_tokens_full(G, H, F):
    # the four projection GEMMs of RoBERTa-Large at batch 256 and of RoBERTa-Base at 512 tokens x 64 (T = 32768), whole
    # outputs, in the output types and with the tile configurations the encoder runs them with
    T = 32768
    for M, N, K, od, res in [(T, 3 * H, H, I8, False), (T, H, H, I16, True), (T, F, H, I32, False), (T, H, F, I16, True)]:
        G.say("gemm T=32768 M=%d N=%d K=%d out=%d" % (M, N, K, od))
        _gemm_case(G, M, N, K, od, 1, True, res, seed=N + K + 1)


# ------------------------------------------------------------------------------------------- layer / encoder
def _layer_case(G, cfg, n_layers=1, route=0):
    return _layer_case_body(G, cfg, n_layers, route)


def _layer_case_body(G, cfg, n_layers, route):
    import torch
    x_q, S_x, _ = synth.input_activations(cfg)
    from paper_2101_01321_amd import binding as B
    model = G.DeviceModel(cfg, S_x, n_layers=n_layers)
    model.set_route(route)
    one_kernel_attention = cfg.seq in (128, 256, 384, 512) and cfg.hidden == 64 * cfg.heads
    cur = x_q
    tx = G.to_dev(x_q)
    for l in range(n_layers):
        raw = synth.layer_raw(cfg, l)
        w, q = P.layer_params(raw, model.scales[l], cfg.hidden, cfg.heads)
        want, inter = oracle.encoder_layer(w, q, cur, cfg.batch, cfg.seq, cfg.hidden, cfg.heads, cfg.ffn, dump=True)
        G.say("layer %s l=%d route=%d" % (cfg.name, l, route))
        model.mark_unwritten()
        ty = model.layer_forward(l, tx)
        torch.cuda.synchronize()
        got_inter = model.intermediates(r_half=not (route & B.ROUTE_I32_LN_INPUT))
        for k in ("qkv", "scores", "probs", "ctx", "r1", "h1", "f1", "g", "r2"):
            if k == "f1" and not (route & B.ROUTE_SEPARATE_GELU):
                continue                                     # not materialised when GELU runs in the MatMul epilogue
            if k in ("r1", "r2"):
                assert model.was_written(k)
            if k in ("scores", "probs") and not (route & B.ROUTE_SEPARATE_ATTENTION) and one_kernel_attention:
                continue                                     # nor these when attention is one kernel
            _eq(got_inter[k], inter[k], "%s layer %d %s" % (cfg.name, l, k))
        _eq(ty.cpu().numpy(), want, "%s layer %d output" % (cfg.name, l))
        cur, tx = want, ty
    return model, x_q, cur


def test_layer_tiny_every_intermediate(G):
    for route in range(8):                                   # every combination of fused and separate kernels
        _layer_case(G, synth.CONFIGS["tiny"], route=route)


def test_layer_whole_tile_shape_fused_and_unfused(G):
    # hidden/ffn/tokens that fit the whole-tile MatMul configurations, so that every fusion really runs its fused kernel
    cfg = synth.EncoderConfig("tiles", 256, 4, 1024, 128, 16, 1)
    for route in range(8):
        _layer_case(G, cfg, route=route)
    _layer_case(G, synth.EncoderConfig("tiles96", 384, 6, 1536, 128, 4, 2), n_layers=2)


@pytest.mark.parametrize("M,N,K", [(4096, 768, 768), (4096, 768, 3072), (4096, 1024, 1024), (256, 768, 768), (1024, 384, 2048),
                                   (100, 96, 128), (130, 250, 64), (5, 3, 16)])
def test_gemm_i16_then_layernorm_i16(G, M, N, K):
    # steps 5+6 / 9+10 as the layer runs them: a projection with residual whose clamped result is stored as int16, and the
    # LayerNorm kernel that reads int16 -- against the oracle's INT32 MatMul and LayerNorm
    from paper_2101_01321_amd import binding as B
    A, W, sw, b = synth.gemm_operands(M, N, K, layer=M + N + K)
    mult, shift = B.ibert_channel_dyadics_from_scales(0.03, sw, 2.5e-4 * math.sqrt(K))   # rows spread over the 16-bit range
    R = np.random.default_rng(K).integers(-127, 128, size=(M, N), dtype=np.int8)
    gamma = np.random.default_rng(N).normal(1.0, 0.1, size=N)
    beta = np.random.default_rng(N + 1).normal(0.0, 0.1, size=N)
    gq, bq, s = B.ibert_layernorm_params_from_float(gamma, beta, 5.0 / 127)
    res_dy = (1717986918, 23)
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=1, out_dtype=I16,
              out_clamp=32767, residual_dy=res_dy)
    spec = GemmSpec(M, N, K, per_channel=1, dy=(1, 0), out_dtype=I32, out_clamp=32767, res_dy=res_dy)
    r = oracle.gemm_requant(spec, A, W, b, mult, shift, R).reshape(M, N)
    top, clamped = int(np.abs(r).max()), float((np.abs(r) == 32767).mean())
    assert top > 2000 and clamped < 0.2, (top, clamped)                           # a real spread, few clamped values
    G.say("gemm int16 + layernorm int16 M=%d N=%d K=%d" % (M, N, K))
    got_r = G.gemm(kw, A, W, b, mult, shift, R, out_elems=M * N).reshape(M, N)
    _eq(got_r.astype(np.int32), r, "int16 MatMul output")
    _eq(G.layernorm(got_r, gq, bq, s, half=True), oracle.layernorm(r, gq, bq, s), "layernorm of the int16 rows")


def test_layer_replayed_from_a_graph(G):
    # the whole layer captured into a HIP graph: every replay (with eager work and synchronisation in between, and a
    # different input each time) must give the oracle's result
    import torch
    from paper_2101_01321_amd import binding as B
    cfg = synth.EncoderConfig("graph", 384, 6, 1536, 128, 4, 1)
    x_q, S_x, _ = synth.input_activations(cfg)
    model = G.DeviceModel(cfg, S_x)
    w, q = P.layer_params(synth.layer_raw(cfg, 0), model.scales[0], cfg.hidden, cfg.heads)
    stream = torch.cuda.Stream()
    tx = G.to_dev(x_q)
    ty = torch.empty_like(tx)

    def run():
        B.ibert_encoder_layer_i(model.layers[0].weights, model.layers[0].quant, tx, ty, cfg.batch, cfg.seq, cfg.hidden,
                                cfg.heads, cfg.ffn, model.ws, stream=stream)
    with torch.cuda.stream(stream):
        run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        run()
    for rep in range(3):
        x_rep = np.roll(x_q, rep * 7 + 1, axis=0) if rep else x_q
        x_rep = np.ascontiguousarray(x_rep)
        want = oracle.encoder_layer(w, q, x_rep, cfg.batch, cfg.seq, cfg.hidden, cfg.heads, cfg.ffn)
        tx.copy_(G.to_dev(x_rep))
        ty.zero_()
        torch.cuda.synchronize()
        G.say("graph replay %d of the layer" % rep)
        graph.replay()
        torch.cuda.synchronize()
        _eq(ty.cpu().numpy(), want, "replay %d" % rep)


def test_layer_ragged_every_intermediate(G):
    _layer_case(G, synth.EncoderConfig("ragged", 192, 3, 320, 40, 2, 1))
    _layer_case(G, synth.EncoderConfig("ragged2", 320, 5, 200, 77, 3, 2), n_layers=2)
    # 32-bit LayerNorm inputs and separate kernels on shapes that take the ragged-tile, K-tail and byte-load MatMul kernels
    _layer_case(G, synth.EncoderConfig("ragged", 192, 3, 320, 40, 2, 1), route=7)
    _layer_case(G, synth.EncoderConfig("ragged2", 320, 5, 200, 77, 3, 2), n_layers=2, route=4)


def test_encoder_base_b1_all_layers(G):
    import torch
    cfg = synth.CONFIGS["base_b1"]
    model, x_q, want = _layer_case(G, cfg, n_layers=cfg.layers)
    G.say("encoder base_b1 12 layers in one call")
    y = model.forward(G.to_dev(x_q))
    torch.cuda.synchronize()
    _eq(y.cpu().numpy(), want, "base_b1 encoder")


def _oracle_sequences(cfg, x_q, scales, seqs, n_layers):
    """Oracle forward of selected sequences (sequences are independent: no op mixes tokens across them)."""
    one = cfg.with_batch(1)
    out = {}
    L, H = cfg.seq, cfg.hidden
    cur = {s: x_q[s * L:(s + 1) * L] for s in seqs}
    for l in range(n_layers):
        raw = synth.layer_raw(cfg, l)
        w, q = P.layer_params(raw, scales[l], cfg.hidden, cfg.heads)
        for s in seqs:
            cur[s] = oracle.encoder_layer(w, q, cur[s], 1, one.seq, H, cfg.heads, cfg.ffn)
    return cur


# Sampled sequences: the first and the last, sequences in the middle of a 256-row MatMul tile and at its edges, on both
# sides of the boundaries between the runs of tiles the eight XCDs work on, and (32768 tokens) far past row 8192, where
# the LayerNorm kernel switches to its wide form.
@pytest.mark.parametrize("name,seqs", [("base_b32", (0, 1, 7, 13, 16, 24, 31)), ("large_b32", (0, 5, 11, 16, 21, 27, 31)),
                                       ("large_b256", (0, 1, 37, 63, 64, 100, 128, 129, 200, 255)),
                                       ("base512_b64", (0, 7, 21, 32, 33, 50, 63))])
def test_encoder_full_size_sampled_sequences(G, name, seqs):
    import torch
    cfg = synth.CONFIGS[name]
    x_q, S_x, _ = synth.input_activations(cfg)
    G.say("encoder %s: building %d layers" % (name, cfg.layers))
    model = G.DeviceModel(cfg, S_x)
    G.say("encoder %s: GPU forward (the default route, which the benchmark times)" % name)
    y = model.forward(G.to_dev(x_q))
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    # the whole output again with every step a kernel of its own and 32-bit LayerNorm inputs: the two routes share the
    # MatMul main loops and little else, and must agree on every element
    model.set_route(7)
    G.say("encoder %s: GPU forward, separate kernels" % name)
    y7 = model.forward(G.to_dev(x_q))
    torch.cuda.synchronize()
    _eq(y7.cpu().numpy(), y, "%s: separate kernels against the default route, whole output" % name)
    del y7
    G.say("encoder %s: oracle on sequences %s" % (name, (seqs,)))
    want = _oracle_sequences(cfg, x_q, model.scales, seqs, cfg.layers)
    L = cfg.seq
    for s in seqs:
        _eq(y[s * L:(s + 1) * L], want[s], "%s sequence %d" % (name, s))
    # properties that hold at any size: int8 range, not degenerate
    assert y.min() >= -127 and y.std() > 5


@pytest.mark.parametrize("shape", ["base", "large"])
@pytest.mark.parametrize("batch", [1, 8])
def test_encoder_latency_grid_shapes(G, shape, batch):
    # the shapes of Table 3 at sequence length 256 (the grid's other half, length 128, is covered by the configurations
    # above and below): all layers, whole output against the oracle
    import torch
    base = synth.CONFIGS["base_b1" if shape == "base" else "large_b32"]
    cfg = synth.EncoderConfig("%s_s256_b%d" % (shape, batch), base.hidden, base.heads, base.ffn, 256, batch, base.layers)
    x_q, S_x, _ = synth.input_activations(cfg)
    model = G.DeviceModel(cfg, S_x)
    G.say("encoder %s: GPU forward" % cfg.name)
    y = model.forward(G.to_dev(x_q))
    torch.cuda.synchronize()
    G.say("encoder %s: oracle" % cfg.name)
    cur = x_q
    for l in range(cfg.layers):
        w, q = P.layer_params(synth.layer_raw(cfg, l), model.scales[l], cfg.hidden, cfg.heads)
        cur = oracle.encoder_layer(w, q, cur, cfg.batch, cfg.seq, cfg.hidden, cfg.heads, cfg.ffn)
    _eq(y.cpu().numpy(), cur, "%s encoder" % cfg.name)


# ------------------------------------------------------------------------------------------- padded sequences
@pytest.mark.parametrize("cols,rpl", [(5, 1), (64, 7), (128, 24), (200, 3), (384, 5), (513, 2), (2500, 4)])
def test_softmax_masked_matches_oracle(G, cols, rpl):
    from paper_2101_01321_amd import binding as B
    nseq = 9
    rows = nseq * rpl - (rpl // 2)                           # the last group of rows is short
    x, S = synth.softmax_logits(rows, cols)
    if oracle.lib().orc_softmax_check(P.softmax_params(S), cols) != 0:
        S = 2.0 ** -4
    x[rpl, :] = -2 ** 31 + 3                                 # real logits at the bottom of the range (a row with one real
                                                             # key): the masked e_j are not 0 there
    lens = np.array([cols, 1, 2, cols - 1, max(1, cols // 2), 3, 4, max(1, cols - 3), max(1, cols // 3)], np.int32).clip(1, cols)
    sp, op = B.ibert_softmax_params_from_scale(S, cols), P.softmax_params(S)
    xm = x.copy()
    for r in range(rows):
        xm[r, lens[r // rpl]:] = -2 ** 31
    want = oracle.softmax(xm, op)
    G.say("softmax masked cols=%d rows_per_len=%d" % (cols, rpl))
    _eq(G.softmax(x, sp, key_lens=lens, rows_per_len=rpl), want, "masked softmax cols=%d" % cols)
    if cols in (5, 513):
        got = G.softmax(x, sp, ldx=cols + 3, ldy=cols + 1, x_off=1, y_off=3, key_lens=lens, rows_per_len=rpl)
        _eq(got[:, :cols], want, "masked softmax unaligned cols=%d" % cols)
    # lengths outside [1, cols] are clamped into it
    wild = lens.copy()
    wild[0], wild[1] = cols + 1000, -5
    _eq(G.softmax(x, sp, key_lens=wild, rows_per_len=rpl), want, "clamped lengths cols=%d" % cols)


@pytest.mark.parametrize("B_,nh,L,S,sdy,cdy,lens", [
    (4, 3, 128, 2.0 ** -6, (1518500250, 36), (1073741824, 37), (128, 1, 77, 64)),
    (3, 2, 128, 2.0 ** -2, (1518500250, 41), (60000, 22), (5, 127, 16)),           # general Softmax / requantization forms
    (2, 2, 256, 2.0 ** -6, (1187698534, 28), (1073741824, 37), (200, 65)),
    (2, 1, 512, 2.0 ** -6, (1187698534, 28), (1518500250, 38), (512, 300)),
    (3, 2, 72, 2.0 ** -6, (1518500250, 36), (1073741824, 37), (72, 10, 71)),       # three kernels through scratch
])
def test_attention_masked(G, B_, nh, L, S, sdy, cdy, lens):
    from paper_2101_01321_amd import binding as B
    H = nh * 64
    rng = np.random.default_rng(B_ * 100 + nh * 10 + L + 1)
    qkv = np.clip(np.rint(rng.normal(0, 40, size=(B_ * L, 3 * H))), -127, 127).astype(np.int8)
    lens = np.array(lens, np.int32)
    sp, op = B.ibert_softmax_params_from_scale(S, L), P.softmax_params(S)
    # oracle: scores, mask, Softmax, context, step by step
    dh, flat = 64, qkv.reshape(-1)
    spec = GemmSpec(L, L, dh, lda=3 * H, ldw=3 * H, ldc=L, batch_outer=B_, batch_inner=nh, sA=(L * 3 * H, dh),
                    sW=(L * 3 * H, dh), sC=(nh * L * L, L * L), per_channel=0, dy=sdy, out_dtype=I32, out_clamp=2 ** 31 - 1)
    scores = oracle.mask_scores(oracle.gemm_requant(spec, flat, flat[H:], out_elems=B_ * nh * L * L), B_, nh, L, lens)
    probs = oracle.softmax(scores.reshape(-1, L), op)
    spec = GemmSpec(L, dh, L, lda=L, ldw=3 * H, ldc=H, batch_outer=B_, batch_inner=nh, trans_w=1, sA=(nh * L * L, L * L),
                    sW=(L * 3 * H, dh), sC=(L * H, dh), per_channel=0, dy=cdy, out_dtype=I8, out_clamp=127)
    want = oracle.gemm_requant(spec, probs.reshape(-1), flat[2 * H:], out_elems=B_ * L * H).reshape(B_ * L, H)
    assert not np.array_equal(want, _attention_oracle(qkv, B_, L, H, nh, sdy, op, cdy))   # the mask matters
    G.say("masked attention B=%d heads=%d L=%d" % (B_, nh, L))
    _eq(G.attention(qkv, B_, L, H, nh, sdy, sp, cdy, key_lens=lens), want, "masked attention")


@pytest.mark.parametrize("cfg,lens", [
    (synth.EncoderConfig("masked", 128, 2, 256, 128, 3, 2), (128, 29, 1)),         # one-kernel attention
    (synth.EncoderConfig("masked_ragged", 192, 3, 320, 40, 3, 1), (40, 7, 39)),    # three-kernel attention
])
def test_layer_masked_every_row(G, cfg, lens):
    import torch
    from paper_2101_01321_amd import binding as B
    x_q, S_x, _ = synth.input_activations(cfg)
    lens = np.array(lens, np.int32)
    tl = G.to_dev(lens)
    for route in (0, 7):
        model = G.DeviceModel(cfg, S_x)
        model.set_route(route)
        cur, tx = x_q, G.to_dev(x_q)
        for l in range(cfg.layers):
            w, q = P.layer_params(synth.layer_raw(cfg, l), model.scales[l], cfg.hidden, cfg.heads)
            want = oracle.encoder_layer(w, q, cur, cfg.batch, cfg.seq, cfg.hidden, cfg.heads, cfg.ffn, key_lens=lens)
            G.say("masked layer %s l=%d route=%d" % (cfg.name, l, route))
            ty = model.layer_forward(l, tx, key_lens=tl)
            torch.cuda.synchronize()
            _eq(ty.cpu().numpy(), want, "%s layer %d" % (cfg.name, l))
            cur, tx = want, ty
        G.say("masked encoder %s in one call" % cfg.name)
        y = model.forward(G.to_dev(x_q), key_lens=tl)
        torch.cuda.synchronize()
        _eq(y.cpu().numpy(), cur, "%s encoder" % cfg.name)


def test_encoder_masked_full_size_sampled_sequences(G):
    # Base, sequence length 128, batch 32 with a mix of lengths: a padded sequence equals, on its real tokens, the
    # same tokens run alone at their own length (the oracle never sees the padding)
    import torch
    cfg = synth.CONFIGS["base_b32"]
    x_q, S_x, _ = synth.input_activations(cfg)
    lens = synth.key_lengths(cfg.batch, cfg.seq)
    G.say("masked encoder base_b32: building")
    model = G.DeviceModel(cfg, S_x)
    y = model.forward(G.to_dev(x_q), key_lens=G.to_dev(lens))
    torch.cuda.synchronize()
    y = y.cpu().numpy().reshape(cfg.batch, cfg.seq, cfg.hidden)
    L, H = cfg.seq, cfg.hidden
    for s in (3, int(np.argmin(lens))):
        n = int(lens[s])
        G.say("masked encoder base_b32: oracle on sequence %d of length %d" % (s, n))
        cur = x_q.reshape(cfg.batch, L, H)[s, :n]
        for l in range(cfg.layers):
            w, q = P.layer_params(synth.layer_raw(cfg, l), model.scales[l], H, cfg.heads)
            cur = oracle.encoder_layer(w, q, cur, 1, n, H, cfg.heads, cfg.ffn)
        _eq(y[s, :n], cur, "sequence %d" % s)


# ------------------------------------------------------------------------------------------- embedding
@pytest.mark.parametrize("H,V,seq,T", [(768, 1000, 128, 4096 + 37), (1024, 300, 512, 1500), (64, 50, 20, 60), (100, 17, 9, 31),
                                       (3, 5, 4, 11), (257, 40, 33, 70)])
def test_embedding_matches_oracle(G, H, V, seq, T):
    emb = synth.embedding_raw(H, V, seq + 2)
    tok_dy, pos_dy, gq, bq, s = P.embedding_params(emb, 5.0 / 127)
    ids = synth.token_ids(T, V)
    ids[:4] = [0, V - 1, -7, V + 100]
    want = oracle.embedding(ids, seq, emb["tok"], emb["pos"], tok_dy, pos_dy, gq, bq, s)
    G.say("embedding H=%d V=%d seq=%d T=%d" % (H, V, seq, T))
    _eq(G.embedding(ids, seq, emb["tok"], emb["pos"], tok_dy, pos_dy, gq, bq, s), want, "embedding")
    if H in (100, 257, 768):
        G.say("embedding H=%d padded/unaligned output rows" % H)
        _eq(G.embedding(ids, seq, emb["tok"], emb["pos"], tok_dy, pos_dy, gq, bq, s, ldy=H + 3, y_off=1), want, "embedding ldy")
    # dyadics that drive the sum into the clamp
    big = ((2 ** 31 - 1, 20), (2 ** 30, 22))
    want = oracle.embedding(ids, seq, emb["tok"], emb["pos"], big[0], big[1], gq, bq, s)
    _eq(G.embedding(ids, seq, emb["tok"], emb["pos"], big[0], big[1], gq, bq, s), want, "embedding, clamped sum")


def test_embedding_feeds_the_encoder(G):
    # ids -> embedding -> masked encoder, all on the device, against the oracle chain
    import torch
    from paper_2101_01321_amd import binding as B
    cfg = synth.EncoderConfig("emb", 128, 2, 256, 128, 2, 2)
    emb = synth.embedding_raw(cfg.hidden, 500, cfg.seq)
    S_x = 5.0 / 127
    tok_dy, pos_dy, gq, bq, s = P.embedding_params(emb, S_x)
    ids = synth.token_ids(cfg.tokens, 500)
    lens = np.array([128, 50], np.int32)
    x_want = oracle.embedding(ids, cfg.seq, emb["tok"], emb["pos"], tok_dy, pos_dy, gq, bq, s)
    model = G.DeviceModel(cfg, S_x)
    cur = x_want
    for l in range(cfg.layers):
        w, q = P.layer_params(synth.layer_raw(cfg, l), model.scales[l], cfg.hidden, cfg.heads)
        cur = oracle.encoder_layer(w, q, cur, cfg.batch, cfg.seq, cfg.hidden, cfg.heads, cfg.ffn, key_lens=lens)
    tx = torch.empty(cfg.tokens, cfg.hidden, dtype=torch.int8, device=G.DEV)
    G.say("embedding + masked encoder")
    B.ibert_embedding_i(G.to_dev(ids), G.to_dev(emb["tok"]), G.to_dev(emb["pos"]), cfg.tokens, cfg.seq, cfg.hidden, 500,
                        cfg.seq, B.Dyadic(*tok_dy), B.Dyadic(*pos_dy), G.to_dev(gq), G.to_dev(bq), s, tx, cfg.hidden)
    y = model.forward(tx, key_lens=G.to_dev(lens))
    torch.cuda.synchronize()
    _eq(tx.cpu().numpy(), x_want, "embedding output")
    _eq(y.cpu().numpy(), cur, "encoder on the embedded tokens")


def test_dequantised_output_tracks_float_layer(G):
    """Tolerance check on GPU outputs: one tiny layer, each op against its float counterpart (teacher-forced)."""
    import torch
    import fpref
    cfg = synth.CONFIGS["tiny"]
    x_q, S_x, _ = synth.input_activations(cfg)
    from paper_2101_01321_amd import binding as B
    model = G.DeviceModel(cfg, S_x)
    model.set_route(7)                                        # every intermediate is materialised, 32 bits wide
    y = model.layer_forward(0, G.to_dev(x_q))
    torch.cuda.synchronize()
    d, sc, raw = model.intermediates(), model.scales[0], synth.layer_raw(cfg, 0)
    assert np.abs(d["scores"]).max() > 0 and d["probs"].max() > 0 and np.abs(d["f1"]).max() > 0 and np.abs(d["r2"]).max() > 0
    assert np.max(np.abs(d["probs"] / 128.0 - fpref.softmax(d["scores"] * sc["S_s"]))) <= 0.02
    want = np.clip(fpref.gelu(d["f1"] * sc["S_g_in"]) / sc["S_g_out"], -127, 127)
    assert np.max(np.abs(d["g"] - want)) <= 0.6
    want = np.clip(fpref.layernorm(d["r2"] * sc["S_r2"], raw["gamma2"], raw["beta2"]) / sc["S_y"], -127, 127)
    assert np.max(np.abs(y.cpu().numpy() - want)) <= 1.0
    want = np.clip(fpref.linear(x_q * S_x, raw["w_qkv"], raw["sw_qkv"], raw["b_qkv"], S_x) / sc["S_q"], -127, 127)
    assert np.max(np.abs(d["qkv"] - want)) <= 0.5 + 1e-5
