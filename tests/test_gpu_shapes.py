"""GPU parity at the edges of the shapes each kernel variant serves: lengths that no block or tile divides, the first and
last member of each range, and the switches between variants -- against the CPU oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from oracle import params as P, GemmSpec, I8, I32
from paper_2101_01321_amd import synth
from test_gpu_parity import G, _attention_oracle, _eq, _layer_case, I16  # noqa: F401  (G is the fixture)


def _qkv(B_, L, H, seed):
    qkv = np.clip(np.rint(np.random.default_rng(seed).normal(0, 40, size=(B_ * L, 3 * H))), -127, 127).astype(np.int8)
    qkv[0, :] = 127                                          # a saturated query/key/value row
    qkv[L - 1, H:2 * H] = -127                               # the last key of a sequence
    return qkv


def _attention_form(sdy, sp, cdy, workgroups):
    import ctypes as C
    from paper_2101_01321_amd import binding as B
    form = C.c_int32()
    assert B.lib().ibert_attention_form(C.byref(B.Dyadic(*sdy)), C.byref(sp), C.byref(B.Dyadic(*cdy)), workgroups, C.byref(form)) == 0
    return form.value


# ------------------------------------------------------------------------------------------- attention, any length
@pytest.mark.parametrize("L", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 191, 192, 193, 251, 255, 257, 319, 321, 384, 385, 447, 449,
                               511, 512])
@pytest.mark.parametrize("S,k,sdy,form", [(2.0 ** -6, 7, (1518500250, 36), 4), (2.0 ** -6, 7, (1187698534, 28), 3),
                                          (2.0 ** -4, 5, (1518500250, 36), 4),        # q_ln2 = 11, fewer output bits
                                          (2.0 ** -8, 7, (1518500250, 36), 1), (2.0 ** -8, 7, (1187698534, 28), 2),   # an exponent of 18 bits: no table
                                          (2.0 ** -6, 7, (-1518500250, 36), 0)])      # a negative multiplier: the general form
def test_attention_any_length(G, L, S, k, sdy, form):
    from paper_2101_01321_amd import binding as B
    B_, nh = 2, 3
    H, cdy = 64 * nh, (1073741824, 37 if k == 7 else 35)
    qkv = _qkv(B_, L, H, L)
    sp, op = B.ibert_softmax_params_from_scale(S, L, k), P.softmax_params(S, k)
    assert _attention_form(sdy, sp, cdy, B_ * nh * -(-L // 64)) == form
    G.say("attention L=%d S=%g k=%d s=%s" % (L, S, k, sdy))
    want = _attention_oracle(qkv, B_, L, H, nh, sdy, op, cdy)
    _eq(G.attention(qkv, B_, L, H, nh, sdy, sp, cdy), want, "attention L=%d" % L)
    if k != 7 or sdy[0] < 0:
        return
    # masked: lengths that cut a block of keys, end with one, leave a single key, and leave all
    for lens in ((L, 1), ((L + 1) // 2, max(1, L - 1)), (min(L, 64), min(L, 65))):
        lens = np.array(lens, np.int32)
        G.say("attention L=%d lens=%s" % (L, lens))
        got = G.attention(qkv, B_, L, H, nh, sdy, sp, cdy, key_lens=lens).reshape(B_, L, H)
        for b in range(B_):
            # (a query attends to the first lens[b] keys: take those keys alone, all queries by the rows of a longer batch)
            n = int(lens[b])
            own = qkv.reshape(B_, L, 3 * H)[b]
            for q0 in range(0, L, n):                        # the queries in groups of n, each group with the same n keys
                rows = np.arange(q0, min(q0 + n, L))
                part = np.zeros((n, 3 * H), np.int8)
                part[:, H:] = own[:n, H:]
                part[:len(rows), :H] = own[rows, :H]
                want_part = _attention_oracle(part, 1, n, H, nh, sdy, op, cdy)
                _eq(got[b][rows], want_part[:len(rows)], "masked attention L=%d n=%d rows %d.." % (L, n, q0))
                if n < 8 and q0 >= 16:
                    break                                    # (one key: every query gives the same; a few groups are enough)


def _buffers(L, form, workgroups):
    import ctypes as C
    from paper_2101_01321_amd import binding as B
    out = [C.c_int32() for _ in range(3)]
    assert B.lib().ibert_attention_buffers(L, form, workgroups, *[C.byref(o) for o in out]) == 0
    return [o.value for o in out]


@pytest.mark.parametrize("L", [385, 448, 449, 512])
@pytest.mark.parametrize("form", [0, 1, 2])
def test_attention_shares_a_buffer_only_where_more_workgroups_fit(G, L, form):
    # one buffer is there to let a compute unit hold more workgroups: it is used where that is so and there are more than 512
    shared, two, one = _buffers(L, form, 513)
    assert two == 2 and shared == (one > two), (shared, two, one)
    assert _buffers(L, form, 512)[0] == 0


@pytest.mark.parametrize("L,form", [(321, 3), (384, 4), (385, 3), (448, 4), (449, 3), (512, 4)])
def test_attention_with_a_table_shares_a_buffer_only_where_more_workgroups_fit(G, L, form):
    shared, two, one = _buffers(L, form, 513)
    assert two == 2 and one > two and shared, (shared, two, one)
    assert _buffers(L, form, 512)[0] == 0


# The table of the exponent: shifts on both sides of 33, the smallest one and the largest; multipliers on both sides of what the 32-bit product holds
# (5000 and 4900 at 23); 11 to 16 bits of the exponent and, at 2^-8, more than the table takes; one entry a step and none for some; at 2^-7 a table from 257
# workgroups on (form: with up to 256 and with more)
@pytest.mark.parametrize("S,k,sdy,form", [(2.0 ** -6, 7, (37581, 23), (3, 3)), (2.0 ** -6, 7, (5000, 23), (3, 3)), (2.0 ** -6, 7, (4900, 23), (2, 2)),
                                          (2.0 ** -6, 7, (1187698534, 33), (3, 3)), (2.0 ** -6, 7, (1187698534, 34), (4, 4)), (2.0 ** -6, 6, (2147483647, 45), (4, 4)),
                                          (2.0 ** -6, 7, (2000000011, 26), (3, 3)), (2.0 ** -4, 7, (1187698534, 30), (3, 3)), (2.0 ** -7, 7, (1187698534, 27), (2, 3)),
                                          (2.0 ** -7, 7, (1518500250, 35), (1, 4)), (2.0 ** -8, 7, (1187698534, 26), (2, 2)), (2.0 ** -8, 7, (1518500250, 34), (1, 1))])
@pytest.mark.parametrize("B_,nh,L", [(2, 3, 67), (43, 3, 128), (43, 2, 190)])         # 12, 258 and 258 workgroups
def test_attention_exponent_from_a_table(G, S, k, sdy, form, B_, nh, L):
    from paper_2101_01321_amd import binding as B
    H, cdy = 64 * nh, (1073741824, 30 + k)
    rng = np.random.default_rng(L)
    x = sdy[0] / 2.0 ** sdy[1] * S                           # of one unit of an accumulator: logits of some units, and rows of the largest products
    qkv = np.clip(np.rint(rng.normal(0, min(60.0, max(1.0, (0.4 / x) ** 0.5)), size=(B_ * L, 3 * H))), -128, 127).astype(np.int8)
    qkv[L - 2] = -128
    qkv[L - 1, H:2 * H] = 127
    sp, op = B.ibert_softmax_params_from_scale(S, L, k), P.softmax_params(S, k)
    workgroups = B_ * nh * -(-L // 64)
    assert _attention_form(sdy, sp, cdy, workgroups) == form[workgroups > 256]
    G.say("attention, table, B=%d heads=%d L=%d S=%g k=%d s=%s" % (B_, nh, L, S, k, sdy))
    got = G.attention(qkv, B_, L, H, nh, sdy, sp, cdy)
    for b in (0, B_ - 1):
        part = qkv[b * L:(b + 1) * L]
        _eq(got[b * L:(b + 1) * L], _attention_oracle(part, 1, L, H, nh, sdy, op, cdy), "attention, sequence %d" % b)
    lens = np.full(B_, 65, np.int32)
    lens[-1] = 3
    masked = G.attention(qkv, B_, L, H, nh, sdy, sp, cdy, key_lens=lens)
    for b, n in ((0, 65), (B_ - 1, 3)):
        part = qkv[b * L:b * L + n]
        _eq(masked[b * L:b * L + n], _attention_oracle(part, 1, n, H, nh, sdy, op, cdy), "masked attention, sequence %d" % b)


# 504 to 546 workgroups, on both sides of the switch at 512; lengths at, before and behind the ends of key blocks
@pytest.mark.parametrize("B_,nh,L,many", [(12, 7, 321, 0), (12, 7, 384, 0), (13, 7, 321, 1), (43, 2, 383, 1), (13, 7, 384, 1), (8, 9, 447, 0), (8, 8, 449, 0), (11, 7, 385, 1), (11, 7, 447, 1), (11, 7, 448, 1), (13, 5, 449, 1),
                                          (13, 5, 511, 1), (13, 5, 512, 1)])
@pytest.mark.parametrize("S,sdy,form", [(2.0 ** -6, (1518500250, 36), 4), (2.0 ** -6, (1187698534, 28), 3), (2.0 ** -8, (1518500250, 36), 1),
                                        (2.0 ** -8, (1187698534, 28), 2), (2.0 ** -6, (-1518500250, 36), 0)])
def test_attention_keys_and_values_in_one_buffer(G, B_, nh, L, many, S, sdy, form):
    # long sequences of more workgroups than find a place at once: V_h takes the place of K_h in LDS where that makes room for more; also
    # with masked blocks of keys, down to a single key, against the oracle on the last sequence
    from paper_2101_01321_amd import binding as B
    H, cdy = 64 * nh, (1073741824, 37)
    workgroups = B_ * nh * -(-L // 64)
    qkv = _qkv(B_, L, H, L + nh)
    sp, op = B.ibert_softmax_params_from_scale(S, L, 7), P.softmax_params(S, 7)
    assert (workgroups > 512) == bool(many) and _attention_form(sdy, sp, cdy, workgroups) == form
    if L > 384 or form >= 3:                                 # (six key blocks: only with a table)
        assert _buffers(L, form, workgroups)[0] == (many and not (form == 0 and L > 448))
    G.say("attention, one buffer, B=%d heads=%d L=%d S=%g s=%s" % (B_, nh, L, S, sdy))
    got = G.attention(qkv, B_, L, H, nh, sdy, sp, cdy)
    last = qkv[(B_ - 1) * L:]
    _eq(got[(B_ - 1) * L:], _attention_oracle(last, 1, L, H, nh, sdy, op, cdy), "attention, last sequence")
    lens = np.array([1 + (L - 1) * b // (B_ - 1) for b in range(B_)], np.int32)
    masked = G.attention(qkv, B_, L, H, nh, sdy, sp, cdy, key_lens=lens)
    _eq(masked[(B_ - 1) * L:], got[(B_ - 1) * L:], "all keys")
    n = int(lens[2])                                         # a sequence that keeps the first n keys: its first n rows, alone
    part = qkv[2 * L:2 * L + n]
    _eq(masked[2 * L:2 * L + n], _attention_oracle(part, 1, n, H, nh, sdy, op, cdy), "masked attention")


def test_layer_of_any_length_keeps_scores_and_probabilities(G):
    # a single layer call leaves every intermediate in the workspace for lengths that are no multiple of 128
    for seq in (33, 100, 131):
        _layer_case(G, synth.EncoderConfig("len%d" % seq, 192, 3, 320, seq, 2, 1))


# ------------------------------------------------------------------------------------------- persistent MatMul
def _stream_case(G, cfg, M, N, K, kind, shift, seed, kernel=None):
    """One MatMul through tile configuration cfg; shift 40: every tile takes the fast epilogue, 30: the 64-bit one.
    kernel: start of the name of the kernel that is to have run (default: the one that cfg stands for)."""
    import torch
    from paper_2101_01321_amd import binding as B
    rng = np.random.default_rng(seed)
    A = rng.integers(-127, 128, size=(M, K), dtype=np.int8)
    W = rng.integers(-127, 128, size=(N, K), dtype=np.int8)
    bias = rng.integers(-50000, 50000, size=N, dtype=np.int32)
    mult = rng.integers(2 ** 29, 2 ** 30, size=N, dtype=np.int64).astype(np.int32)
    shifts = np.full(N, {"i8": shift, "i16": shift, "i16res": shift, "gelu": min(shift, 40)}[kind], np.int32)
    R = rng.integers(-127, 128, size=(M, N), dtype=np.int8) if kind == "i16res" else None
    res_dy = (1717986918, 23)
    word = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    B.lib().ibert_gemm_config_override(cfg)
    B.ibert_gemm_epilogue_record(word)
    try:
        G.say("persistent gemm cfg %d M=%d N=%d K=%d %s shift=%d" % (cfg, M, N, K, kind, shift))
        kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=1, residual_dy=res_dy)
        if kind == "gelu":
            gp, op = B.ibert_gelu_params_from_scale(2.0 ** -6, 0.7), P.gelu_params(2.0 ** -6, 0.7)
            got, scratch = G.gemm_gelu(dict(kw, out_dtype=I8, out_clamp=5), A, W, bias, mult, shifts, gp, M * N)
            assert np.all(scratch == -5)
        else:
            clamp = 127 if kind == "i8" else 32767
            got = G.gemm(dict(kw, out_dtype=I8 if kind == "i8" else I16, out_clamp=clamp), A, W, bias, mult, shifts, R, out_elems=M * N)
    finally:
        B.ibert_gemm_epilogue_record(None)
        B.lib().ibert_gemm_config_override(-1)
    name = B.lib().ibert_last_kernel().decode()
    assert name.startswith(kernel or G.kernel_of(cfg)), name
    # (the few-row kernel stores no record; of the tiles that are not persistent only some have room for a GELU table)
    want_form = [B.EPILOGUE_STAGED] if shift < 33 else ([B.EPILOGUE_DIRECT_GELU_TABLE] if kind == "gelu" else [B.EPILOGUE_DIRECT])
    if cfg >= 25:
        want_form = [0]
    elif kind == "gelu" and shift >= 33 and "stream" not in name:
        want_form = [B.EPILOGUE_DIRECT, B.EPILOGUE_DIRECT_GELU_TABLE]
    assert int(word.item()) in want_form, (int(word.item()), want_form)
    spec = GemmSpec(M, N, K, per_channel=1, dy=(1, 0), out_dtype=I8 if kind == "i8" else I32,
                    out_clamp={"i8": 127, "gelu": gp.q_max if kind == "gelu" else 0}.get(kind, 32767), res_dy=res_dy)
    want = oracle.gemm_requant(spec, A, W, bias, mult, shifts, R).reshape(-1)
    if kind == "gelu":
        want = oracle.gelu(want, op)
    _eq(got.astype(np.int64), want.astype(np.int64), "persistent gemm")


@pytest.mark.parametrize("cfg,bn", [(23, 256), (24, 192)])
@pytest.mark.parametrize("kind", ["i8", "i16", "i16res", "gelu"])
def test_gemm_persistent_tiles(G, cfg, bn, kind):
    # K down to one pair of slices; M at, one past and far off a tile edge; more tiles than workgroups (several tiles each,
    # with and without a change of tile column); shares of the XCDs that are empty
    for M, N, K, shift in [(1, bn, 128, 40), (255, bn, 128, 40), (256, 2 * bn, 256, 40), (257, bn, 384, 40), (300, bn, 256, 30),
                           (1000, 3 * bn, 640, 40), (256 * 90 + 17, 3 * bn, 128, 40), (256 * 130 + 1, 2 * bn, 256, 40)]:
        _stream_case(G, cfg, M, N, K, kind, shift, seed=M + N + K)


@pytest.mark.parametrize("cfg,bn", [(23, 256), (24, 192)])
@pytest.mark.parametrize("kind", ["i8", "i16", "i16res"])
def test_gemm_persistent_tiles_inside_wider_rows(G, cfg, bn, kind):
    # operands, residual and output as columns of wider rows, the last tile row ragged: rows past M are neither read into the result
    # nor stored, and nothing beside the output's own columns changes (buffers end with the last row's last column)
    import torch
    from paper_2101_01321_amd import binding as B
    rng = np.random.default_rng(bn)
    for M, N, K in [(1, bn, 128), (249, 2 * bn, 256), (257, bn, 384), (256 * 34 + 5, 2 * bn, 128)]:
        pa, pw, pc, pr = 48, 16, 32, 64                            # columns beside the problem's own
        A, W = (rng.integers(-127, 128, size=(n, K + p), dtype=np.int8) for n, p in ((M + 9, pa), (N, pw)))
        R = rng.integers(-127, 128, size=(M + 9, N + pr), dtype=np.int8) if kind == "i16res" else None
        bias = rng.integers(-50000, 50000, size=N, dtype=np.int32)
        mult = rng.integers(2 ** 29, 2 ** 30, size=N, dtype=np.int64).astype(np.int32)
        shifts = np.full(N, 40, np.int32)
        d = B.GemmDesc()
        for k, v in dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K + pa, ldw=K + pw, ldc=N + pc, ldr=N + pr, per_channel=1,
                         residual_dy=B.Dyadic(1717986918, 23), out_dtype=I8 if kind == "i8" else I16,
                         out_clamp=127 if kind == "i8" else 32767).items():
            setattr(d, k, v)
        dt = np.int8 if kind == "i8" else np.int16
        tC = G.to_dev(np.full((M + 9, N + pc), 77, dt))
        B.lib().ibert_gemm_config_override(cfg)
        try:
            G.say("persistent gemm inside wider rows cfg %d M=%d N=%d K=%d %s" % (cfg, M, N, K, kind))
            B.ibert_gemm_i8_requant(d, G.to_dev(A), G.to_dev(W), G.to_dev(bias), G.to_dev(mult), G.to_dev(shifts),
                                    None if R is None else G.to_dev(R), tC)
            torch.cuda.synchronize()
        finally:
            B.lib().ibert_gemm_config_override(-1)
        assert B.lib().ibert_last_kernel().decode().startswith(G.kernel_of(cfg))
        spec = GemmSpec(M, N, K, per_channel=1, dy=(1, 0), out_dtype=I8 if kind == "i8" else I32,
                        out_clamp=127 if kind == "i8" else 32767, res_dy=(1717986918, 23))
        dense = [np.ascontiguousarray(t) for t in (A[:M, :K], W[:, :K])]
        want = oracle.gemm_requant(spec, *dense, bias, mult, shifts, None if R is None else np.ascontiguousarray(R[:M, :N])).reshape(M, N)
        got = tC.cpu().numpy()
        _eq(got[:M, :N].astype(np.int64), want.astype(np.int64), "persistent gemm inside wider rows")
        assert np.all(got[M:] == 77) and np.all(got[:, N:] == 77), "wrote beside the output"


@pytest.mark.parametrize("M,N,K,kind,kernel", [(4096, 3072, 768, "gelu", "gemm_stream_kernel<256, 192, "),      # one tile a unit, longer loops
                                               (4096, 3072, 1024, "i8", "gemm_stream_kernel<256, 192, "),
                                               (4096, 2304, 768, "i8", "gemm_stream_kernel<256, 192, ")])
def test_gemm_persistent_tile_chosen(G, M, N, K, kind, kernel):
    _stream_case(G, -1, M, N, K, kind, 40, seed=M, kernel=kernel)


@pytest.mark.parametrize("M,N,K,kind,kernel", [(4096, 3072, 128, "gelu", "gemm_nt_mfma_kernel<256, 192, "),     # 256 tiles of one step
                                               (3072, 3072, 128, "gelu", "gemm_nt_mfma_kernel<256, 192, "),     # 192
                                               (16072, 768, 128, "gelu", "gemm_nt_mfma_kernel<256, 192, "),     # 252, uneven shares
                                               (16385, 768, 128, "gelu", "gemm_stream_kernel<256, "),           # a second round
                                               (4096, 3072, 256, "gelu", "gemm_stream_kernel<256, 192, "),      # two steps
                                               (16072, 768, 256, "gelu", "gemm_stream_kernel<256, 192, "),
                                               (16385, 768, 256, "gelu", "gemm_stream_kernel<256, "),
                                               (4096, 3072, 128, "i8", "gemm_stream_kernel<256, 192, "),        # without GELU: any K
                                               (4096, 3072, 768, "i8", "gemm_stream_kernel<256, 192, ")])
def test_gemm_tile_chosen_for_one_round(G, M, N, K, kind, kernel):
    # 256x192 tiles, at most one for every compute unit: persistent except with GELU on a single K step, where it was slower at every
    # number of tiles measured (192 to 256); the line does not depend on the tiles being exactly one for every unit
    _stream_case(G, -1, M, N, K, kind, 40, seed=M, kernel=kernel)


@pytest.mark.parametrize("cfg,bn", [(23, 256), (24, 192)])
@pytest.mark.parametrize("kind", ["i8", "i16", "i16res", "gelu"])
@pytest.mark.parametrize("constants", ["one multiplier", "no bias", "neither", "large shifts", "one slow column"])
def test_gemm_persistent_tiles_constants(G, cfg, bn, kind, constants):
    # constants that are filled in by hand where the caller has no array of them, in the first tile and after a change of tile
    # column; shifts of 44 to 62 (with GELU: the table address is no longer folded into the constants); a column of the second
    # tile column that sends all of it, and no other, through the 64-bit epilogue
    from paper_2101_01321_amd import binding as B
    M, N, K = 256 * 90 + 17, 3 * bn, 256
    rng = np.random.default_rng(cfg)
    A, W = (rng.integers(-127, 128, size=(n, K), dtype=np.int8) for n in (M, N))
    large = constants == "large shifts"
    bias = rng.integers(-2 ** 29, 2 ** 29, size=N, dtype=np.int32) if large else rng.integers(-50000, 50000, size=N, dtype=np.int32)
    mult = rng.integers(2 ** 29, 2 ** 30, size=N, dtype=np.int64).astype(np.int32)
    shifts = np.resize(np.array([44, 45, 46, 47, 50, 62], np.int32), N) if large else np.full(N, 37, np.int32)
    if constants == "one slow column":
        shifts[bn + 5] = 32
    bias = None if constants in ("no bias", "neither") else bias
    pc = 0 if constants in ("one multiplier", "neither") else 1
    dy = (1518500250, 37) if pc == 0 else (1, 0)
    R = rng.integers(-127, 128, size=(M, N), dtype=np.int8) if kind == "i16res" else None
    res_dy = (1717986918, 23)
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=pc, requant=dy, residual_dy=res_dy,
              out_dtype=I16 if kind[:3] == "i16" else I8, out_clamp=127 if kind == "i8" else 32767)
    arrays = (bias, mult if pc else None, shifts if pc else None)
    gp, op = B.ibert_gelu_params_from_scale(2.0 ** -6, 0.7), P.gelu_params(2.0 ** -6, 0.7)
    B.lib().ibert_gemm_config_override(cfg)
    try:
        G.say("persistent gemm cfg %d %s %s" % (cfg, kind, constants))
        got = G.gemm_gelu(kw, A, W, *arrays, gp, M * N)[0] if kind == "gelu" else G.gemm(kw, A, W, *arrays, R, out_elems=M * N)
    finally:
        B.lib().ibert_gemm_config_override(-1)
    assert B.lib().ibert_last_kernel().decode().startswith(G.kernel_of(cfg))
    spec = GemmSpec(M, N, K, per_channel=pc, dy=dy, out_dtype=I8 if kind == "i8" else I32,
                    out_clamp={"i8": 127, "gelu": gp.q_max}.get(kind, 32767), res_dy=res_dy)
    want = oracle.gemm_requant(spec, A, W, *arrays, R).reshape(-1)
    if kind == "gelu":
        want = oracle.gelu(want, op)
    assert len(np.unique(want)) > 20
    _eq(got.astype(np.int64), want.astype(np.int64), "persistent gemm, constants")


# (clamp, shift, residual): on both sides of the forms of the persistent tiles' epilogue -- INT8 with every shift from 40 on and the type's own
# clamp, or not; INT16 with the type's own clamp and a residual whose multiplier may lose its low eight bits, or not.  The last but one
# product is a tie, 127 * 2^30 / 2^31 = 63.5, that the low bits decide; residual shifts from 8 to 62
@pytest.mark.parametrize("cfg,bn", [(23, 256), (24, 192)])
@pytest.mark.parametrize("clamp,shift,res", [(127, 39, None), (127, 40, None), (100, 41, None), (127, 62, None), (32767, 35, (1352745605, 33)),
                                             (32767, 35, (-1352745605, 33)), (2000, 35, (1352745605, 33)), (32767, 36, (1073741823, 31)),
                                             (32767, 36, (1073741825, 31)), (32767, 34, (1717986918, 8)), (32767, 34, (1717986918, 23)),
                                             (32767, 34, (1717986918, 39)), (32767, 34, (1717986918, 62))])
def test_gemm_persistent_tiles_forms_of_the_epilogue(G, cfg, bn, clamp, shift, res):
    # ragged rows in the last tile, more than one tile for a workgroup; values in and beyond the clamp
    from paper_2101_01321_amd import binding as B
    M, N, K = 256 * 90 + 17, 3 * bn, 128
    rng = np.random.default_rng(shift + clamp)
    A, W = (rng.integers(-127, 128, size=(n, K), dtype=np.int8) for n in (M, N))
    bias = rng.integers(-50000, 50000, size=N, dtype=np.int32)
    mult = rng.integers(2 ** 30, 2 ** 31, size=N, dtype=np.int64).astype(np.int32)
    shifts = (shift + rng.integers(0, 2, size=N) * (shift < 62)).astype(np.int32)
    R = None if res is None else rng.integers(-127, 128, size=(M, N), dtype=np.int8)
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=1, residual_dy=res or (0, 0),
              out_dtype=I8 if res is None else I16, out_clamp=clamp)
    B.lib().ibert_gemm_config_override(cfg)
    try:
        G.say("persistent gemm cfg %d clamp %d shift %d residual %s" % (cfg, clamp, shift, res))
        got = G.gemm(kw, A, W, bias, mult, shifts, R, out_elems=M * N)
    finally:
        B.lib().ibert_gemm_config_override(-1)
    assert B.lib().ibert_last_kernel().decode().startswith(G.kernel_of(cfg))
    spec = GemmSpec(M, N, K, per_channel=1, out_dtype=I8 if res is None else I32, out_clamp=clamp, res_dy=res or (0, 0))
    _eq(got.astype(np.int64), oracle.gemm_requant(spec, A, W, bias, mult, shifts, R).reshape(-1).astype(np.int64), "persistent gemm, forms")


# Constants made once a tile, one to three steps before they are used; residuals whose product fits 32 bits and (a
# multiplier that rounds to 2^23, a shift of 8) does not, and 16-bit results that packing saturates or a smaller clamp does.
@pytest.mark.parametrize("cfg,bn", [(7, 128), (9, 96), (13, 192), (14, 128), (17, 96), (18, 96), (19, 128), (21, 96), (22, 128)])
@pytest.mark.parametrize("res,clamp", [(None, 32767), ((1717986816, 23), 32767), ((1717986816, 24), 30011), ((2147483647, 31), 32767), ((40000, 8), 32767),
                                       ((2147483392, 38), 32767)])
@pytest.mark.parametrize("K,shift", [(128, 33), (256, 40), (384, 62)])
def test_gemm_direct_tiles_16_bit_epilogue(G, cfg, bn, res, clamp, K, shift):
    from paper_2101_01321_amd import binding as B
    M, N = 256 + 77, 2 * bn
    rng = np.random.default_rng(cfg + K)
    A, W = (rng.integers(-128, 128, size=(n, K), dtype=np.int8) for n in (M, N))
    A[5], W[3] = -128, -128
    bias = rng.integers(-(1 << 29), 1 << 29, size=N, dtype=np.int32) if shift > 40 else rng.integers(-50000, 50000, size=N, dtype=np.int32)
    mult = (rng.integers(2 ** 28, 2 ** 31, size=N, dtype=np.int64) * rng.choice([-1, 1], size=N)).astype(np.int32)
    shifts = np.clip(shift + np.arange(N) % 3 - 1, 33, 62).astype(np.int32)
    R = None if res is None else rng.integers(-128, 128, size=(M, N), dtype=np.int8)
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=1, out_dtype=I16, out_clamp=clamp)
    B.lib().ibert_gemm_config_override(cfg)
    try:
        G.say("16-bit epilogue cfg %d K=%d shift=%d res=%s clamp=%d" % (cfg, K, shift, res, clamp))
        got = G.gemm(dict(kw, residual_dy=res or (1, 0)), A, W, bias, mult, shifts, R, out_elems=M * N)
    finally:
        B.lib().ibert_gemm_config_override(-1)
    assert B.lib().ibert_last_kernel().decode().startswith(G.kernel_of(cfg))
    spec = GemmSpec(M, N, K, per_channel=1, dy=(1, 0), out_dtype=I32, out_clamp=clamp, res_dy=res or (1, 0))
    _eq(got.astype(np.int64), oracle.gemm_requant(spec, A, W, bias, mult, shifts, R).reshape(-1).astype(np.int64), "16-bit epilogue")


# Output scales and the length of the table that they take: a usual one, one of 20 thousand entries, the largest that 256x256 (26624) and 256x192 (44544)
# have room for and one or two more; saturated from 127 S_out / S_in on
@pytest.mark.parametrize("bn,S,S_out,fits", [(256, 2.0 ** -6, 0.7, 1), (256, 2.0 ** -6, 2.5, 1), (256, 2.0 ** -6, 3.2685, 1), (256, 2.0 ** -6, 3.2688, 0),
                                             (192, 2.0 ** -6, 2.5, 1), (192, 2.0 ** -5, 10.9846, 1), (192, 2.0 ** -5, 10.9848, 0),
                                             (256, 2.0 ** -9, 0.06, 0), (192, 2.0 ** -9, 0.06, 0)])                   # no table at all
def test_gemm_gelu_table_larger_than_the_persistent_tiles_have_room_for(G, bn, S, S_out, fits):
    import torch
    from paper_2101_01321_amd import binding as B
    M, N, K = 256 * 90 - 7, 4 * bn, 128
    rng = np.random.default_rng(bn)
    A, W = (rng.integers(-127, 128, size=(n, K), dtype=np.int8) for n in (M, N))
    mult = rng.integers(2 ** 30, 2 ** 31, size=N, dtype=np.int64).astype(np.int32)
    shifts = np.full(N, 33, np.int32)
    gp, op = B.ibert_gelu_params_from_scale(S, S_out), P.gelu_params(S, S_out)
    kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=1)
    want = oracle.gelu(oracle.gemm_requant(GemmSpec(M, N, K, per_channel=1, out_dtype=I32, out_clamp=gp.q_max), A, W, None, mult, shifts, None).reshape(-1), op)
    word = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    for cfg in (-1, 23 if bn == 256 else 24):
        B.lib().ibert_gemm_config_override(cfg)
        B.ibert_gemm_epilogue_record(word)
        try:
            G.say("GELU with a large table, cfg %d bn %d S_out %g" % (cfg, bn, S_out))
            got = G.gemm_gelu(dict(kw, out_dtype=I8, out_clamp=5), A, W, None, mult, shifts, gp, M * N)[0]
        finally:
            B.ibert_gemm_epilogue_record(None)
            B.lib().ibert_gemm_config_override(-1)
        # chosen where its table fits; forced on one that does not, it computes GELU value by value
        assert B.lib().ibert_last_kernel().decode().startswith("gemm_stream_kernel") == bool(fits or cfg >= 0)
        if fits or cfg >= 0:
            assert int(word.item()) == (B.EPILOGUE_DIRECT_GELU_TABLE if fits else B.EPILOGUE_STAGED)
        _eq(got.astype(np.int64), want.astype(np.int64), "GELU with a large table")


@pytest.mark.parametrize("cfg,bn", [(23, 256), (24, 192)])
@pytest.mark.parametrize("kind", ["i8", "i16", "i16res", "gelu"])
@pytest.mark.parametrize("cols,shift", [(3, 40), (9, 40), (3, 30)])
def test_gemm_persistent_tiles_of_one_step(G, cfg, bn, kind, cols, shift):
    # K 128: a tile is a single K step, so the constants of the next tile's columns, requested behind it, have the epilogue alone to
    # arrive in.  More than four tiles for every workgroup, in another tile column each time (3 and 9 do not divide the 32
    # workgroups of an XCD), and constants that differ from column to column by far more than an output step.  The rows
    # repeat after 509 (which no tile edge does), so that the oracle's work stays small.
    import torch
    from paper_2101_01321_amd import binding as B
    P_, M, N, K = 509, 256 * (4 * 256 // cols + 8) + 3, cols * bn, 128
    rng = np.random.default_rng(cfg + cols + shift)
    A, W = (rng.integers(-127, 128, size=(n, K), dtype=np.int8) for n in (P_, N))
    R = rng.integers(-127, 128, size=(P_, N), dtype=np.int8) if kind == "i16res" else None
    col = np.arange(N) // bn                                       # (one sign and size of the constants per tile column)
    bias = ((col % 2 * 2 - 1) * (40000 + 30000 * col) + np.arange(N) % 97).astype(np.int32)
    mult = ((2 ** 28 + 2 ** 26 * col) * (1 - 2 * (col % 3 == 1))).astype(np.int32)
    shifts = (34 if kind == "gelu" and shift == 40 else shift) + (col % 3 if shift == 40 else 0 * col).astype(np.int32)
    res_dy = (1717986918, 23)
    rows = torch.arange(M, device=G.DEV) % P_
    tA, tW, tb, tm, ts = G.to_dev(A)[rows], G.to_dev(W), G.to_dev(bias), G.to_dev(mult), G.to_dev(shifts)
    d = B.GemmDesc()
    for k, v in dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=1,
                     residual_dy=B.Dyadic(*res_dy), out_dtype=I16 if kind[:3] == "i16" else I8,
                     out_clamp=127 if kind == "i8" else 32767).items():
        setattr(d, k, v)
    tC = torch.full((M, N), 77, dtype=torch.int16 if kind[:3] == "i16" else torch.int8, device=G.DEV)
    gp, op = B.ibert_gelu_params_from_scale(2.0 ** -6, 0.7), P.gelu_params(2.0 ** -6, 0.7)
    B.lib().ibert_gemm_config_override(cfg)
    try:
        G.say("persistent gemm of one step cfg %d M=%d N=%d %s shift=%d" % (cfg, M, N, kind, shift))
        if kind == "gelu":
            B.ibert_gemm_i8_gelu(d, tA, tW, tb, tm, ts, gp, tC, torch.empty(M * N, dtype=torch.int32, device=G.DEV))
        else:
            B.ibert_gemm_i8_requant(d, tA, tW, tb, tm, ts, None if R is None else G.to_dev(R)[rows], tC)
        torch.cuda.synchronize()
    finally:
        B.lib().ibert_gemm_config_override(-1)
    assert B.lib().ibert_last_kernel().decode().startswith(G.kernel_of(cfg))
    spec = GemmSpec(P_, N, K, per_channel=1, dy=(1, 0), out_dtype=I8 if kind == "i8" else I32,
                    out_clamp={"i8": 127, "gelu": gp.q_max}.get(kind, 32767), res_dy=res_dy)
    want = oracle.gemm_requant(spec, A, W, bias, mult, shifts, R).reshape(P_, N)
    if kind == "gelu":
        want = oracle.gelu(want.reshape(-1), op).reshape(P_, N)
    assert len(np.unique(want)) > 20
    bad = (tC != G.to_dev(want.astype(np.int16 if kind[:3] == "i16" else np.int8))[rows]).sum().item()
    assert bad == 0, "%d of %d values differ" % (bad, M * N)


@pytest.mark.parametrize("cfg,bm,bn", [(6, 256, 192), (7, 128, 128), (8, 256, 256), (9, 128, 96), (10, 256, 128), (11, 128, 96),
                                       (12, 128, 128), (13, 256, 192), (14, 256, 128), (16, 256, 256), (17, 64, 96), (18, 64, 96),
                                       (19, 64, 128), (20, 128, 96), (21, 128, 96), (22, 128, 128)])
def test_gemm_direct_to_lds_ragged_rows(G, cfg, bm, bn):
    # direct-to-LDS tiles whose last tile row is not whole: one row, one less and one more than a tile, several tiles and some
    kinds = ["i8", "i16res"] + (["gelu"] if cfg in (6, 7, 8, 9, 10, 13, 14, 16) else [])
    for M, N, K in [(1, bn, 128), (bm - 1, 2 * bn, 256), (bm + 1, bn, 512), (3 * bm + 37, 2 * bn, 384)]:
        for kind in kinds:
            _stream_case(G, cfg, M, N, K, kind, 40, seed=M + N + K)


@pytest.mark.parametrize("cfg,bm,bn", [(21, 128, 96), (22, 128, 128)])
def test_gemm_gelu_on_tiles_with_loaders(G, cfg, bm, bn):
    # GELU where four wavefronts only request tiles: one K step (fewer than stages) to more steps than stages, rows at and off a tile
    # edge, one and several tiles a unit; the table and (shift 30) the 64-bit form
    for M, N, K, shift in [(1, bn, 128, 40), (bm - 1, 2 * bn, 256, 40), (bm + 1, bn, 512, 40), (3 * bm + 37, 24 * bn, 384, 40),
                           (33 * bm + 5, 9 * bn, 128, 40), (bm + 9, 3 * bn, 640, 30)]:
        _stream_case(G, cfg, M, N, K, "gelu", shift, seed=M + N + K)


@pytest.mark.parametrize("kind,cfg,bm,bn", [(kind, *t) for kind in ("i8", "i16res", "gelu") for t in
                                            [(7, 128, 128), (9, 128, 96), (13, 256, 192), (14, 256, 128), (17, 64, 96), (18, 64, 96),
                                             (19, 64, 128), (21, 128, 96), (22, 128, 128)] if kind != "gelu" or t[0] not in (17, 18, 19)])
@pytest.mark.parametrize("constants", ["one multiplier", "no bias", "neither"])
@pytest.mark.parametrize("shift", [37, 30])
def test_gemm_direct_to_lds_constants_filled_in_by_hand(G, kind, cfg, bm, bn, constants, shift):
    # without an array of them the constants of a tile's columns are written to LDS by the wavefronts themselves; each then reads all of
    # them to choose the form of the epilogue (shift 37 register-direct, 30 through LDS with barriers): one K step and several, the
    # last tile row cut
    import torch
    from paper_2101_01321_amd import binding as B
    gp, op = B.ibert_gelu_params_from_scale(2.0 ** -6, 0.7), P.gelu_params(2.0 ** -6, 0.7)
    pc, res_dy, dy = int(constants == "no bias"), (1717986918, 23), (1518500250 >> (37 - shift), shift)
    word = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    for M, N, K in [(bm + 3, bn, 128), (9 * bm + 37, 3 * bn, 640)]:
        rng = np.random.default_rng(cfg + M + shift)
        A, W = (rng.integers(-127, 128, size=(n, K), dtype=np.int8) for n in (M, N))
        bias = rng.integers(-50000, 50000, size=N, dtype=np.int32) if constants == "one multiplier" else None
        mult, shifts = (rng.integers(2 ** 29, 2 ** 30, size=N, dtype=np.int32) >> (37 - shift), np.full(N, shift, np.int32)) if pc else (None, None)
        R = rng.integers(-127, 128, size=(M, N), dtype=np.int8) if kind == "i16res" else None
        kw = dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=K, ldc=N, ldr=N, per_channel=pc, requant=dy, residual_dy=res_dy,
                  out_dtype=I16 if kind == "i16res" else I8, out_clamp=127 if kind == "i8" else 32767)
        B.lib().ibert_gemm_config_override(cfg)
        B.ibert_gemm_epilogue_record(word)
        try:
            G.say("constants by hand cfg %d %s %s shift=%d M=%d N=%d K=%d" % (cfg, kind, constants, shift, M, N, K))
            got = G.gemm_gelu(kw, A, W, bias, mult, shifts, gp, M * N)[0] if kind == "gelu" else G.gemm(kw, A, W, bias, mult, shifts, R, out_elems=M * N)
        finally:
            B.ibert_gemm_epilogue_record(None)
            B.lib().ibert_gemm_config_override(-1)
        assert B.lib().ibert_last_kernel().decode().startswith(G.kernel_of(cfg))
        assert (int(word.item()) == B.EPILOGUE_STAGED) == (shift < 33)
        spec = GemmSpec(M, N, K, per_channel=pc, dy=dy, out_dtype=I8 if kind == "i8" else I32,
                        out_clamp={"i8": 127, "gelu": gp.q_max}.get(kind, 32767), res_dy=res_dy)
        want = oracle.gemm_requant(spec, A, W, bias, mult, shifts, R).reshape(-1)
        if kind == "gelu":
            want = oracle.gelu(want, op)
        assert len(np.unique(want)) > 20
        _eq(got.astype(np.int64), want.astype(np.int64), "constants by hand")


INT8_TILES = [(15, 32, 32), (3, 64, 64), (2, 128, 128), (4, 64, 128), (7, 128, 128), (9, 128, 96), (13, 256, 192), (14, 256, 128), (17, 64, 96),
              (18, 64, 96), (19, 64, 128), (21, 128, 96), (22, 128, 128), (-1, 128, 64), (-1, 128, 128)]        # the last two: W as [K, N]


@pytest.mark.parametrize("kind,cfg,bm,bn", [(kind, *t) for kind in ("plain", "residual", "gelu") for t in INT8_TILES
                                            if kind != "gelu" or t[0] in (15, 3, 7, 9, 13, 14, 21, 22)])
def test_gemm_int8_tiles_leave_in_every_way(G, kind, cfg, bm, bn):
    # INT8 outputs leave lane-transposed, through LDS (with a residual) or by the lanes' own 4-byte stores, by the alignment of the
    # output's rows; as columns of wider rows, so that whatever is written beside them shows.  Shift 45: GELU's table is not folded
    import torch
    from paper_2101_01321_amd import binding as B
    tw, K = int(cfg < 0), 256
    gp, op = B.ibert_gelu_params_from_scale(2.0 ** -6, 0.7), P.gelu_params(2.0 ** -6, 0.7)
    for M, beside, at, shift in [(2 * bm, 16, 0, 40), (2 * bm, 4, 0, 40), (2 * bm, 16, 4, 40), (2 * bm, 1, 0, 40), (2 * bm, 16, 0, 30), (2 * bm + 5, 16, 0, 40)] + \
                                ([(2 * bm, 16, 0, 45), (2 * bm, 4, 0, 45)] if kind == "gelu" else []):
        N = 2 * bn if not tw else bn
        rng = np.random.default_rng(M + beside + at + shift)
        A = rng.integers(-127, 128, size=(M, K), dtype=np.int8)
        W = rng.integers(-127, 128, size=(K, N) if tw else (N, K), dtype=np.int8)
        bias = rng.integers(-50000, 50000, size=N, dtype=np.int32)
        mult = rng.integers(2 ** 29, 2 ** 30, size=N, dtype=np.int32)
        mult, shifts = {30: mult >> 10, 40: mult, 45: mult + 2 ** 30 - 1}[shift], np.full(N, shift, np.int32)
        R = rng.integers(-127, 128, size=(M, N), dtype=np.int8) if kind == "residual" else None
        d = B.GemmDesc()
        for k, v in dict(M=M, N=N, K=K, batch_outer=1, batch_inner=1, lda=K, ldw=N if tw else K, ldc=N + beside, ldr=N, trans_w=tw, per_channel=1,
                         residual_dy=B.Dyadic(1717986918, 31), out_dtype=I8, out_clamp=127).items():
            setattr(d, k, v)
        tC = torch.full((at + (M + 1) * (N + beside),), 77, dtype=torch.int8, device=G.DEV)
        dev = [G.to_dev(t) for t in (A, W, bias, mult, shifts)]
        B.lib().ibert_gemm_config_override(cfg)
        try:
            G.say("INT8 tiles leave cfg %d %s M=%d N=%d +%d @%d shift=%d" % (cfg, kind, M, N, beside, at, shift))
            if kind == "gelu":
                B.ibert_gemm_i8_gelu(d, *dev, gp, tC[at:], torch.empty((M, N), dtype=torch.int32, device=G.DEV))
            else:
                B.ibert_gemm_i8_requant(d, *dev, None if R is None else G.to_dev(R), tC[at:])
            torch.cuda.synchronize()
        finally:
            B.lib().ibert_gemm_config_override(-1)
        assert B.lib().ibert_last_kernel().decode().startswith("gemm_nt_mfma_kernel<%d, %d, " % (bm, bn))
        spec = GemmSpec(M, N, K, per_channel=1, dy=(1, 0), out_dtype=I32 if kind == "gelu" else I8,
                        out_clamp=gp.q_max if kind == "gelu" else 127, res_dy=(1717986918, 31))
        want = oracle.gemm_requant(spec, A, np.ascontiguousarray(W.T) if tw else W, bias, mult, shifts, R).reshape(M, N)
        if kind == "gelu":
            want = oracle.gelu(want.reshape(-1), op).reshape(M, N)
        got = tC.cpu().numpy()
        rows = got[at:].reshape(M + 1, N + beside)
        _eq(rows[:M, :N].astype(np.int64), want.astype(np.int64), "INT8 tiles leave")
        assert np.all(got[:at] == 77) and np.all(rows[M:] == 77) and np.all(rows[:, N:] == 77), "wrote beside the output"


@pytest.mark.parametrize("cfg,bn,lda,M", [(7, 128, 1 << 22, 1025), (9, 96, 1 << 22, 1030), (13, 192, 1 << 22, 1025), (14, 128, 1 << 22, 1033),
                                          (17, 96, 1 << 22, 1025), (21, 96, 1 << 22, 1025), (22, 128, 1 << 22, 1025),
                                          (23, 256, 1 << 19, 8193), (24, 192, 1 << 19, 8198)])
def test_gemm_rows_four_gigabytes_apart(G, cfg, bn, lda, M):
    # rows of A that lie more than 2^32 bytes behind a tile's first row: the distance to the last row, which a ragged tile's
    # addresses are clamped by, does not wrap around (M - 1 rows are 2^32 bytes, or a few rows more)
    import torch
    from paper_2101_01321_amd import binding as B
    N, K = 2 * bn, 256
    rng = np.random.default_rng(cfg)
    A, W = (rng.integers(-127, 128, size=(n, K), dtype=np.int8) for n in (M, N))
    bias, mult, shift = np.arange(N, dtype=np.int32), np.full(N, 2 ** 30, np.int32), np.full(N, 41, np.int32)
    tA = torch.empty(M * lda, dtype=torch.int8, device=G.DEV)
    tA.view(M, lda)[:, :K] = G.to_dev(A)
    tC = torch.full((M, N), 77, dtype=torch.int8, device=G.DEV)
    d = B.GemmDesc()
    d.M, d.N, d.K, d.batch_outer, d.batch_inner = M, N, K, 1, 1
    d.lda, d.ldw, d.ldc, d.ldr = lda, K, N, N
    d.per_channel, d.out_dtype, d.out_clamp = 1, I8, 127
    B.lib().ibert_gemm_config_override(cfg)
    try:
        G.say("gemm rows far apart cfg %d M=%d lda=%d" % (cfg, M, lda))
        B.ibert_gemm_i8_requant(d, tA, G.to_dev(W), G.to_dev(bias), G.to_dev(mult), G.to_dev(shift), None, tC)
        torch.cuda.synchronize()
    finally:
        B.lib().ibert_gemm_config_override(-1)
    assert B.lib().ibert_last_kernel().decode().startswith(G.kernel_of(cfg))
    spec = GemmSpec(M, N, K, per_channel=1, dy=(1, 0), out_dtype=I8, out_clamp=127)
    _eq(tC.cpu().numpy(), oracle.gemm_requant(spec, A, W, bias, mult, shift, None).reshape(M, N), "gemm, rows far apart")


@pytest.mark.parametrize("cfg,bm,bn", [(25, 16, 16), (26, 16, 32), (27, 32, 32), (28, 32, 64), (29, 32, 96), (30, 64, 64)])
@pytest.mark.parametrize("kind", ["i8", "i16", "i16res", "gelu"])
def test_gemm_few_rows(G, cfg, bm, bn, kind):
    # K from one step (fewer than wavefronts) to more steps than are in flight at once, where a stage is used again; rows at, one
    # past and off a tile edge; tile columns that do and do not divide by the XCDs; both epilogue forms
    for M, N, K, shift in [(1, bn, 128, 40), (bm, 8 * bn, 640, 40), (bm + 1, 3 * bn, 1024, 40), (3 * bm + 7, 12 * bn, 1152, 40),
                           (2 * bm - 1, 2 * bn, 5248, 40), (bm + 3, 5 * bn, 256, 30), (17 * bm, 9 * bn, 384, 40)]:
        _stream_case(G, cfg, M, N, K, kind, shift, seed=M + N + K)


# ------------------------------------------------------------------------------------------- Softmax, rows that start anywhere
@pytest.mark.parametrize("cols", [1, 3, 4, 5, 7, 61, 62, 63, 65, 127, 129, 251, 257, 511, 513, 1023, 1025, 2045])
@pytest.mark.parametrize("k,od", [(7, I8), (24, I32)])
def test_softmax_rows_at_any_address(G, cols, k, od):
    # the last chunk of a row is moved back over the one before it: its columns count once, nothing outside the row is written,
    # and a mask that ends before, inside and after the columns that are read twice is kept
    from paper_2101_01321_amd import binding as B
    rows = 19
    S = 2.0 ** -6
    x, _ = synth.softmax_logits(rows, cols, scale=S)
    x[0, :], x[1, :] = 5, -2 ** 31
    x[2, -1], x[3, 0] = x.max() + 1, x.max() + 1
    sp, op = B.ibert_softmax_params_from_scale(S, cols, k, od), P.softmax_params(S, k, od)
    for ldx, ldy, xo, yo in [(cols, cols, 0, 0), (cols + 1, cols + 2, 1, 1), (cols + 4 - cols % 4, cols + 4 - cols % 4, 0, 0)]:
        G.say("softmax cols=%d ldx=%d ldy=%d out=%d" % (cols, ldx, ldy, od))
        got = G.softmax(x, sp, ldx=ldx, ldy=ldy, x_off=xo, y_off=yo)
        _eq(got[:, :cols], oracle.softmax(x, op), "softmax cols=%d" % cols)
        assert np.all(got[:, cols:] == 77)
        lens = np.array([max(1, cols - 5), max(1, cols - 2), cols, 1] * 5, np.int32)[:rows]
        masked = np.where(np.arange(cols)[None, :] < lens[:, None], x, np.int32(-2 ** 31)).astype(np.int32)
        got = G.softmax(x, sp, ldx=ldx, ldy=ldy, x_off=xo, y_off=yo, key_lens=lens)
        _eq(got[:, :cols], oracle.softmax(masked, op), "masked softmax cols=%d" % cols)
        assert np.all(got[:, cols:] == 77)


# ------------------------------------------------------------------------------------------- weights read ahead
@pytest.mark.parametrize("hidden,heads,ffn,seq,batch", [(256, 4, 1152, 61, 2), (256, 4, 128, 17, 1), (384, 6, 640, 200, 9),
                                                        (768, 12, 3072, 77, 3), (256, 4, 1024, 300, 40)])
def test_encoder_that_reads_weights_ahead(G, hidden, heads, ffn, seq, batch):
    # the attention of each layer also reads the weights of the MatMuls that follow, up to the next layer's first (the last layer has
    # none to follow): three layers of sizes that every kind of tile serves, with and without the separate GELU that leaves it out,
    # a graph of it replayed, and the oracle's layers on the last sequence
    import torch
    from paper_2101_01321_amd import binding as B
    cfg = synth.EncoderConfig("ahead", hidden, heads, ffn, seq, batch, 3)
    x_q, S_x, _ = synth.input_activations(cfg)
    model = G.DeviceModel(cfg, S_x)
    x = G.to_dev(x_q)
    G.say("encoder that reads ahead H=%d F=%d L=%d B=%d" % (hidden, ffn, seq, batch))
    y = model.forward(x)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    model.set_route(B.ROUTE_SEPARATE_GELU)
    other = model.forward(x)
    torch.cuda.synchronize()
    _eq(got, other.cpu().numpy(), "route that does not read ahead")
    model.set_route(0)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        yg = model.forward(x)
    for _ in range(3):
        yg.zero_()
        graph.replay()
        torch.cuda.synchronize()
        _eq(yg.cpu().numpy(), got, "replay")
    cur = x_q[(batch - 1) * seq:]
    for l in range(3):
        w, q = P.layer_params(synth.layer_raw(cfg, l), model.scales[l], hidden, heads)
        cur = oracle.encoder_layer(w, q, cur, 1, seq, hidden, heads, ffn)
    _eq(got[(batch - 1) * seq:], cur, "the oracle's layers")


def test_encoder_reads_ahead_weights_at_odd_addresses(G):
    # the plan of what to read ahead is the first layer's; weights of a later layer may lie at any byte
    import torch
    cfg = synth.EncoderConfig("odd", 256, 4, 640, 61, 3, 3)
    x_q, S_x, _ = synth.input_activations(cfg)
    model = G.DeviceModel(cfg, S_x)
    x = G.to_dev(x_q)
    G.say("encoder that reads ahead, odd weights")
    want = model.forward(x)
    moved = []
    for l, name, off in ((1, "w_o", 3), (1, "w_2", 1), (2, "w_qkv", 7), (2, "w_1", 16)):
        w = model.layers[l].tensors[name].reshape(-1)
        t = torch.zeros(w.numel() + 64, dtype=torch.int8, device=w.device)
        t[off:off + w.numel()] = w
        setattr(model.weights[l], name, t.data_ptr() + off)
        moved.append(t)
    got = model.forward(x)
    torch.cuda.synchronize()
    _eq(got.cpu().numpy(), want.cpu().numpy(), "weights at odd addresses")


# ------------------------------------------------------------------------------------------- QKV projection and attention as one kernel
def _qkv_layer(G, heads, B_, L, lens=None, edit=None):
    """One layer of 64 x heads channels: weights and quantization (edit: changes made to both sides), input, masks."""
    import torch
    from paper_2101_01321_amd import binding as B
    cfg = synth.EncoderConfig("qkv", 64 * heads, heads, 128, L, B_, 1)
    x_q, S_x, _ = synth.input_activations(cfg)
    model = G.DeviceModel(cfg, S_x)
    w, q = P.layer_params(synth.layer_raw(cfg, 0), model.scales[0], cfg.hidden, heads)
    if edit:
        edit(model, w, q)
    x = G.to_dev(x_q)
    key_lens = None if lens is None else G.to_dev(np.asarray(lens, np.int32))

    def run(tile):
        B.lib().ibert_qkv_attention_override(tile)
        try:
            model.ws.fill_(0x55)
            y = model.layer_forward(0, x, key_lens)
            torch.cuda.synchronize()
            # a layer call that stores scores (any length but 128 and 256) runs the steps apart; the encoder call of one layer stores no qkv
            model.ws.fill_(0x55)
            z = model.forward(x, key_lens)
            torch.cuda.synchronize()
            got = model.intermediates(r_half=True)
            assert (got["qkv"] == 0x55).all(), "steps 1 to 4 did not run as one kernel"
            return y.cpu().numpy(), z.cpu().numpy(), got
        finally:
            B.lib().ibert_qkv_attention_override(-1)
    return cfg, x_q, w, q, run


def _qkv_tiles(L):
    r = -(-L // 32)
    if L > 128:
        return [16313, 16412] if L <= 192 else [16412]
    return [8012 + 100 * r, 8014 + 100 * r, 8412, 8414] + ([8222, 8442] if L <= 32 else []) + ([8422] if L <= 64 else [])


# rows at, before and behind the ends of the tiles; groups that are not full; one K step, an odd number of them, more than there are stages
@pytest.mark.parametrize("heads", [2, 6, 10])
@pytest.mark.parametrize("L", [1, 16, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 192, 193, 255, 256])
def test_qkv_attention_every_tile(G, heads, L):
    import torch
    B_ = 5 if L <= 128 else 2
    cfg, x_q, w, q, run = _qkv_layer(G, heads, B_, L)
    want, inter = oracle.encoder_layer(w, q, x_q, B_, L, cfg.hidden, heads, cfg.ffn, dump=True)
    for tile in _qkv_tiles(L):
        G.say("qkv + attention, tile %d, heads=%d L=%d" % (tile, heads, L))
        y, z, got = run(tile)
        _eq(got["ctx"], inter["ctx"], "tile %d ctx" % tile)
        _eq(y, want, "tile %d layer" % tile)
        _eq(z, want, "tile %d encoder" % tile)


@pytest.mark.parametrize("tile,L", [(8112, 20), (8442, 30), (8222, 32), (8422, 61), (8312, 70), (8412, 128), (8414, 100), (16313, 150), (16412, 251)])
def test_qkv_attention_masked(G, tile, L):
    lens = [L, 1, (L + 1) // 2, max(1, L - 1), min(L, 64)]
    cfg, x_q, w, q, run = _qkv_layer(G, 4, 5, L, lens)
    want = oracle.encoder_layer(w, q, x_q, 5, L, cfg.hidden, 4, cfg.ffn, key_lens=np.asarray(lens, np.int32))
    G.say("qkv + attention, masked, tile %d L=%d" % (tile, L))
    y, z, _ = run(tile)
    _eq(z, want, "masked, tile %d" % tile)
    _eq(y, want, "masked, tile %d, one layer" % tile)


def test_qkv_attention_stores_qkv_for_a_single_layer(G):
    # a layer call with a workspace leaves Q, K and V there, as the MatMul by itself stores them
    from paper_2101_01321_amd import binding as B
    import torch
    cfg = synth.EncoderConfig("qkv", 256, 4, 128, 128, 3, 1)
    x_q, S_x, _ = synth.input_activations(cfg)
    model = G.DeviceModel(cfg, S_x)
    w, q = P.layer_params(synth.layer_raw(cfg, 0), model.scales[0], cfg.hidden, cfg.heads)
    want, inter = oracle.encoder_layer(w, q, x_q, 3, 128, 256, 4, 128, dump=True)
    for tile in (8412, 8414, 16412):
        B.lib().ibert_qkv_attention_override(tile)
        try:
            model.ws.fill_(0x55)
            G.say("qkv stored, tile %d" % tile)
            model.layer_forward(0, G.to_dev(x_q))
            torch.cuda.synchronize()
        finally:
            B.lib().ibert_qkv_attention_override(-1)
        got = model.intermediates(r_half=True)
        _eq(got["qkv"], inter["qkv"], "tile %d qkv" % tile)
        _eq(got["ctx"], inter["ctx"], "tile %d ctx" % tile)


# which arithmetic a matrix's channels take: every shift at least 40, at least 33, any; biases at the ends of 2^30 and beyond; sums that saturate
@pytest.mark.parametrize("shift,mult,bias", [(40, 1 << 30, 0), (47, 2147483647, (1 << 30) - 1), (44, -2147483647, -(1 << 30)), (39, 1 << 30, 5), (33, 3, 1 << 20),
                                             (32, 1, 1000), (0, 1, -3), (62, 2147483647, 1 << 29), (45, 2147483647, 1 << 30), (40, 2147483647, -(1 << 30) - 1)])
@pytest.mark.parametrize("tile", [8212, 8414])
def test_qkv_attention_any_constants(G, shift, mult, bias, tile):
    import torch

    def edit(model, w, q):
        # the constants go to one matrix (K) whole and to single channels of the others' halves; the device's arrays are changed in place
        H = 256
        for name, value in (("m_qkv", mult), ("s_qkv", shift), ("b_qkv", bias)):
            host = w[name]
            host[H:2 * H] = value
            host[5] = value
            t = model.layers[0].tensors[name]
            t.copy_(torch.from_numpy(np.ascontiguousarray(host)).to(t.device))
    cfg, x_q, w, q, run = _qkv_layer(G, 4, 3, 61, edit=edit)
    want, inter = oracle.encoder_layer(w, q, x_q, 3, 61, 256, 4, cfg.ffn, dump=True)
    G.say("qkv + attention, shift %d mult %d bias %d tile %d" % (shift, mult, bias, tile))
    y, z, _ = run(tile)
    _eq(z, want, "shift %d mult %d bias %d" % (shift, mult, bias))


def _set_constants(kind):
    """An edit for _qkv_layer: the constants of a kind, on both sides."""
    import torch
    import qkv_constants as QC

    def edit(model, w, q):
        QC.deal(w, model.cfg.hidden, kind)
        for name in ("m_qkv", "s_qkv", "b_qkv"):
            t = model.layers[0].tensors[name]
            t.copy_(torch.from_numpy(np.ascontiguousarray(w[name], dtype=np.int32)).to(t.device))
    return edit


# (128 tokens: a layer call with a workspace stores what the kernel made of the constants, in Q, K and V)
@pytest.mark.parametrize("kind", ["tall", "fast", "slow", "bias", "mixed"])
@pytest.mark.parametrize("tile", [8412, 8414, 16313, 16412])
def test_qkv_attention_constants_in_q_k_and_v(G, kind, tile):
    import torch
    from paper_2101_01321_amd import binding as B
    import qkv_constants as QC
    heads, B_, L = 4, 2, 128
    cfg, x_q, S_x, w, q = QC.layer(heads, B_, L)
    model = G.DeviceModel(cfg, S_x)
    _set_constants(kind)(model, w, q)
    want, inter = oracle.encoder_layer(w, q, x_q, B_, L, cfg.hidden, heads, cfg.ffn, dump=True)
    G.say("qkv + attention, %s constants, tile %d" % (kind, tile))
    B.lib().ibert_qkv_attention_override(tile)
    try:
        y = model.layer_forward(0, G.to_dev(x_q))
        torch.cuda.synchronize()
    finally:
        B.lib().ibert_qkv_attention_override(-1)
    got = model.intermediates(r_half=True)
    for name in ("qkv", "ctx"):
        _eq(got[name], inter[name], "%s, tile %d, %s" % (kind, tile, name))
    _eq(y.cpu().numpy(), want, "%s, tile %d" % (kind, tile))


# (several sequences to a workgroup, rows of half a key block, tiles that no layer call stores Q, K and V of: in V, which the context shows)
@pytest.mark.parametrize("kind", ["values tall", "values fast", "values slow", "values bias"])
@pytest.mark.parametrize("tile,L", [(8112, 29), (8114, 32), (8212, 61), (8214, 64), (8222, 32), (8442, 30), (8422, 61), (8312, 96), (8314, 70)])
def test_qkv_attention_constants_in_v(G, kind, tile, L):
    cfg, x_q, w, q, run = _qkv_layer(G, 4, 5, L, edit=_set_constants(kind))
    want, inter = oracle.encoder_layer(w, q, x_q, 5, L, cfg.hidden, 4, cfg.ffn, dump=True)
    G.say("qkv + attention, %s constants, tile %d L=%d" % (kind, tile, L))
    y, z, got = run(tile)
    _eq(got["ctx"], inter["ctx"], "%s, tile %d, ctx" % (kind, tile))
    _eq(z, want, "%s, tile %d" % (kind, tile))


def _scores(sdy, S, cdy):
    """An edit for _qkv_layer: the attention's constants, on both sides."""
    from paper_2101_01321_amd import binding as B

    def edit(model, w, q):
        q.scores_m, q.scores_s = sdy
        q.ctx_m, q.ctx_s = cdy
        q.softmax = P.softmax_params(S, 7)
        for quant in (model.layers[0].quant, model.quant[0]):
            quant.scores_dy, quant.ctx_dy = B.Dyadic(*sdy), B.Dyadic(*cdy)
            quant.softmax = B.ibert_softmax_params_from_scale(S, model.cfg.seq, 7)
    return edit


def _kernels(run):
    """(step, kernel) of what run() launches in layers."""
    from paper_2101_01321_amd import binding as B
    B.ibert_profile_begin(64)
    try:
        run()
    finally:
        records = B.ibert_profile_end(64)
    return [(r[0], r[4]) for r in records]


# every instantiation of the form for scores shifts from 34 on, and beside it the other one; context shifts on both sides of 32; masks past both ends of a sequence
@pytest.mark.parametrize("tile,L", [(8112, 20), (8212, 64), (8312, 70), (8412, 128), (8114, 32), (8214, 33), (8314, 96), (8414, 100), (8222, 32), (8422, 61), (8442, 30),
                                    (16313, 150), (16412, 251)])
@pytest.mark.parametrize("sdy,form", [((1518500250, 36), 4), ((1187698534, 34), 4), ((1187698534, 33), 3), ((1187698534, 28), 3)])
def test_qkv_attention_both_forms(G, tile, L, sdy, form):
    import torch
    from paper_2101_01321_amd import binding as B
    B_, heads, S = 5 if L <= 128 else 2, 2, 2.0 ** -6
    for cdy in ((1073741824, 37), (8388608, 30)):
        assert _attention_form(sdy, B.ibert_softmax_params_from_scale(S, L, 7), cdy, B_ * heads * -(-L // 64)) == form
        cfg, x_q, w, q, run = _qkv_layer(G, heads, B_, L, edit=_scores(sdy, S, cdy))
        want, inter = oracle.encoder_layer(w, q, x_q, B_, L, cfg.hidden, heads, cfg.ffn, dump=True)
        G.say("qkv + attention, form %d, tile %d L=%d s=%s c=%s" % (form, tile, L, sdy, cdy))
        out = []
        ran = [k for step, k in _kernels(lambda: out.extend(run(tile))) if step == 1 and k.startswith("qkv_attention")]
        digits = str(tile)
        name = "qkv_attention_kernel<%s, %s, %s, %d, %s>" % (digits[:-3], digits[-3], digits[-2], form, digits[-1])
        assert ran and all(k == name for k in ran), (ran, name)
        _eq(out[2]["ctx"], inter["ctx"], "form %d, tile %d, ctx" % (form, tile))
        _eq(out[1], want, "form %d, tile %d" % (form, tile))
        lens = [L, 1, (L + 1) // 2, max(1, L - 1), min(L, 64)][:B_]
        given = [L + 7, 0, (L + 1) // 2, max(1, L - 1), min(L, 64)][:B_]       # (taken as the nearest length there is)
        cfg, x_q, w, q, run = _qkv_layer(G, heads, B_, L, given, edit=_scores(sdy, S, cdy))
        want = oracle.encoder_layer(w, q, x_q, B_, L, cfg.hidden, heads, cfg.ffn, key_lens=np.asarray(lens, np.int32))
        _eq(run(tile)[1], want, "masked, form %d, tile %d" % (form, tile))


# constants that the attention has no table of the exponent for: the steps run apart, also where a tile is asked for
@pytest.mark.parametrize("S,sdy,form", [(2.0 ** -8, (1518500250, 36), 1), (2.0 ** -8, (1187698534, 28), 2), (2.0 ** -6, (-1518500250, 36), 0), (2.0 ** -6, (1518500250, 46), 0)])
@pytest.mark.parametrize("tile,L", [(8412, 128), (8222, 30), (16412, 200)])
def test_qkv_attention_without_a_table_runs_apart(G, S, sdy, form, tile, L):
    import torch
    from paper_2101_01321_amd import binding as B
    import qkv_constants as QC
    B_, heads, cdy = 2, 4, (1073741824, 37)
    assert _attention_form(sdy, B.ibert_softmax_params_from_scale(S, L, 7), cdy, B_ * heads * -(-L // 64)) == form
    cfg, x_q, S_x, w, q = QC.layer(heads, B_, L)
    model = G.DeviceModel(cfg, S_x)
    _scores(sdy, S, cdy)(model, w, q)
    want, inter = oracle.encoder_layer(w, q, x_q, B_, L, cfg.hidden, heads, cfg.ffn, dump=True)
    x = G.to_dev(x_q)
    G.say("qkv and attention apart, form %d, tile %d L=%d" % (form, tile, L))
    B.lib().ibert_qkv_attention_override(tile)
    try:
        model.ws.fill_(0x55)
        out = []
        kernels = _kernels(lambda: out.append(model.forward(x)))
        torch.cuda.synchronize()
    finally:
        B.lib().ibert_qkv_attention_override(-1)
    assert not any(k.startswith("qkv_attention") for _, k in kernels), kernels
    got = model.intermediates(r_half=True)
    _eq(got["qkv"], inter["qkv"], "form %d, qkv" % form)
    _eq(got["ctx"], inter["ctx"], "form %d, ctx" % form)
    _eq(out[0].cpu().numpy(), want, "form %d" % form)
