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


# ------------------------------------------------------------------------------------------- attention, any length
@pytest.mark.parametrize("L", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 191, 192, 193, 251, 255, 257, 319, 321, 384, 385, 447, 449,
                               511, 512])
@pytest.mark.parametrize("S,k,sdy", [(2.0 ** -6, 7, (1518500250, 36)), (2.0 ** -6, 7, (1187698534, 28)),
                                     (2.0 ** -4, 5, (1518500250, 36)),        # q_ln2 = 11, fewer output bits
                                     (2.0 ** -6, 7, (-1518500250, 36))])      # a negative multiplier: the general form
def test_attention_any_length(G, L, S, k, sdy):
    from paper_2101_01321_amd import binding as B
    B_, nh = 2, 3
    H, cdy = 64 * nh, (1073741824, 37 if k == 7 else 35)
    qkv = _qkv(B_, L, H, L)
    sp, op = B.ibert_softmax_params_from_scale(S, L, k), P.softmax_params(S, k)
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


def test_layer_of_any_length_keeps_scores_and_probabilities(G):
    # a single layer call leaves every intermediate in the workspace for lengths that are no multiple of 128
    for seq in (33, 100, 131):
        _layer_case(G, synth.EncoderConfig("len%d" % seq, 192, 3, 320, seq, 2, 1))
