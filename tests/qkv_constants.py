"""Requantization constants for the QKV projection at which its results lie around a rounding or at both ends of the clamp, by the arithmetic that
they leave a kernel: every shift at least 40 ("tall"), at least 33 ("fast"), any ("slow"), biases from 2^30 on ("bias").  Sums of products are below 2^23."""
import numpy as np

from oracle import params as P
from paper_2101_01321_amd import synth

B30, TOP = 1 << 30, (1 << 31) - 1
# (shift, multiplier, bias, do the results of a channel vary?)
TALL = [(40, 129536, B30 - 1, True), (40, 129536, -B30, True), (40, -129536, -B30, True), (40, -129536, B30 - 1, True),     # around +-126.5
        (62, TOP, B30 - 1, True), (62, -TOP, -B30, True),                                                                # around 0.5
        (40, TOP, 0, True), (41, -TOP, 777, True), (44, TOP, 1 << 20, True), (44, TOP, -(1 << 20), True),                   # to both ends of the clamp
        (40, TOP, B30 - 1, False), (40, TOP, -B30, False)]                                                                  # far behind them
FAST = [(33, 1012, B30 - 1, True), (33, 1012, -B30, True), (33, -1012, -B30, True), (39, 64768, B30 - 1, True), (39, -64768, B30 - 1, True), (33, 1 << 24, 5, True),
        (39, B30, -777, True), (38, -B30, 3, True), (62, TOP, B30 - 1, True), (40, TOP, 0, True), (33, TOP, B30 - 1, False), (33, -TOP, B30 - 1, False)]
SLOW = [(0, 1, 0, True), (0, -3, 5, True), (9, 1, -3, True), (1, 1, 5, True), (32, 506, B30 - 1, True), (32, -506, B30 - 1, True), (32, 506, -B30, True),
        (33, 1012, -B30, True), (40, TOP, 0, True), (62, TOP, B30 - 1, True), (0, 0, 7, False)]
BIAS = [(40, 129536, B30, True), (40, 129536, -B30 - 1, True), (40, 65536, 253 << 23, True), (40, -65536, 253 << 23, True), (40, 65536, -(253 << 23), True),
        (40, TOP, 0, True), (62, TOP, B30 + 1, True), (40, TOP, 2113929215, False), (40, TOP, -2113929215, False)]
KINDS = {"tall": (TALL, TALL, TALL), "fast": (FAST, FAST, FAST), "slow": (SLOW, SLOW, SLOW), "bias": (BIAS, BIAS, BIAS), "mixed": (TALL, FAST, SLOW),
         "values tall": (None, None, TALL), "values fast": (None, None, FAST), "values slow": (None, None, SLOW), "values bias": (None, None, BIAS)}


def deal(w, H, kind):
    """Puts the constants of a kind into the three matrices' channels in turn.  Returns which channels are meant to vary."""
    vary = np.zeros(3 * H, bool)
    for part, constants in enumerate(KINDS[kind]):
        if constants is None:
            continue
        for c in range(H):
            at = part * H + c
            w["s_qkv"][at], w["m_qkv"][at], w["b_qkv"][at], vary[at] = constants[c % len(constants)]
    return vary


def layer(heads, B_, L):
    """(configuration, input, scale of the input, weights, quantization) of one layer of 64 x heads channels."""
    cfg = synth.EncoderConfig("qkv", 64 * heads, heads, 128, L, B_, 1)
    x_q, S_x, _ = synth.input_activations(cfg)
    w, q = P.layer_params(synth.layer_raw(cfg, 0), synth.model_scales(cfg, S_x)[0], cfg.hidden, heads)
    return cfg, x_q, S_x, w, q
