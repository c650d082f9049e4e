"""fp32 networks over the range of fp32: weights up to FLT_MAX, activations that
overflow, and values down to where the third bf16 plane runs out of exponent.
Probe networks pass constants from biases, so every score is one known product
or the infinity or NaN that fp32 arithmetic gives."""
import numpy as np
import pytest
import torch

from oracle import donerf_oracle as O
from paper_2103_03231_amd import binding as b
from paper_2103_03231_amd import inputs

pytestmark = pytest.mark.gpu

MAX = np.finfo(np.float32).max
B = 64


def probe(layer1, layer2, head, bias0, rays):
    """Scores of a depth network whose layer 0 outputs bias0, then layer1, layer2
    (256 x 256 each), four identities and the head (B x 256)."""
    eye, zero = np.eye(256, dtype=np.float32), np.zeros(256, np.float32)
    layers = [(np.zeros((256, 90), np.float32), bias0), (layer1, zero), (layer2, zero)] + [(eye, zero)] * 4
    layers += [(head, np.zeros(B, np.float32))]
    layers += O.split_weights(inputs.make_weights(B, 0), B)[1]
    blob = np.concatenate([np.concatenate([np.asarray(w, np.float32).ravel(), np.asarray(c, np.float32)])
                           for w, c in layers])
    r = b.Renderer(b.Config(n_bins=B, n_max=4, precision=b.FP32), blob)
    out = r.render(inputs.make_poses([0]), 1, rays, 4, debug=True)
    torch.cuda.synchronize()
    s = out["scores"].cpu().numpy().reshape(-1, B)
    r.close()
    assert (s == s[0]).all() or np.isnan(s[0]).any()
    return s


def column(values):
    w = np.zeros((256, 256), np.float32)
    w[:len(values), 0] = values
    return w


EYE = np.eye(256, dtype=np.float32)
HEAD = np.eye(B, 256, dtype=np.float32)


# 33 rays run on tiles of 32, 30,000 on tiles of 64
@pytest.mark.parametrize("rays", [33, 30000])
def test_weights_up_to_the_largest_float(rays):
    w = np.array([MAX, -MAX, 0.0, np.float32(2.0 ** 127 * 1.99609375), np.float32(2.0 ** 127 * 1.9980), 3.0e38,
                  np.float32(2.0 ** 127 * 1.99609381)], np.float32)
    x = np.float32(1.2345678e-9)
    got = probe(column(w), EYE, HEAD, np.eye(256, dtype=np.float32)[0] * x, rays)[:, :len(w)]
    want = np.maximum(w.astype(np.float64) * float(x), 0.0)
    # three bf16 values hold w and x exactly; the dropped products and two fp32
    # roundings per sum are below 2^-22 of the product
    assert np.isfinite(got).all()
    assert (np.abs(got - want) <= want * 2.0 ** -22).all(), got[0]


@pytest.mark.parametrize("rays", [33, 30000])
def test_overflow_gives_the_infinities_of_fp32(rays):
    # layer 1: unit 0 overflows, unit 1 is finite, unit 2 the ReLU of -infinity
    bias0 = np.eye(256, dtype=np.float32)[0] * np.float32(1e20)
    w1 = column([1.003e25, 7.0, -1.003e25])   # w's second bf16 value has the other sign: its product is -inf
    sums = np.float32(1e20) * np.float32(7.0)
    got = probe(w1, EYE, HEAD, bias0, rays)
    # in the identities infinity * 0 = NaN reaches every other unit and the ReLU
    # makes it 0; unit 0 stays infinite
    assert (got[:, 0] == np.inf).all(), got[0, :4]
    # the head reads the infinity of unit 0 with a zero weight: NaN, as in fp32
    assert np.isnan(got[:, 1:]).all()
    # every weight on the infinite unit nonzero: signs decide
    head = HEAD.copy()
    head[:, 0] = np.where(np.arange(B) % 2 == 0, 0.5, -0.25)
    got = probe(w1, EYE, head, bias0, rays)
    assert (got[:, 0::2] == np.inf).all() and (got[:, 1::2] == -np.inf).all()
    # without the infinite unit the same network is finite
    w1[0, 0] = 0.0
    got = probe(w1, EYE, HEAD, bias0, rays)
    assert (got[:, 1] == sums).all() and (got[:, 0] == 0.0).all() and (got[:, 2] == 0.0).all()


@pytest.mark.parametrize("side", ["activation", "weight"])
@pytest.mark.parametrize("k,bound", [(100, 2.0 ** -22), (110, 2.0 ** -22), (118, 2.0 ** -16), (126, 2.0 ** -8)])
def test_small_values_lose_only_what_is_below_bf16_subnormals(side, k, bound):
    """v 2^-k times 2^k: exact parts down to 2^-133, so the relative error is at
    most 2^-134 / 2^-k (plus the products' 2^-22)."""
    v = np.float32(1.23456789)
    small, big = np.float32(float(v) * 2.0 ** -k), np.float32(2.0 ** k)
    x, w = (small, big) if side == "activation" else (big, small)
    got = probe(column([w]), EYE, HEAD, np.eye(256, dtype=np.float32)[0] * x, 33)[:, 0]
    assert 2.0 ** -134 / 2.0 ** -k <= bound
    assert (np.abs(got / float(v) - 1.0) <= bound).all(), got[0]
