"""The 4-bit quantizer's rows, byte for byte (integer results: exact), where
its split of the work can go wrong: rows of one to many groups that do not
divide a block's 256 groups, every pair of bf16 significands as value and
scale (the quotient's ties among them), and groups whose scale is zero, tiny,
huge, infinite or beside a NaN.  The reference is the format's own divisions
in fp32."""
import numpy as np
import pytest

import synth
from test_gpu_q4 import quantize_on_gpu

pytestmark = pytest.mark.gpu


def stored_rows(v):
    """Codes and scales of fp32 rows of bf16 values by fp32 division."""
    with np.errstate(all="ignore"):
        g = v.reshape(v.shape[0], -1, 32)
        a = np.fmax.reduce(np.abs(g), axis=-1, initial=np.float32(0))
        s = synth.f32_to_bf16_bits((a / np.float32(7)).astype(np.float32))
        sf = synth.bf16_bits_to_f32(s).reshape(a.shape)[..., None]
        r = np.where(sf > 0, g / sf, np.float32(0))
        q = np.clip(np.rint(np.where(np.isnan(r), 0, r)), -8, 7).astype(np.int32)
    n = (q + 8).astype(np.uint8).reshape(v.shape)
    scales = np.ascontiguousarray(s.reshape(a.shape)).view(np.uint8).reshape(v.shape[0], -1)
    return np.concatenate([n[:, 0::2] | (n[:, 1::2] << 4), scales], axis=1)


def check(v):
    got, exact = quantize_on_gpu(v)
    bad = np.argwhere(got != stored_rows(exact))
    assert bad.size == 0, f"{len(bad)} bytes differ, first at {bad[:5].tolist()}"


@pytest.mark.parametrize("rows,K", [(1, 32), (255, 32), (257, 64), (85, 96), (3, 2080), (129, 2048), (5, 8192)])
def test_shapes(rows, K):
    rng = np.random.default_rng(rows * 10007 + K)
    check((0.02 * rng.standard_normal((rows, K))).astype(np.float32))


def test_every_pair_of_significands():
    # Rows: the group's largest value (so its scale); within: every significand
    # at each exponent that still leaves a code, either sign.
    sig = np.arange(128, 256, dtype=np.float32)
    vals = np.concatenate([sign * sig * np.float32(2.0 ** e) for e in range(-6, 1) for sign in (1, -1)])
    rows = []
    for top in sig:
        g = vals.reshape(-1, 31)[: len(vals) // 31] if len(vals) % 31 == 0 else np.resize(vals, (len(vals) // 31 + 1, 31))
        g = np.where(np.abs(g) > top, np.float32(0), g)
        rows.append(np.concatenate([np.full((len(g), 1), top, np.float32), g], axis=1).reshape(-1))
    check(np.stack(rows))


def test_scales_at_the_ends():
    rng = np.random.default_rng(3)
    base = rng.standard_normal((12, 64)).astype(np.float32)
    mags = [0.0, 1e-40, 1e-38, 2.0 ** -101, 2.0 ** -98, 1e-20, 1e20, 2.0 ** 99, 2.0 ** 104, 1e38, 1.0, 1.0]
    with np.errstate(all="ignore"):
        v = (base.astype(np.float64) * np.array(mags)[:, None]).astype(np.float32)
    v[10, 5] = np.inf
    v[11, 7], v[11, 40:64] = np.nan, np.nan
    check(v)
