"""GPU tests of the many-row LM head (HH_LOGITS_ALL): on a model without
layers the logits are RMSNorm(E[token]) . E^T, so the head stands alone
against fp64, at the precision of 32-bit inputs."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import new_context
from paper_2606_12154_amd import hh

pytestmark = pytest.mark.gpu


def reference(shape, tensors, toks):
    w = synth.weights_as_f64(shape, tensors)
    x = w["embed"][toks]
    h = x / np.sqrt((x * x).mean(-1, keepdims=True) + shape.rms_eps) * w["final_norm"]
    return h @ w["embed"].T, np.abs(h) @ np.abs(w["embed"]).T


# Widths that end inside a group of 64 columns, with and without 16-byte rows; one
# row (fp32: up to seven of these widths), which have heads of their own, also
# behind a launch of 1,024; rows at the edges of the 16-row blocks, the tiles and
# the launches.
@pytest.mark.parametrize("dtype", [synth.BF16, synth.F32])
@pytest.mark.parametrize("vocab,n", [(1000, 1), (1003, 2), (1003, 3), (1003, 7), (1003, 8), (1003, 15), (1000, 16), (1003, 17), (700, 64),
                                     (700, 65), (530, 130), (257, 1025), (257, 1026), (257, 1033)])
def test_head_alone(dtype, vocab, n):
    import torch
    shape = synth.ModelShape(0, 512, 4, 2, 64, 64, vocab, 1e-5, 1e4, True, dtype)
    tensors = synth.make_weights(shape, 31, gain_std=0.5)
    toks = synth.make_tokens(vocab, n, 32)
    ref, size = reference(shape, tensors, toks)
    # The split keeps values to 2^-23 of themselves and sums are 32-bit: 2^-17 of
    # the sum of magnitudes leaves room for both, and is 64 times below what
    # plain fp16 rows can err by.
    tol = 2.0 ** -17 * size
    ctx = new_context(shape, tensors, streams=1, context=n + 4)
    try:
        # One float past a 16-byte boundary, with guards on both sides.
        buf = torch.full((n * vocab + 8,), 7.0, dtype=torch.float32, device="cuda")
        out = buf[1:1 + n * vocab]
        nxt = np.zeros(1, dtype=np.int32)
        torch.cuda.synchronize()
        hh.hh_prefill(ctx.ctx, 0, toks, hh.HH_LOGITS_ALL, out.data_ptr(), nxt.ctypes.data)
        got = out.cpu().numpy().reshape(n, vocab)
        assert float(buf[0]) == 7.0 and bool((buf[1 + n * vocab:] == 7.0).all())
        assert (np.abs(got - ref) <= tol).all(), float((np.abs(got - ref) / size).max())
        assert int(nxt[0]) == int(np.argmax(got[-1]))
        ctx.reset()
        nxt2, host = ctx.prefill(0, toks, logits="all")  # through the staging rows
        assert nxt2 == int(nxt[0]) and (np.abs(host - ref) <= tol).all()
    finally:
        ctx.close()


# The rows' sums as a whole: with the norm in 64 bits, operands to 2^-23 and
# sums kept apart from their roundings, the relative error (2-norm) stays under
# one unit in fp32's last place, 2^-23 (measured 0.6e-7 .. 0.8e-7); one chain of
# MFMA accumulations over these 2,048 products has 2.8e-7 (bf16) and 7.8e-7 (fp32).
@pytest.mark.parametrize("dtype", [synth.BF16, synth.F32])
@pytest.mark.parametrize("d,n", [(256, 40), (2048, 40), (2112, 200)])
def test_sums(dtype, d, n):
    shape = synth.ModelShape(0, d, 4, 2, 64, 64, 4096, 1e-5, 1e4, True, dtype)
    tensors = synth.make_weights(shape, 33, gain_std=0.1)
    toks = synth.make_tokens(shape.vocab, n, 34)
    ref, _ = reference(shape, tensors, toks)
    ctx = new_context(shape, tensors, streams=1, context=n + 4)
    try:
        _, got = ctx.prefill(0, toks, logits="all")
    finally:
        ctx.close()
    err = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    print(f"d {d}, {n} rows: {err:.3g}")
    assert err <= 2.0 ** -23


def many_tiles(shape, w, toks, tol_of, aligned, **config):
    """The logits of every row, written by the kernels into the caller's
    buffer (on a 16-byte boundary or 4 bytes past one, guards on both sides)."""
    import torch
    n, vocab, (tensors, embed, head) = len(toks), shape.vocab, w
    x = embed[toks]
    h = x / np.sqrt((x * x).mean(-1, keepdims=True) + shape.rms_eps)
    ref, tol = h @ head.T, tol_of(np.abs(h) @ np.abs(head).T)
    ctx = hh.Context(hh.make_config(shape, 1, n + 4, **config))
    try:
        ctx.load_weights(tensors)
        first = 4 if aligned else 5
        buf = torch.full((n * vocab + 16,), 7.0, dtype=torch.float32, device="cuda")
        out = buf[first:first + n * vocab]
        nxt = np.zeros(1, dtype=np.int32)
        torch.cuda.synchronize()
        hh.hh_prefill(ctx.ctx, 0, toks, hh.HH_LOGITS_ALL, out.data_ptr(), nxt.ctypes.data)
        got = out.cpu().numpy().reshape(n, vocab)
        assert bool((buf[:first] == 7.0).all()) and bool((buf[first + n * vocab:] == 7.0).all())
    finally:
        ctx.close()
    assert (np.abs(got - ref) <= tol).all(), float((np.abs(got - ref) / tol).max())
    assert int(nxt[0]) == int(np.argmax(got[-1]))


# More tiles than workgroups, so that each walks several with its loads running
# ahead: 64 rows take 313 tiles of 128 x 128, 65 rows 313 and 200 rows 626 of
# 256 x 128; a vocabulary that ends inside a group of 64 columns, with 16-byte rows
# (stored as such in an aligned buffer) and without.  Tolerance as above.
@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("vocab,n", [(40004, 64), (40004, 65), (40004, 200), (40001, 200)])
def test_many_tiles(vocab, n, aligned):
    shape = synth.ModelShape(0, 512, 4, 2, 64, 64, vocab, 1e-5, 1e4, True, synth.BF16)
    tensors = synth.make_weights(shape, 35)
    embed = synth.weights_as_f64(shape, tensors)["embed"]
    many_tiles(shape, (tensors, embed, embed), synth.make_tokens(vocab, n, 36), lambda size: 2.0 ** -17 * size, aligned)


# 4-bit heads: fp16 rows against the fp16 copy of the values, in the tile kernel
# from 128 rows on (up to seven weight rows past the head are read with the
# last columns, and not stored) with the greedy key of the last row only.  A row's
# values are rounded to fp16, 2^-11 of themselves; sums are 32-bit.
@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("vocab,n", [(1003, 127), (1003, 128), (1004, 130), (1001, 597), (40004, 300)])
def test_four_bit_rows(vocab, n, aligned):
    shape = synth.ModelShape(0, 512, 4, 2, 64, 64, vocab, 1e-5, 1e4, True, synth.BF16)
    tensors = synth.make_weights(shape, 37)
    w = oracle.q4_model_weights(shape, synth.weights_as_f64(shape, tensors))
    many_tiles(shape, (tensors, w["embed"], w["lm_head"]), synth.make_tokens(vocab, n, 38), lambda size: 1.05 * 2.0 ** -11 * size, aligned,
               weight_format=hh.HH_WF_Q4G32)
