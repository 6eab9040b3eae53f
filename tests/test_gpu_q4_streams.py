"""GPU parity of lockstep decoding on 4-bit codes (products of at most 32 rows)
at the edges of its row counts, K groups, K splits and columns, against the
fp64 oracle on the dequantized weights at 2e-2 (fp16 activations and
cache)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import check_logits, top2_margin
from paper_2606_12154_amd import hh

pytestmark = pytest.mark.gpu
TOL = 2e-2
# (d, heads, kv heads, FFN, vocabulary).  "whole" and "uneven" split every product's
# K over workgroups of one K group each: d 1,152 is nine 128-wide K blocks in splits
# of five and four, FFN 4,224 33 blocks in splits of five; their heads split K too,
# which leaves them to the fp16 tiles.  Unsplit products have two K groups and the
# head walks its column blocks: "head" has nine blocks as four and five, gate/up
# unsplit and 258 head blocks for 256 workgroups, the last one 9 columns wide;
# "groups" two groups of four blocks in gate/up and a head of 257 whole blocks;
# "short" splits nothing (five blocks as two and three, down as well).  d 1,088 and
# FFN 4,160 are no multiples of 128: the fp16 tiles serve those products.
SHAPES = {"whole": (1024, 16, 4, 4096, 1024), "uneven": (1152, 18, 9, 4224, 1001), "fp16 tiles": (1088, 17, 17, 4160, 1001),
          "head": (1152, 18, 9, 8192, 16457), "groups": (1024, 16, 4, 8192, 16448), "short": (640, 10, 5, 640, 1001)}


@pytest.fixture(scope="module", params=list(SHAPES))
def model(request):
    d, hq, hkv, ffn, vocab = SHAPES[request.param]
    sh = synth.ModelShape(2, d, hq, hkv, 64, ffn, vocab, 1e-5, 1e4, True, synth.BF16)
    tensors = synth.make_weights(sh, 51, gain_std=0.1)
    dec = oracle.Decoder(sh, oracle.q4_model_weights(sh, synth.weights_as_f64(sh, tensors)))
    ctx = hh.Context(hh.make_config(sh, 33, 64, 64, weight_format=hh.HH_WF_Q4G32))
    ctx.load_weights(tensors)
    yield request.param, sh, ctx, dec
    ctx.close()


@pytest.mark.parametrize("n", [2, 15, 16, 17, 31, 32, 33])
def test_lockstep_rows(model, n):
    name, sh, ctx, dec = model
    ctx.reset()
    prompts = [synth.make_tokens(sh.vocab, 1 + (5 * s) % 23, 600 + s) for s in range(n)]
    nxt = ctx.prefill_batch(list(range(n)), prompts)
    caches, worst = [], 0.0
    for s, p in enumerate(prompts):
        ref, cache = dec.prefill(p, rows="last")
        caches.append(cache)
        if top2_margin(ref[0]) > 1e-2:
            assert nxt[s] == int(np.argmax(ref[0])), (name, n, s)
    rng = np.random.default_rng(n)
    for step in range(2):
        feed = rng.integers(0, sh.vocab, size=n).astype(np.int32)
        tok, lg = ctx.decode_step(list(range(n)), feed, logits=True)
        worst = max(worst, check_logits(lg, dec.decode_batch(caches, feed), TOL, what=f"{name}, {n} rows, step {step}"))
        assert (tok == np.argmax(lg, -1)).all()
    print(f"{name}, {n} rows: max-abs {worst:.4g}")


def test_small_scales():
    """A head whose scales are 2^-19 .. 2^-17 in the fp16 operands' units (the
    embedding sets the unit): 32 rows multiply its codes, 64 rows the fp16
    copy of its values, so the same operands give the same errors but for the
    order of sums.  Scales rounded before the product gave 4 times the error."""
    sh = synth.ModelShape(1, 256, 4, 2, 64, 128, 1000, 1e-5, 1e4, False, synth.BF16)
    rng = np.random.default_rng(5)
    tensors = synth.make_weights(sh, 52)
    for i, (name, shp) in enumerate(sh.tensor_specs()):
        std = {"embed": 2.0 ** 10, "l0.wo": 0.0, "l0.w_down": 0.0, "lm_head": 2.0 ** -17}.get(name)
        if std is not None:
            tensors[i] = synth.f32_to_bf16_bits((std * rng.standard_normal(shp)).astype(np.float32))
    w = oracle.q4_model_weights(sh, synth.weights_as_f64(sh, tensors))
    toks = synth.make_tokens(sh.vocab, 64, 6)
    x = w["embed"][toks]
    ref = x / np.sqrt((x * x).mean(-1, keepdims=True) + sh.rms_eps) @ w["lm_head"].T
    ctx = hh.Context(hh.make_config(sh, 2, 80, 80, weight_format=hh.HH_WF_Q4G32))
    try:
        ctx.load_weights(tensors)
        _, copy = ctx.prefill(0, toks, logits="all")
        ctx.reset()
        _, codes = ctx.prefill(0, toks[:32], logits="all")
    finally:
        ctx.close()
    e_copy, e_codes = (float(np.linalg.norm(g[:32] - ref[:32]) / np.linalg.norm(ref[:32])) for g in (copy, codes))
    print(f"error of the copy {e_copy:.3g}, of the codes {e_codes:.3g}")
    assert e_codes <= 1.05 * e_copy
