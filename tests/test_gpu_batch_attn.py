"""GPU parity of the multi-stream prefill pass's MFMA attention (rows of
several streams, query-block pairs as work items) at the edges of its blocks,
key-split forms and dispatch, against the fp64 oracle at 2e-2 (fp16
activations and cache, as for every bf16 model here)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import check_logits, new_context, top2_margin

pytestmark = pytest.mark.gpu
TOL = 2e-2


def shape(hkv):
    return synth.ModelShape(2, 256, 8, hkv, 64, 512, 1024, 1e-5, 1e4, True, synth.BF16)


# Four heads per kv head run two key-split groups below 768 workgroups (4 per
# item here) and one from there on; eight heads always one.  Fewer than
# 192 rows (two kv heads) or 384 (one) stay with the row kernel, and so do
# streams of few rows each on longer contexts.
EDGES = [1, 31, 32, 33, 63, 64, 65, 100]
CASES = {
    "edges": (2, EDGES, 0, 0),
    "appended": (2, EDGES, 13, 0),
    "passes": (2, [150, 7, 97, 200, 30], 5, 210),
    "below the row threshold": (2, [95, 96], 0, 0),
    "at the row threshold": (2, [95, 97], 0, 0),
    "one group": (2, [1 + (17 * i) % 70 for i in range(190)], 3, 0),
    "few rows a stream": (2, [1] * 195, 260, 0),
    "eight heads": (1, EDGES, 2, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_batch_attention(name):
    hkv, lens, before, max_prefill = CASES[name]
    sh = shape(hkv)
    tensors = synth.make_weights(sh, 11, gain_std=0.1)
    model = oracle.Decoder(sh, synth.weights_as_f64(sh, tensors))
    n = len(lens)
    heads = [synth.make_tokens(sh.vocab, before, 500 + s) for s in range(n)]
    prompts = [synth.make_tokens(sh.vocab, k, 900 + s) for s, k in enumerate(lens)]
    # All rows in one pass, or with max_prefill in passes that split between
    # and inside prompts.
    ctx = new_context(sh, tensors, streams=n, context=sum(lens) + before + 8, max_prefill=max_prefill)
    try:
        if before:
            for s in range(n):
                ctx.prefill(s, heads[s])
        order = list(range(n))[::-1]
        nxt = ctx.prefill_batch(order, [prompts[s] for s in order])
        caches, refs = [], []
        for s in range(n):
            ref, cache = model.prefill(np.concatenate([heads[s], prompts[s]]), rows="last")
            refs.append(ref[0])
            caches.append(cache)
        for i, s in enumerate(order):
            if top2_margin(refs[s]) > 1e-2:
                assert nxt[i] == int(np.argmax(refs[s])), (name, s)
        toks = [int(np.argmax(r)) for r in refs]
        _, lg = ctx.decode_step(list(range(n)), toks, logits=True)
        worst = check_logits(lg, model.decode_batch(caches, toks), TOL, what=name)
    finally:
        ctx.close()
    print(f"{name}: max-abs {worst:.4g}")


# ---- precision: queries and softmax weights enter as two fp16 terms each.
# Embedding rows are +-1 (so the RMSNorm leaves them as they are) and every
# weight is a power of two or an integer of few bits, so keys and values are
# exact; rotary angles of the dimensions in use are below 1e-11.  The first
# layer's attention output reaches the residual stream, whose normalised rows
# are the second layer's values; a lockstep step then attends to all of them
# evenly, and its logits are compared with the fp64 oracle.
TAIL = 800


def precision_model(kind, heads):
    d, vocab = 256, 64
    rng = np.random.default_rng(77)
    x = rng.choice([-1.0, 1.0], size=(vocab, d))
    t = np.arange(vocab)
    x[:, 0] = 1
    x[:, 1], x[:, 2], x[:, 3] = 1 - 2 * (t & 1), np.where(t == 0, 1, -1), 1 - (t & 2)
    sh = synth.ModelShape(2, d, heads, 1, 64, 64, vocab, 1e-12, 1e30, False, synth.BF16)
    wq, wk, wv = np.zeros((64, d)), np.zeros((64, d)), np.zeros((64, d))
    if kind == "low part of q":
        # q = (256 + 2^-4 x1, 256), k = 512 x3 (1, -1): scores of +-4 that come
        # from the part of q below half an fp16 ulp alone.
        wq[20, 0], wq[20, 1], wq[21, 0] = 256, 2.0 ** -4, 256
        wk[20, 3], wk[21, 3] = 512, -512
        wv[np.arange(64), 4 + np.arange(64)] = 1
        out = 1.0
    elif kind == "q past fp16":
        # q = 2^18, k = 2^-14 x3: scores of +-2.
        wq[20, 0], wk[20, 3] = 2.0 ** 18, 2.0 ** -14
        wv[np.arange(64), 4 + np.arange(64)] = 1
        out = 1.0
    else:
        # Token 0's key leads by 15.625 and its value is zero: what is left is
        # a tail of weights of about 2.7 2^-24, each beside a sum of 1.
        wq[20, 0], wk[20, 0], wk[20, 2] = 8, 7.8125, 7.8125
        wv[:, 0], wv[:, 2] = 64, -64
        out = 2.0 ** 6 / 64
    wo = np.zeros((d, 64 * heads))
    wo[4 + np.arange(64 * 3), rng.integers(0, 64 * heads, 64 * 3)] = out * 64 if kind == "flat tail" else out
    zero = np.zeros((64, d))
    wv2, wo2 = np.zeros((64, d)), np.zeros((d, 64 * heads))
    wv2[np.arange(64), rng.choice(np.arange(4, 196), 64, replace=False)] = 1
    wo2[np.arange(192, 256), np.arange(64)] = 4
    head = rng.choice([-1.0, 1.0], size=(vocab, d)) * 2.0 ** -4
    one = np.ones(d)
    w = [x]
    for q, k, v, o in ((wq, wk, wv, wo), (zero, zero, wv2, wo2)):
        w += [one, np.tile(q, (heads, 1)), k, v, o, one, zero, zero, zero.T.copy()]
    tensors = [synth.f32_to_bf16_bits(m.astype(np.float32)) for m in w + [one, head]]
    return sh, tensors


# The outputs are rounded to fp16 four times on the way (attention output,
# second norm, values, final norm; 2^-12 each of values whose logits are about
# 1): 4 x 2^-12 is the bound at full precision.  Queries in one fp16 term are
# off by 0.2 in the first case, weights without a scale by 0.04 in the last.
PRECISION_TOL = 2.0 ** -10


@pytest.mark.parametrize("heads", [4, 8])
@pytest.mark.parametrize("kind", ["low part of q", "q past fp16", "flat tail"])
def test_two_terms(kind, heads):
    sh, tensors = precision_model(kind, heads)
    model = oracle.Decoder(sh, synth.weights_as_f64(sh, tensors))
    prompts = [np.concatenate([[0], 1 + synth.make_tokens(sh.vocab - 1, TAIL + 7 * s, 40 + s)]) for s in range(2)]
    ctx = new_context(sh, tensors, streams=2, context=TAIL + 32, max_prefill=2 * TAIL + 32)
    try:
        ctx.prefill_batch([0, 1], prompts)
        caches = [model.prefill(p, rows="last")[1] for p in prompts]
        _, got = ctx.decode_step([0, 1], [5, 6], logits=True)
        ref = model.decode_batch(caches, [5, 6])
    finally:
        ctx.close()
    assert bool(np.isfinite(got).all()), "non-finite logits"
    worst = float(np.abs(got - ref).max())
    print(f"{kind}, {heads} heads: max-abs {worst:.4g} (logits to {np.abs(ref).max():.3g})")
    assert worst <= PRECISION_TOL
