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
# 192 rows (two kv heads) or 384 (one) stay with the row kernel.
EDGES = [1, 31, 32, 33, 63, 64, 65, 100]
CASES = {
    "edges": (2, EDGES, 0, 0),
    "appended": (2, EDGES, 13, 0),
    "passes": (2, [150, 7, 97, 200, 30], 5, 210),
    "below the row threshold": (2, [95, 96], 0, 0),
    "at the row threshold": (2, [95, 97], 0, 0),
    "one group": (2, [1 + (17 * i) % 70 for i in range(190)], 3, 0),
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
