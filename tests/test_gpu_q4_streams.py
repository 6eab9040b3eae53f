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
# d 1,152: nine 128-wide K blocks over two K groups; FFN 4,224: 33 blocks in splits
# of five; a vocabulary that ends inside a block of 64 columns.  d 1,088 and
# FFN 4,160 are no multiples of 128: the fp16 tiles serve those products.
SHAPES = {"whole": (1024, 16, 4, 4096, 1024), "uneven": (1152, 18, 9, 4224, 1001), "fp16 tiles": (1088, 17, 17, 4160, 1001)}


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
