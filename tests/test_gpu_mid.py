"""GPU parity of the short-prompt GEMMs (at most 128 rows) at the edges of their
row counts, with K splits that end unevenly and an FFN width that ends
inside a group of 32 gate + 32 up columns.  Against the fp64 oracle at 2e-2
(fp16 activations and cache)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import check_logits, new_context

pytestmark = pytest.mark.gpu
TOL = 2e-2
# (d, heads, kv heads, FFN): K splits over 16 or 17 and 64 or 65 steps; an FFN of
# 4,104 leaves the down projection to the generic kernel.
SHAPES = {"whole": (1024, 16, 4, 4096), "odd": (1088, 17, 17, 4160), "ffn": (1024, 16, 4, 4104)}


@pytest.fixture(scope="module", params=list(SHAPES))
def model(request):
    d, hq, hkv, ffn = SHAPES[request.param]
    sh = synth.ModelShape(1, d, hq, hkv, 64, ffn, 512, 1e-5, 1e4, True, synth.BF16)
    tensors = synth.make_weights(sh, 41, gain_std=0.1)
    toks = synth.make_tokens(sh.vocab, 128, 42)
    ref, _ = oracle.Decoder(sh, synth.weights_as_f64(sh, tensors)).prefill(toks)
    ctx = new_context(sh, tensors, streams=1, context=160)
    yield request.param, ctx, toks, ref
    ctx.close()


@pytest.mark.parametrize("n", [1, 8, 31, 32, 33, 50, 64, 65, 99, 127, 128])
def test_rows(model, n):
    name, ctx, toks, ref = model
    ctx.reset()
    nxt, got = ctx.prefill(0, toks[:n], logits="all")
    worst = check_logits(got, ref[:n], TOL, what=f"{name}, {n} rows")
    assert nxt == int(np.argmax(got[-1]))
    # The rest as an appended chunk: the same products on other rows.
    if n < 128:
        _, rest = ctx.prefill(0, toks[n:], logits="all")
        worst = max(worst, check_logits(rest, ref[n:], TOL, what=f"{name}, rows {n} .. 127"))
    print(f"{name}, {n} rows: max-abs {worst:.4g}")
