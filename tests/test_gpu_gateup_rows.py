"""GPU parity of prompts whose last rows take a gate/up launch of their own (a
whole round of tiles, then 1 .. 200 rows through each of the kernels for so
few), with an FFN width that ends inside a group of 32 gate + 32 up columns.
Against the fp64 oracle at 2e-2 (fp16 activations and cache)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import check_logits, new_context

pytestmark = pytest.mark.gpu
TOL = 2e-2
ROWS = 1224


@pytest.fixture(scope="module")
def model():
    sh = synth.ModelShape(1, 1024, 16, 4, 64, 8168, 512, 1e-5, 1e4, True, synth.BF16)
    tensors = synth.make_weights(sh, 51, gain_std=0.1)
    toks = synth.make_tokens(sh.vocab, ROWS, 52)
    ref, _ = oracle.Decoder(sh, synth.weights_as_f64(sh, tensors)).prefill(toks)
    ctxs = [new_context(sh, tensors, streams=s, context=ROWS + 8) for s in (1, 2)]
    yield ctxs, toks, ref
    for c in ctxs:
        c.close()


@pytest.mark.parametrize("streams", [1, 2])  # 2: the context also keeps operand tiles for at most 32 rows
@pytest.mark.parametrize("n", [1024, 1025, 1056, 1057, 1089, 1152, 1153, ROWS])
def test_last_rows(model, n, streams):
    ctxs, toks, ref = model
    ctx = ctxs[streams - 1]
    ctx.reset()
    nxt, got = ctx.prefill(0, toks[:n], logits="all")
    worst = check_logits(got, ref[:n], TOL, what=f"{n} rows")
    assert nxt == int(np.argmax(got[-1]))
    print(f"{n} rows, {streams} stream(s): max-abs {worst:.4g}")
