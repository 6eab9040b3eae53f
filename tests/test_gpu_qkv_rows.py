"""GPU parity of the QKV product of 256 .. 511 prompt rows, whose K is split as
often as fills one round of tiles: four, three and two times (24 column tiles,
and 26 of which the last is half full) and, with 36, three times, twice and not
at all.  Against the fp64 oracle at 2e-2 (fp16 activations and cache)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import check_logits, new_context

pytestmark = pytest.mark.gpu
TOL = 2e-2
ROWS = 511


@pytest.fixture(scope="module", params=[(32, 8), (17, 17), (48, 12)], ids=["24 tiles", "26 tiles", "36 tiles"])
def model(request):
    hq, hkv = request.param
    sh = synth.ModelShape(1, 1024, hq, hkv, 64, 512, 512, 1e-5, 1e4, True, synth.BF16)
    tensors = synth.make_weights(sh, 61, gain_std=0.1)
    toks = synth.make_tokens(sh.vocab, ROWS, 62)
    ref, _ = oracle.Decoder(sh, synth.weights_as_f64(sh, tensors)).prefill(toks)
    ctx = new_context(sh, tensors, streams=1, context=ROWS + 9)
    yield ctx, toks, ref
    ctx.close()


@pytest.mark.parametrize("n", [255, 256, 257, 384, 385, ROWS])
def test_rows(model, n):
    ctx, toks, ref = model
    ctx.reset()
    nxt, got = ctx.prefill(0, toks[:n], logits="all")
    worst = check_logits(got, ref[:n], TOL, what=f"{n} rows")
    assert nxt == int(np.argmax(got[-1]))
    print(f"{n} rows: max-abs {worst:.4g}")
