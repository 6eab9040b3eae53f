"""GPU parity of the prompt GEMMs' tile kernel on sizes that no 1B product has:
column counts that end inside a tile, an FFN width that ends inside a group of
32 gate + 32 up columns, uneven K splits, few K steps, more tiles than
workgroups (each then walks several, its loads running ahead across them), and
row counts that end inside an 8-row group.  Against the fp64 oracle at 2e-2
(fp16 activations and cache)."""
import os

import numpy as np
import pytest

import oracle
import synth
from gpu_util import check_logits, new_context

pytestmark = pytest.mark.gpu
TOL = 2e-2
KINDS = ("HH_GEMM_QKV", "HH_GEMM_RESID", "HH_GEMM_DOWN", "HH_GEMM_GATEUP")
# d 320: 5 K steps, 1,280 QKV columns; FFN 1,000 leaves the down projection
# to the generic kernel, 1,088 gives it 17 K steps.
ROWS = 2001


@pytest.fixture(scope="module", params=[1000, 1088])
def model(request):
    sh = synth.ModelShape(2, 320, 10, 5, 64, request.param, 512, 1e-5, 1e4, True, synth.BF16)
    tensors = synth.make_weights(sh, 21, gain_std=0.1)
    ref, _ = oracle.Decoder(sh, synth.weights_as_f64(sh, tensors)).prefill(synth.make_tokens(sh.vocab, ROWS, 22))
    ctx = new_context(sh, tensors, streams=1, context=ROWS + 7)
    yield sh, ctx, ref
    ctx.close()


@pytest.mark.parametrize("tile", ["256x256x1", "256x128x1", "256x128x2", "128x128x1", "128x128x3", "256x256x4"])
@pytest.mark.parametrize("n", [129, 597, ROWS])
def test_tile_edges(model, tile, n):
    sh, ctx, ref = model
    saved = {k: os.environ.get(k) for k in KINDS}
    try:
        for k in KINDS:
            os.environ[k] = tile
        ctx.reset()
        toks = synth.make_tokens(sh.vocab, ROWS, 22)[:n]
        nxt, got = ctx.prefill(0, toks, logits="all")
    finally:
        for k, v in saved.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v
    worst = check_logits(got, ref[:n], TOL, what=f"{n} rows, tiles {tile}")
    assert nxt == int(np.argmax(got[-1]))
    print(f"FFN {sh.ffn_dim}, {n} rows, tiles {tile}: max-abs {worst:.4g}")
