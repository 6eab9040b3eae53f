"""What a user of the decoder runtime has it do, as cases to time and to compare.

A case is a dict of plain values; ``what`` names the kind of call:

* ``prefill``  one prompt through ``hh_prefill``: the time-to-first-token call
               (last row's logits and the greedy next token);
* ``turns``    a conversation: a first prompt longer than one prefill pass,
               then a second prompt appended to the same stream;
* ``score``    a prompt with the logits of every row (rating given text);
* ``decode``   a request: prompt, then ``steps`` device-fed batch-1 steps;
* ``batch``    several requests arriving together: ``hh_prefill_batch`` over
               ragged prompts, then the first lockstep step;
* ``lockstep`` several streams served together: batch prefill, then ``steps``
               device-fed lockstep steps;
* ``quantize`` the 4-bit quantizer on its own.

Models are the two shapes of the workload table.  Matrices are N(0, 0.02^2)
and gains 1 + N(0, 0.1^2); embedding rows are N(0, 1), so that with the tied
head the greedy token leads by many standard deviations, as a trained model's
does on text that it copies (random rows of 0.02 leave near-ties that the
smallest change of rounding flips).  Every pass ends as a serving program's
does, with the token ids in host memory.
"""
import math

import numpy as np
import torch

from paper_2606_12154_amd import hh

SHAPES = {
    "tiny": dict(layers=2, d=256, hq=4, hkv=2, ffn=688, vocab=4096, theta=1e4),
    "1b": dict(layers=16, d=2048, hq=32, hkv=8, ffn=8192, vocab=128256, theta=5e5),
}
EPS = 1e-5


class _Shape:
    """The attributes hh.make_config reads."""

    def __init__(self, case):
        s = SHAPES[case["model"]]
        self.n_layers, self.d_model, self.n_heads, self.n_kv_heads = s["layers"], s["d"], s["hq"], s["hkv"]
        self.head_dim, self.ffn_dim, self.vocab, self.rms_eps, self.rope_theta = 64, s["ffn"], s["vocab"], EPS, s["theta"]
        self.tied, self.dtype = True, hh.HH_F32 if case["weights"] == "f32" else hh.HH_BF16


# ------------------------------------------------------------------ cases

def listed():
    return [
        # The smallest model and request: launches and latency are all there is.
        dict(name="tiny f32 request", what="decode", model="tiny", weights="f32", prompt=64, steps=32),
        # The time to first token of one rendered answer (about 100 ids).
        dict(name="first token 99", what="prefill", model="1b", weights="bf16", prompt=99),
        # The same at the prefill-dominated workload's prompt.
        dict(name="first token 1024", what="prefill", model="1b", weights="bf16", prompt=1024),
        # A conversation in 512-row passes; the second turn starts mid page.
        dict(name="two turns 1100+77", what="turns", model="1b", weights="bf16", prompt=1100, second=77, rows=512),
        # Rating given text: every row's logits.
        dict(name="score 200", what="score", model="1b", weights="bf16", prompt=200),
        # The headline request (shorter by its later steps, which cost the same).
        dict(name="decode 256+64", what="decode", model="1b", weights="bf16", prompt=256, steps=64),
        # The same on 4-bit weights, the precision of the deployed model.
        dict(name="q4 decode 256+64", what="decode", model="1b", weights="q4", prompt=256, steps=64),
        # Long context: an 8192-token prompt, then steps that attend to all of it.
        dict(name="long 8192+24", what="decode", model="1b", weights="bf16", prompt=8192, steps=24),
        # 32 requests of about 100 ids arriving together, to their first tokens.
        dict(name="batch 32 x 99", what="batch", model="1b", weights="bf16", streams=32, prompt=99),
        # The multi-stream serving workload.
        dict(name="lockstep 32 x 256+48", what="lockstep", model="1b", weights="bf16", streams=32, prompt=256, steps=48),
        # A few users at once on the 4-bit model.
        dict(name="q4 lockstep 6 x 120+48", what="lockstep", model="1b", weights="q4", streams=6, prompt=120, steps=48),
        # Quantizing the largest matrix of the load, the LM head's table.
        dict(name="quantize 128256 x 2048", what="quantize", rows=128256, cols=2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["decode", "decode", "prefill", "prefill", "turns", "score", "batch", "lockstep", "lockstep", "quantize"])
    c = dict(what=what)
    if what == "quantize":
        c["cols"] = 32 * _log_int(rng, 2, 256)
        c["rows"] = _log_int(rng, 16, (1 << 28) // c["cols"])
        return c
    tiny = what in ("decode", "prefill", "batch") and rng.random() < 0.2
    c["model"] = "tiny" if tiny else "1b"
    c["weights"] = "f32" if tiny else ("q4" if rng.random() < 0.3 else "bf16")
    if what == "prefill":
        c["prompt"] = _log_int(rng, 8, 1024 if tiny else 4096)
    elif what == "turns":
        c["prompt"], c["second"], c["rows"] = _log_int(rng, 300, 3000), _log_int(rng, 3, 600), _log_int(rng, 128, 1024)
    elif what == "score":
        c["prompt"] = _log_int(rng, 8, 400)
    elif what == "decode":
        c["prompt"], c["steps"] = _log_int(rng, 8, 600 if tiny else 6000), _log_int(rng, 4, 64)
    else:
        # From a pair of users to twice the workload table's 32.
        c["streams"] = _log_int(rng, 2, 64)
        c["prompt"] = _log_int(rng, 16, max(24, min(400, 6000 // c["streams"])))
        if what == "lockstep":
            c["steps"] = _log_int(rng, 4, 48 if c["streams"] <= 32 else 24)
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _weights(case, seed):
    """The model's tensors on the GPU, in load order and storage type."""
    s = SHAPES[case["model"]]
    dt = torch.float32 if case["weights"] == "f32" else torch.bfloat16
    g = _gen(seed)

    def mat(rows, cols, std=0.02):
        return torch.empty((rows, cols), dtype=dt, device="cuda").normal_(0.0, std, generator=g)

    def gain():
        return torch.empty(s["d"], dtype=dt, device="cuda").normal_(1.0, 0.1, generator=g)

    d, f, q, kv = s["d"], s["ffn"], 64 * s["hq"], 64 * s["hkv"]
    t = [mat(s["vocab"], d, 1.0)]
    for _ in range(s["layers"]):
        t += [gain(), mat(q, d), mat(kv, d), mat(kv, d), mat(d, q), gain(), mat(f, d), mat(f, d), mat(d, f)]
    return t + [gain()]


def _prompts(case, seed):
    """Each stream's prompt: uniform ids; several streams' lengths spread
    from 0.6 to 1.4 times ``prompt``, except in the workload table's
    lockstep case (32 equal prompts of 256)."""
    rng = np.random.RandomState(int(seed) % (1 << 31))
    v, p, n = SHAPES[case["model"]]["vocab"], case["prompt"], case.get("streams", 1)
    # Lengths are the case's, not the seed's.
    lens = [p] * n
    if n > 1 and (n, p) != (32, 256):
        lens = [max(1, int(round(p * (0.6 + 0.8 * ((7 * i + 3) % n) / (n - 1))))) for i in range(n)]
    if case["what"] == "turns":
        lens = [p, case["second"]]
    return [rng.randint(0, v, size=k).astype(np.int32) for k in lens]


def _matrix(case, seed):
    w = torch.empty((case["rows"], case["cols"]), dtype=torch.bfloat16, device="cuda")
    return w.normal_(0.0, 0.02, generator=_gen(seed))


def prepare(case, seed):
    if case["what"] == "quantize":
        k = case["cols"]
        return dict(case=case, src=_matrix(case, seed),
                    dst=torch.empty((case["rows"], k // 2 + k // 16), dtype=torch.uint8, device="cuda"))
    prompts = _prompts(case, seed)
    n, steps = case.get("streams", 1), case.get("steps", 1)
    longest = sum(map(len, prompts)) if case["what"] == "turns" else max(map(len, prompts))
    cap = case.get("rows") or (max(longest, min(8192, sum(map(len, prompts)))) if n > 1 else longest)
    context = max(longest + steps + 1, cap)
    fmt = hh.HH_WF_Q4G32 if case["weights"] == "q4" else hh.HH_WF_DTYPE
    ctx = hh.Context(hh.make_config(_Shape(case), n, context, cap, weight_format=fmt))
    w = _weights(case, seed)
    torch.cuda.synchronize()  # the weights are written on torch's stream, read on the context's
    ctx.load_weights(w)
    rows = len(prompts[0]) if case["what"] == "score" else n
    logits = torch.empty((rows, SHAPES[case["model"]]["vocab"]), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    return dict(case=case, ctx=ctx, prompts=prompts, logits=logits, ids=np.arange(n, dtype=np.int32))


# ------------------------------------------------------------------ a pass

def _history(ctx, stream, first):
    return ctx.read_argmax(stream, first, ctx.length(stream) - first)


def run(state):
    case = state["case"]
    if case["what"] == "quantize":
        src, dst = state["src"], state["dst"]
        hh.hh_q4g32_quantize(src.data_ptr(), case["rows"], case["cols"], dst.data_ptr(), torch.cuda.current_stream().cuda_stream)
        return dst
    ctx, prompts, logits, ids = state["ctx"], state["prompts"], state["logits"], state["ids"]
    out = np.zeros(len(ids), dtype=np.int32)
    ctx.reset()
    if case["what"] in ("prefill", "score"):
        mode = hh.HH_LOGITS_ALL if case["what"] == "score" else hh.HH_LOGITS_LAST
        hh.hh_prefill(ctx.ctx, 0, prompts[0], mode, logits.data_ptr(), out.ctypes.data)
        return dict(next=out, logits=logits)
    if case["what"] == "turns":
        first, _ = ctx.prefill(0, prompts[0])
        hh.hh_prefill(ctx.ctx, 0, prompts[1], hh.HH_LOGITS_LAST, logits.data_ptr(), out.ctypes.data)
        return dict(first=first, next=out, logits=logits)
    if case["what"] == "decode":
        ctx.prefill(0, prompts[0])
        for k in range(case["steps"]):
            last = k + 1 == case["steps"]
            hh.hh_decode_step(ctx.ctx, 1, ids, None, logits.data_ptr() if last else None, None)
        return dict(tokens=_history(ctx, 0, len(prompts[0]) - 1), logits=logits)
    ctx.prefill_batch(ids, prompts)
    steps = case.get("steps", 1)
    for k in range(steps):
        last = k + 1 == steps
        hh.hh_decode_step(ctx.ctx, len(ids), ids, None, logits.data_ptr() if last else None, None)
    tokens = [_history(ctx, s, len(prompts[s]) - 1) for s in range(len(ids))]
    return dict(tokens=np.stack(tokens), logits=logits)


# ------------------------------------------------------------------ cost and tolerance

def work(case):
    if case["what"] == "quantize":
        n = case["rows"] * case["cols"]
        return dict(bytes=n * 2 + n // 2 + n // 16, flops=2 * n)
    s = SHAPES[case["model"]]
    d, hq, hkv, v = s["d"], s["hq"], s["hkv"], s["vocab"]
    layer = d * 64 * (2 * hq + 2 * hkv) + 3 * d * s["ffn"]  # matrix elements
    size = {"f32": 4.0, "bf16": 2.0, "q4": 0.5625}[case["weights"]]
    kv_row = 2 * hkv * 64 * s["layers"] * (4 if case["weights"] == "f32" else 2)
    mats = (layer * s["layers"] + v * d) * size
    lens = [len(p) for p in _prompts(case, 0)]
    if case["what"] == "turns":
        lens = [sum(lens)]
    rows = sum(lens)
    heads = rows if case["what"] == "score" else len(lens)
    nbytes = mats + rows * kv_row + heads * v * 4
    flops = 2.0 * (layer * s["layers"] * rows + v * d * heads)
    flops += sum(4.0 * 64 * hq * s["layers"] * n * (n + 1) / 2 for n in lens)
    steps = case.get("steps", 1 if case["what"] == "batch" else 0)
    for k in range(steps):
        attended = rows + len(lens) * (k + 1)
        nbytes += mats + attended * kv_row
        flops += 2.0 * len(lens) * (layer * s["layers"] + v * d) + 4.0 * 64 * hq * s["layers"] * attended
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    if case["what"] == "quantize":
        return "exact"
    # Against exact(): fp32 1e-6, 16-bit and 4-bit weights (fp16 activations
    # and KV cache, fp32 sums) 1e-3 of the logits' norm.
    return dict(rel=1e-5) if case["weights"] == "f32" else dict(rel=4e-3, max=0.05)


# ------------------------------------------------------------------ 64-bit results

def _q4(w):
    """Codes and scales of the 4-bit groups of a bf16 matrix's rows.  The
    format divides in fp32; a quotient rounded from 64 bits is the same."""
    g = w.double().reshape(w.shape[0], -1, 32)
    s = (g.abs().amax(-1) / 7.0).float().bfloat16()
    sd = s.double().unsqueeze(-1)
    r = torch.where(sd > 0, (g / sd).float(), torch.zeros((), device=w.device))
    return r.round().clamp(-8, 7).to(torch.int16), s


def _values(case, w):
    """The 64-bit values that a matrix of the model is computed with."""
    if case["weights"] != "q4":
        return w.double()
    q, s = _q4(w)
    return (q.double() * s.double().unsqueeze(-1)).reshape(w.shape)


def _norm(x, gain):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _forward(case, tensors, seqs):
    """Residual rows after the last block of each sequence (its positions
    from 0), concatenated."""
    s = SHAPES[case["model"]]
    hq, hkv = s["hq"], s["hkv"]
    x = tensors[0][torch.from_numpy(np.concatenate(seqs).astype(np.int64)).cuda()].double()
    pos = torch.cat([torch.arange(len(t), device="cuda") for t in seqs]).double()
    ang = pos[:, None] * s["theta"] ** (-2.0 * torch.arange(32, device="cuda", dtype=torch.float64) / 64.0)
    cos, sin = ang.cos()[:, None, :], ang.sin()[:, None, :]

    def rope(t):
        a, b = t[..., :32], t[..., 32:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    longest = max(len(t) for t in seqs)
    hidden = torch.ones((longest, longest), dtype=torch.bool, device="cuda").triu(1)
    for l in range(s["layers"]):
        an, wq, wk, wv, wo, mn, wg, wu, wd = tensors[1 + 9 * l:10 + 9 * l]
        h = _norm(x, an)
        q = rope((h @ _values(case, wq).T).reshape(-1, hq, 64))
        k = rope((h @ _values(case, wk).T).reshape(-1, hkv, 64))
        v = (h @ _values(case, wv).T).reshape(-1, hkv, 64)
        o = torch.empty_like(q)
        r0 = 0
        for t in seqs:
            n = len(t)
            for j in range(hq):
                g = j // (hq // hkv)
                sc = (q[r0:r0 + n, j].contiguous() @ k[r0:r0 + n, g].T.contiguous()) * 0.125
                sc.masked_fill_(hidden[:n, :n], -math.inf)
                o[r0:r0 + n, j] = torch.softmax(sc, -1) @ v[r0:r0 + n, g].contiguous()
            r0 += n
        x = x + o.reshape(x.shape[0], -1) @ _values(case, wo).T
        h = _norm(x, mn)
        gate = h @ _values(case, wg).T
        x = x + (gate * torch.sigmoid(gate) * (h @ _values(case, wu).T)) @ _values(case, wd.T.contiguous())
    return x


def exact(case, seed):
    if case["what"] == "quantize":
        q, s = _q4(_matrix(case, seed))
        n = (q + 8).to(torch.uint8).reshape(case["rows"], -1)
        scales = s.contiguous().view(torch.uint8).reshape(case["rows"], -1)
        return torch.cat([n[:, 0::2] | (n[:, 1::2] << 4), scales], 1)
    tensors = _weights(case, seed)
    head = _values(case, tensors[0])

    def logits(x):
        return _norm(x, tensors[-1]) @ head.T

    prompts = _prompts(case, seed)
    if case["what"] in ("prefill", "score"):
        x = _forward(case, tensors, prompts)
        y = logits(x if case["what"] == "score" else x[-1:])
        return dict(next=y[-1].argmax().reshape(1).to(torch.int32), logits=y)
    if case["what"] == "turns":
        y = logits(_forward(case, tensors, [np.concatenate(prompts)])[[len(prompts[0]) - 1, -1]])
        return dict(first=int(y[0].argmax()), next=y[1].argmax().reshape(1).to(torch.int32), logits=y[1:])
    # Greedy continuations: guess that each stream repeats its last token (the
    # embedding's lead makes it so), run prompt and guess as one sequence, and
    # put right what the argmax says otherwise until nothing changes.
    steps = case.get("steps", 1)
    tails = [[int(p[-1])] * steps for p in prompts]
    for _ in range(8):
        x = _forward(case, tensors, [np.concatenate([p, np.array(t, dtype=np.int32)]) for p, t in zip(prompts, tails)])
        said, last, r0 = [], [], 0
        for p in prompts:
            y = logits(x[r0 + len(p) - 1:r0 + len(p) + steps])
            said.append([int(i) for i in y.argmax(-1)])
            last.append(y[-1])
            r0 += len(p) + steps
        if all(a[:steps] == t for a, t in zip(said, tails)):
            break
        tails = [a[:steps] for a in said]
    else:
        return None
    tokens = np.array(said, dtype=np.int32)
    return dict(tokens=tokens[0] if case["what"] == "decode" else tokens, logits=torch.stack(last))
