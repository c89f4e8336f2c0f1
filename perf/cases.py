"""The work a user of the library has it do, as measurable cases: whole passes of fill jobs and of the main-job stage
through the public entry points, from one fp32 layer to a training step of a 12-layer decoder.

Three kinds of case:
  infer  forward of a fill job's whole chain (embedding, layers, final LayerNorm) by pf_fill_chunk_fwd, weights resident
         or streamed from pinned host memory; result: the final hidden states
  train  one optimizer step of a training fill job: `accum` replicas of the chain (forward, tied-head loss, recomputing
         backward, Adam at the end) by pf_fill_chunk; result: master weights and first moments
  stage  one optimizer step of the emulated main-job stage: `accum` microbatches forward and backward, Adam; result: the
         last microbatch's output and input gradient, master weights and first moments
"""
import math

import torch
import torch.utils.checkpoint

from paper_2410_07192_amd import binding as pf
from paper_2410_07192_amd import device as dev
from paper_2410_07192_amd import synth


def _case(name, kind, layers, d, heads, ff, seq, batch, vocab, causal, dtype="bf16", g=1, slots=0, accum=1):
    c = dict(kind=kind, layers=layers, d=d, heads=heads, ff=ff, seq=seq, batch=batch, vocab=vocab, causal=causal,
             dtype=dtype, g=g, slots=slots, accum=accum)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest configuration (cfg1): one fp32 encoder layer on 512 tokens, hidden states in and out
        _case("layer_fp32", "infer", 1, 256, 4, 1024, 128, 4, 0, False, "f32"),
        # one short request to the 12-layer encoder of cfg2: 84 dependent launches of little work each
        _case("encode_single", "infer", 12, 768, 12, 3072, 128, 1, 30522, False),
        # the same encoder on a small batch whose lengths fit no tile
        _case("encode_ragged", "infer", 12, 768, 12, 3072, 237, 7, 30522, False),
        # cfg2: batch inference of the encoder
        _case("encode_batch", "infer", 12, 768, 12, 3072, 512, 32, 30522, False),
        # prefill of one prompt of odd length through 8 of the layers of cfg3's decoder
        _case("prefill_prompt", "infer", 8, 2048, 16, 8192, 333, 1, 50257, True),
        # cfg3's decoder, 6 layers, weights streamed through 3 HBM slots, two microbatches per layer visit
        _case("decode_streamed", "infer", 6, 2048, 16, 8192, 1024, 16, 50257, True, g=2, slots=3),
        # two of its layers on one long document
        _case("decode_long", "infer", 2, 2048, 16, 8192, 8192, 1, 50257, True),
        # training a small decoder on batches whose token count is no multiple of 64
        _case("train_small", "train", 4, 512, 8, 2048, 200, 3, 10007, True),
        # cfg4: training the 12-layer decoder, an optimizer step every two microbatches
        _case("train_batch", "train", 12, 1024, 16, 4096, 1024, 8, 50257, True, accum=2),
        # cfg5: one layer of the d = 8192 main stage, four microbatches to the optimizer step
        _case("stage_step", "stage", 1, 8192, 64, 32768, 2048, 1, 0, True, accum=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: sizes log-uniform, sequence lengths and vocabularies as they come, work and
    memory no more than the largest listed case of the kind."""
    most = {}
    for c in listed():
        w = work(c)
        most[c["kind"]] = max(most.get(c["kind"], 0.0), w["flops"] / 50, w["bytes"])
    while True:
        kind = rng.choice(["infer", "infer", "infer", "infer", "train", "train", "stage"])
        dtype = "f32" if kind == "infer" and rng.random() < 0.2 else "bf16"
        if dtype == "f32":
            dh = rng.choice([32, 64])
            heads = _log(rng, 2, 8)
            layers, seq, batch = rng.randint(1, 2), _log(rng, 24, 256), _log(rng, 1, 8)
        else:
            dh = rng.choice([64, 128])
            heads = _log(rng, 4, {"infer": 24, "train": 16, "stage": 64}[kind])
            layers = {"infer": _log(rng, 1, 12), "train": _log(rng, 2, 12), "stage": 1}[kind]
            seq, batch = _log(rng, 16, 8192 if kind == "infer" else 2048), _log(rng, 1, 32 if kind == "infer" else 8)
        if kind != "infer":
            seq = (seq + 7) // 8 * 8    # bf16 weight gradients contract over the tokens, eight at a time
        d = dh * heads
        ff = 4 * d if rng.random() < 0.7 else (int(d * rng.uniform(2.0, 4.5)) + 7) // 8 * 8
        vocab = 0 if kind == "stage" or (kind == "infer" and rng.random() < 0.3) else _log(rng, 2000, 50257)
        causal = kind != "infer" or rng.random() < 0.5
        slots = 3 if kind == "infer" and dtype == "bf16" and layers >= 4 and rng.random() < 0.2 else 0
        g = rng.choice([1, 2]) if slots else 1
        accum = rng.choice([1, 2, 4]) if kind != "infer" else 1
        c = _case(None, kind, layers, d, heads, ff, seq, batch, vocab, causal, dtype, g, slots, accum)
        w = work(c)
        cost = max(w["flops"] / 50, w["bytes"])
        params = layers * (4 * d * d + 2 * d * ff)
        if cost <= most[kind] and 8 <= seq * batch <= 32768 and params <= (8 << 26 if slots else 8 << 27):
            return c


def _shape(c):
    return synth.ModelShape(c["layers"], c["d"], c["heads"], c["ff"], c["seq"], c["batch"], c["vocab"], c["causal"],
                            c["dtype"])


def _storage(shape, case, gen, std=1.0, mean=0.0):
    t = torch.randn(shape, device="cuda", generator=gen) * std + mean
    return t.to(torch.bfloat16) if case["dtype"] == "bf16" else t


def _f32_bytes(md):
    """Bytes pf_ctx_read_params delivers for a layer and for the embedding block."""
    md32 = pf.pf_model_desc.from_buffer_copy(md)
    md32.dtype = pf.PF_DTYPE_F32
    layer, _ = pf.pf_layer_blob_layout(md32)
    up = lambda n: (n + 255) // 256 * 256
    vp = (md.vocab + 63) // 64 * 64
    emb = up(vp * md.d_model * 4) + up(md.seq_len * md.d_model * 4) + 2 * up(md.d_model * 4) if md.vocab else 0
    return layer, emb


def _draw(case, seed):
    """Parameters and inputs of a case: layer blobs on the device, embedding and final LayerNorm, input, stage gradient."""
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    md = pf.model_desc(_shape(c))
    g = c["accum"] if c["kind"] == "stage" else c["g"]     # the stage keeps the step's microbatches in flight
    blobs = [dev.random_layer_blob(md, seed * 1000 + l, pinned=c["slots"] > 0) for l in range(c["layers"])]
    tok = pos = grad = None
    if c["vocab"]:
        tok = _storage((c["vocab"], c["d"]), c, gen, 0.02)
        pos = _storage((c["seq"], c["d"]), c, gen, 0.02)
    lnf_g = _storage((c["d"],), c, gen, 0.02, 1.0)
    lnf_b = _storage((c["d"],), c, gen, 0.02)
    rows = (c["batch"], c["seq"])
    n_in = c["accum"] if c["kind"] == "train" else 1
    if c["vocab"]:
        x = torch.randint(0, c["vocab"], (n_in, g) + rows, device="cuda", generator=gen, dtype=torch.int32)
    else:
        x = _storage((g,) + rows + (c["d"],), c, gen)
    if c["kind"] == "stage":
        grad = _storage((g,) + rows + (c["d"],), c, gen, 1e-3)
    return md, g, n_in, blobs, tok, pos, lnf_g, lnf_b, x, grad


def prepare(case, seed):
    c, shape = case, _shape(case)
    md, g, n_in, blobs, tok, pos, lnf_g, lnf_b, x, grad = _draw(c, seed)
    training = c["kind"] != "infer"
    adam = pf.pf_adam(1e-4, 0.9, 0.999, 1e-8, c["accum"]) if training else None
    model = dev.RawModel(shape, blobs, tok, pos, lnf_g, lnf_b, g=g, streamed=c["slots"] > 0, n_slots=c["slots"],
                         training=training, adam=adam)
    s = {"case": c, "model": model, "in": x}
    rows = (c["batch"], c["seq"])
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    if c["kind"] == "infer":
        s["out"] = torch.empty((g,) + rows + (c["d"],), device="cuda", dtype=dt)
        model.set_io(s["in"], 1, s["out"], 1)
        s["chunk"] = pf.pf_chunk(0, 0, 0, len(model.chain), 0, 0)
        return s
    layer, emb = _f32_bytes(md)
    if c["kind"] == "train":
        model.set_io(s["in"], n_in, None, 0)
        s["chunk"] = pf.pf_chunk(0, 0, 0, n_in * len(model.chain), 0, 0)
    else:
        s["grad"] = grad
        s["y"] = torch.empty(rows + (c["d"],), device="cuda", dtype=dt)
        s["dx"] = torch.empty_like(s["y"])
    n = c["layers"] * layer + emb
    s["read"] = [(l, l * layer, layer) for l in range(c["layers"])] + ([(-1, c["layers"] * layer, emb)] if emb else [])
    s["master"] = torch.empty(n // 4, device="cuda", dtype=torch.float32)
    s["moment"] = torch.empty(n // 4, device="cuda", dtype=torch.float32)
    return s


def run(s):
    c, ctx = s["case"], s["model"].ctx
    stream = torch.cuda.current_stream().cuda_stream or None
    if c["kind"] == "infer":
        ctx.pf_fill_chunk_fwd(s["chunk"], s["model"].chain, stream=stream)
        return s["out"]
    if c["kind"] == "train":
        ctx.pf_fill_chunk(s["chunk"], s["model"].chain, stream=stream)
        out = {}
    else:
        for i in range(c["accum"]):
            ctx.pf_main_stage_step(pf.PF_INSTR_FWD, i, s["in"][i].data_ptr(), stream)
            ctx.pf_main_stage_step(pf.PF_INSTR_BWD, i, s["grad"][i].data_ptr(), stream)
        ctx.pf_main_stage_read(0, c["accum"] - 1, s["y"].data_ptr(), s["y"].nbytes, stream)
        ctx.pf_main_stage_read(1, c["accum"] - 1, s["dx"].data_ptr(), s["dx"].nbytes, stream)
        ctx.pf_main_stage_step(pf.PF_INSTR_OPT, c["accum"], None, stream)
        out = dict(y=s["y"], dx=s["dx"])
    for what, key in ((1, "master"), (2, "moment")):
        for layer, off, size in s["read"]:
            ctx.pf_ctx_read_params(what, layer, s[key].data_ptr() + off, size, stream)
    return dict(out, master=s["master"], moment=s["moment"])


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    d, f, S, L = c["d"], c["ff"], c["seq"], c["layers"]
    reps = c["accum"] if c["kind"] != "infer" else c["g"]
    T = c["batch"] * S                                           # tokens of a microbatch
    per_layer = 4 * d * d + 2 * d * f
    params = L * (per_layer + 9 * d + f)
    fwd = L * (2 * T * per_layer + 4 * c["batch"] * S * S * d * (0.5 if c["causal"] else 1.0))
    act = T * d * e
    ids = 4 * T if c["vocab"] else act
    if c["kind"] == "infer":
        emb = min(T, c["vocab"]) * d * e + S * d * e if c["vocab"] else 0
        return dict(bytes=params * e + emb + reps * (ids + act), flops=reps * fwd)
    emb = (c["vocab"] + S + 2) * d if c["vocab"] else 0
    flops = 3 * reps * (fwd + 2 * T * d * c["vocab"])
    # weights read and written, both moments read and written, and the two results this pass hands out
    return dict(bytes=(params + emb) * 4 * 8 + reps * (ids + (3 * act if c["kind"] == "stage" else 0)), flops=flops)


def tolerance(case):
    """fp32 storage: sums of up to 1024 terms in another order.  bf16 storage: every tensor of a layer is rounded to 8
    significant bits on its way through memory; against the same path with fp32 storage the hidden states after 2 to 12
    layers differ by 0.007 to 0.009 (largest value 0.05), first moments by 0.003 to 0.011 (largest value 1.0: the rms of
    a gradient tensor is far below its few large values), master weights by 0.0005."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 2e-2, "max": 0.2 if case["kind"] == "infer" else 0.99}


# rows and columns of a layer's parameters in blob order, as multiples of d and ff (0: a vector)
_PARAMS = (("d", 0), ("d", 0), ("3d", "d"), ("3d", 0), ("d", "d"), ("d", 0), ("d", 0), ("d", 0), ("ff", "d"), ("ff", 0),
           ("d", "ff"), ("d", 0))


def _layer64(blob, md, c):
    """The twelve parameters of a layer in 64 bits: LayerNorm gain and bias, QKV, output, LayerNorm, FFN 1, FFN 2."""
    n = {"d": c["d"], "3d": 3 * c["d"], "ff": c["ff"], 0: 1}
    flat = blob.cuda().view(torch.bfloat16 if c["dtype"] == "bf16" else torch.float32)
    off = pf.pf_layer_blob_layout(md)[1]
    out = []
    for o, (r, k) in zip(off, _PARAMS):
        o //= flat.element_size()
        p = flat[o:o + n[r] * n[k]].double()
        out.append(p.view(n[r], n[k]) if k else p)
    return out


def _forward64(x, P, c):
    B, S, d = x.shape
    h = c["heads"]
    norm = lambda t, g, b: torch.nn.functional.layer_norm(t, (d,), g, b, 1e-5)
    q, k, v = ((norm(x, P[0], P[1]) @ P[2].t() + P[3]).view(B, S, 3, h, d // h).permute(2, 0, 3, 1, 4).contiguous())
    heads = []
    for b in range(B):
        s = q[b] @ k[b].transpose(1, 2).contiguous() / math.sqrt(d // h)
        if c["causal"]:
            s = s.masked_fill(torch.ones(S, S, dtype=torch.bool, device=x.device).triu(1), -math.inf)
        heads.append((s.softmax(-1) @ v[b]).transpose(0, 1).reshape(S, d))
    x = x + torch.stack(heads) @ P[4].t() + P[5]
    u = torch.nn.functional.gelu(norm(x, P[6], P[7]) @ P[8].t() + P[9])
    return x + u @ P[10].t() + P[11]


def exact(case, seed):
    """The same pass in 64-bit torch: hidden states, or the moments (1 - beta1) * mean gradient after the first step and,
    for the stage, its output and input gradient.  Master weights have none: after one step Adam moves every weight by the
    learning rate with the gradient's sign, which rounding decides where a gradient is as good as zero."""
    c = case
    md, g, n_in, blobs, tok, pos, lnf_g, lnf_b, x, grad = _draw(c, seed)
    layers = [_layer64(b, md, c) for b in blobs]
    emb = [t.double() for t in (tok, pos, lnf_g, lnf_b)] if c["vocab"] else []
    final = [lnf_g.double(), lnf_b.double()]
    d = c["d"]
    norm = lambda t, a, b: torch.nn.functional.layer_norm(t, (d,), a, b, 1e-5)
    if c["kind"] == "infer":
        outs = []
        with torch.no_grad():
            for i in range(g):
                t = emb[0][x[0, i].long()] + emb[1] if emb else x[i].double()
                for P in layers:
                    t = _forward64(t, P, c)
                outs.append(norm(t, *final))
        return torch.stack(outs)
    leaves = [p.requires_grad_() for P in layers for p in P] + [t.requires_grad_() for t in emb]
    y = dx = None
    for i in range(c["accum"]):
        if c["kind"] == "stage":
            t0 = t = x[i].double().requires_grad_()
        else:
            ids = x[i, 0].long()
            t = emb[0][ids] + emb[1]
        for P in layers:
            t = torch.utils.checkpoint.checkpoint(_forward64, t, P, c, use_reentrant=False)
        if c["kind"] == "stage":
            t.backward(grad[i].double())
            y, dx = t.detach(), t0.grad
        else:
            logits = norm(t, emb[2], emb[3])[:, :-1] @ emb[0].t()
            torch.nn.functional.cross_entropy(logits.reshape(-1, c["vocab"]), ids[:, 1:].reshape(-1)).backward()
            del logits
    layer, block = _f32_bytes(md)
    up = lambda n: (n + 255) // 256 * 64
    moment = torch.zeros((c["layers"] * layer + block) // 4, device="cuda", dtype=torch.float64)
    at = 0
    for i, p in enumerate(leaves):
        moment[at:at + p.numel()] = p.grad.reshape(-1) * (0.1 / c["accum"])
        n = (c["vocab"] + 63) // 64 * 64 * d if emb and i == len(leaves) - 4 else p.numel()   # the vocabulary is padded
        at += up(n * 4)
    out = dict(y=y, dx=dx) if c["kind"] == "stage" else {}
    return dict(out, master=None, moment=moment)
