"""The optimizer step writes the working copies that the next microbatch runs on: sizes whose matrices end inside a 64x64 or
64x128 tile and whose vectors end inside a workgroup's share.  After one step the loss and every gradient of the next microbatch (input
gradients go through the transposed copies) match the checker on the updated master weights, rounded to the model dtype."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import transformer as ot                                     # noqa: E402
from paper_2410_07192_amd import synth                                   # noqa: E402
from test_gpu_training import _mods, read_emb, read_layer, rel_err      # noqa: E402

SHAPES = [synth.ModelShape(2, 200, 25, 328, 20, 2, 70, True, "f32"),       # d_head 8
          synth.ModelShape(2, 72, 9, 136, 24, 2, 130, True, "bf16"),
          synth.ModelShape(2, 192, 3, 520, 64, 2, 65, False, "bf16"),      # d_head 64, one row in the last tile of E
          synth.ModelShape(2, 64, 1, 64, 8, 1, 64, True, "bf16"),          # whole tiles only
          # more than 20 M parameters: tiles of 128 columns, past the caches; every matrix ends inside a tile along both sides
          synth.ModelShape(2, 1096, 137, 2200, 12, 2, 2050, True, "bf16"),
          synth.ModelShape(2, 1096, 137, 2200, 12, 2, 2050, False, "f32")]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s.dtype}-d{s.d_model}-f{s.d_ff}")
def test_the_next_microbatch_runs_on_the_updated_weights(shape):
    pf, dev = _mods()
    tol = 1e-4 if shape.dtype == "f32" else 2e-2          # as for the first microbatch
    # Queries and keys have elements of std * sqrt(d): about one, before and after the step.  (0.08 at d = 1096 makes 2.6, scores of
    # twenty, and a score's rounding in bf16, 2^-9 of it, changes its probability by 4 %: beyond the tolerance, whatever the kernel.)
    std, lr = (0.08, 2e-2) if shape.d_model <= 200 else (0.03, 5e-3)
    d, f = shape.d_model, shape.d_ff
    assert (shape.n_layers * (4 * d * d + 2 * d * f) + shape.vocab * d >= 20_000_000) == (d > 200)
    params = synth.make_model_params(shape, seed=5, std=std)
    m = dev.DeviceModel(shape, params, training=True, adam=pf.pf_adam(lr, 0.9, 0.999, 1e-8, 1))
    try:
        ids = np.stack([synth.make_token_ids(shape, seed=90 + i)[None] for i in range(2)])
        m.set_io(dev.to_device(ids.astype(np.int32)), 2, None, 0)
        nF = len(m.chain)
        m.ctx.pf_fill_chunk(m.chunk(0, nF), m.chain)
        m.ctx.pf_ctx_sync()
        assert m.ctx.pf_ctx_train_state()[1] == 1
        stored = synth.round_to_bf16 if shape.dtype == "bf16" else (lambda a: a)
        P = ot.cast_params(params)
        moved = 0.0
        for l in range(shape.n_layers):
            for k, v in read_layer(m, 1, l).items():
                moved = max(moved, float(np.abs(P["layers"][l][k] - v).max()))
                P["layers"][l][k] = stored(v.astype(np.float32)).astype(np.float64)
        emb = read_emb(m, 1)
        for k in ("tok_emb", "pos_emb", "lnf_g", "lnf_b"):
            P[k] = stored(emb[k].astype(np.float32)).astype(np.float64)
        assert moved > lr / 2                             # a step of lr in nearly every weight
        m.ctx.pf_fill_chunk(m.chunk(nF, 2 * nF - 1), m.chain)      # the next microbatch up to its optimizer node
        loss, _ = m.ctx.pf_ctx_train_state()
        ref_loss, G = ot.model_loss_and_grads(ids[1, 0], P, shape.n_heads, shape.causal, shape.eps)
        assert abs(loss - ref_loss) < tol * max(1.0, abs(ref_loss))
        for l in range(shape.n_layers):
            got = read_layer(m, 0, l)
            for k, ref in G["layers"][l].items():
                assert rel_err(got[k], ref) < tol, (l, k)
        got = read_emb(m, 0)
        for k in ("lnf_g", "lnf_b"):
            assert rel_err(got[k], G[k]) < tol, k
    finally:
        m.close()


def test_tokens_past_the_last_are_zeros_whatever_lds_held():
    """The weight-gradient kernel takes tokens 64 at a time; with 48 tokens the rest of its only step must not come from what an
    earlier kernel left in LDS (here NaN, left by the same kernel).  Such token counts reach it above 192 tiles of 128x128: the
    head's gradient, 8200 x 368."""
    pf, dev = _mods()
    bad = torch.full((1024, 2048), float("nan"), dtype=torch.bfloat16, device="cuda")
    sink = torch.zeros(2048, 2048, device="cuda")
    pf.pf_op_gemm_tn(pf.PF_DTYPE_BF16, bad.data_ptr(), bad.data_ptr(), sink.data_ptr(), 2048, 2048, 1024)
    shape = synth.ModelShape(1, 368, 46, 1480, 24, 2, 8200, True, "bf16")
    params = synth.make_model_params(shape, seed=7, std=0.08)
    m = dev.DeviceModel(shape, params, training=True, adam=pf.pf_adam(1e-3, 0.9, 0.999, 1e-8, 2))
    try:
        ids = synth.make_token_ids(shape, seed=8)
        m.set_io(dev.to_device(ids[None, None].astype(np.int32)), 1, None, 0)
        m.ctx.pf_fill_chunk(m.chunk(0, len(m.chain)), m.chain)      # one of two microbatches: gradients stay
        m.ctx.pf_ctx_sync()
        _, G = ot.model_loss_and_grads(ids, ot.cast_params(params), shape.n_heads, shape.causal, shape.eps)
        assert rel_err(read_emb(m, 0)["tok_emb"], G["tok_emb"]) < 2e-2
    finally:
        m.close()
