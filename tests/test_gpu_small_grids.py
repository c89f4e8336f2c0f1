"""Launches that leave most CUs idle: attention with 32 queries per workgroup (which sizes, and numbers at the edges of its tiles and
of the waves' shares of the keys), and the workgroups on idle CUs that read weights ahead (they change nothing)."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import transformer as ot          # noqa: E402
from paper_2410_07192_amd import synth        # noqa: E402

# B, S, h, d_head, causal: one query, edges of 32 queries and of 64 keys, one to nine tiles for four waves, several heads
SMALL = [(1, 1, 1, 64, True), (1, 31, 3, 64, False), (2, 33, 2, 64, True), (1, 127, 2, 128, True), (1, 128, 1, 128, False),
         (1, 65, 2, 64, True), (1, 128, 12, 64, False), (1, 257, 2, 64, True), (1, 257, 2, 128, False), (1, 320, 2, 128, True),
         (3, 200, 8, 64, True), (1, 333, 16, 128, True), (1, 520, 2, 64, False), (1, 577, 1, 128, True)]
# us: 256 or 128 queries per workgroup, 32 (MI355X); whether 32 are chosen
TIMED = [((16, 128, 12, 64, False), 7.7, 8.4), ((8, 128, 12, 64, False), 7.1, 5.9), ((4, 512, 12, 64, False), 15.6, 12.9),
         ((1, 1024, 16, 64, True), 23.4, 12.9), ((2, 333, 16, 128, False), 14.2, 17.1), ((4, 333, 16, 128, True), 13.6, 21.3),
         ((1, 700, 24, 128, False), 21.5, 31.8), ((1, 1024, 16, 128, True), 26.6, 20.8), ((1, 2048, 16, 128, True), 47.9, 55.6),
         ((1, 2048, 8, 128, True), 45.5, 29.5), ((32, 512, 12, 64, False), 42.0, 58.0),
         # more workgroups than are resident, with and without a mask
         ((7, 237, 12, 64, False), 11.1, 10.2),
         ((4, 438, 20, 64, True), 13.5, 15.8), ((2, 4400, 4, 64, False), 84.1, 94.0), ((47, 274, 2, 64, True), 10.8, 11.8),
         ((3, 370, 24, 64, True), 11.8, 12.3), ((1, 2318, 20, 64, True), 45.7, 47.3),
         ((1, 426, 20, 128, True), 13.7, 14.3), ((3, 719, 4, 128, False), 21.1, 21.7), ((2, 4547, 1, 128, False), 92.3, 87.8),
         ((20, 133, 2, 128, False), 10.1, 7.0), ((1, 224, 32, 128, True), 10.2, 7.3)]


def by_32(B, S, h, dh, causal):
    from paper_2410_07192_amd import binding as pf
    f = pf.lib.pf_attention_bf16_by_32
    f.restype, f.argtypes = C.c_int32, [C.c_int64, C.c_int64, C.c_int64, C.c_int32, C.c_int32]
    return bool(f(B, S, h, dh, causal))


@pytest.mark.parametrize("a", SMALL)
def test_these_run_with_32_queries_per_workgroup(a):
    assert by_32(*a)


@pytest.mark.parametrize("a,many,few", TIMED)
def test_the_faster_form_is_chosen(a, many, few):
    assert by_32(*a) == (few < many)


@pytest.mark.gpu
@pytest.mark.parametrize("B,S,h,dh,causal", SMALL)
def test_attention(B, S, h, dh, causal):
    """Against float64: 1e-2 of the largest value (probabilities and results are rounded to bf16, 2^-9 each); log-sum-exp 1e-4."""
    from paper_2410_07192_amd import binding as pf
    from paper_2410_07192_amd import device as dev
    md = pf.pf_model_desc()
    md.dtype = pf.PF_DTYPE_BF16
    d = h * dh
    rng = np.random.default_rng(S + 7 * h + dh)
    qkv = synth.round_to_bf16((rng.standard_normal((B, S, 3 * d)) * 1.5).astype(np.float32))
    dq, out = dev.storage_tensor(qkv, md), dev.empty_storage((B + 1, S, d), md)   # one sequence more: must stay untouched
    out.zero_()
    lse = torch.empty((B, h, S), dtype=torch.float32, device="cuda")
    pf.pf_op_attention(md.dtype, dq.data_ptr(), out.data_ptr(), B, S, h, dh, causal, lse.data_ptr())
    torch.cuda.synchronize()
    q, k, v = (ot.split_heads(qkv[..., i * d:(i + 1) * d].astype(np.float64), h) for i in range(3))
    ref = ot.merge_heads(ot.attention_probs(q, k, causal) @ v)
    s = q @ k.transpose(0, 1, 3, 2) / np.sqrt(dh)
    if causal:
        s = np.where(np.triu(np.ones((S, S), dtype=bool), 1), -np.inf, s)
    ref_lse = s.max(-1) + np.log(np.exp(s - s.max(-1, keepdims=True)).sum(-1))
    got = dev.read_storage(out, md)
    assert np.abs(got[:B] - ref).max() < 1e-2 * np.abs(ref).max() and not got[B].any()
    assert np.abs(lse.cpu().numpy() - ref_lse).max() < 1e-4


@pytest.mark.gpu
@pytest.mark.parametrize("S,h", [(70, 2), (200, 1)])
def test_scores_far_apart_and_infinite(S, h):
    """Scores of the order of 1e4 (the running maximum jumps between tiles and waves), and keys whose scores are -inf."""
    from paper_2410_07192_amd import binding as pf
    from paper_2410_07192_amd import device as dev
    md = pf.pf_model_desc()
    md.dtype = pf.PF_DTYPE_BF16
    dh, d = 64, h * 64
    rng = np.random.default_rng(S)
    qkv = rng.standard_normal((1, S, 3 * d)).astype(np.float32)
    qkv[..., :d] = 30.0
    qkv[..., d:2 * d] = (rng.integers(-40, 41, (1, S, 1)) * np.ones((1, S, d))).astype(np.float32)   # score 240 x key's number
    qkv[:, 3, d:2 * d] = -np.inf
    qkv = synth.round_to_bf16(qkv)
    dq, out = dev.storage_tensor(qkv, md), dev.empty_storage((1, S, d), md)
    assert by_32(1, S, h, dh, False)
    pf.pf_op_attention(md.dtype, dq.data_ptr(), out.data_ptr(), 1, S, h, dh, False)
    torch.cuda.synchronize()
    q, k, v = (ot.split_heads(qkv[..., i * d:(i + 1) * d].astype(np.float64), h) for i in range(3))
    s = q @ np.where(np.isinf(k), 0, k).transpose(0, 1, 3, 2) / 8.0
    s[..., 3] = -np.inf
    p = np.exp(s - s.max(-1, keepdims=True))
    ref = ot.merge_heads((p / p.sum(-1, keepdims=True)) @ v)
    assert np.abs(dev.read_storage(out, md) - ref).max() < 1e-2 * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [synth.ModelShape(3, 768, 12, 3072, 128, 1, 0, False, "bf16"),
                                   synth.ModelShape(2, 256, 4, 1024, 33, 3, 0, True, "bf16"),
                                   synth.ModelShape(2, 64, 1, 72, 1, 1, 0, True, "bf16"),
                                   synth.ModelShape(2, 256, 4, 1024, 128, 2, 0, False, "f32")], ids=lambda s: f"{s.dtype}-d{s.d_model}-S{s.seq_len}")
def test_layers_that_read_ahead(shape):
    from test_gpu_forward import TOL, _oracle_model, _run_model, rel_err
    params = synth.make_model_params(shape, seed=3)
    x = synth.make_hidden(shape, seed=4)
    assert rel_err(_run_model(shape, params, x[None])[0], _oracle_model(shape, params, x)) < TOL[shape.dtype]
