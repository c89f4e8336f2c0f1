"""GPU parity of the training path (forward, tied-head loss, recomputing backward, gradient
accumulation, Adam) and of the emulated main-job stage, against the CPU checker.

Gradient tolerance: max |gpu - ref| / max |ref| per gradient tensor, 1e-4 for fp32 storage and 2e-2
for bf16 storage (the checker gets the bf16-rounded parameters widened to float64)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import transformer as ot          # noqa: E402
from paper_2410_07192_amd import synth        # noqa: E402


def _mods():
    from paper_2410_07192_amd import binding as pf
    from paper_2410_07192_amd import device as dev
    return pf, dev


def rel_err(got, ref):
    ref = np.asarray(ref, dtype=np.float64)
    return float(np.abs(np.asarray(got, dtype=np.float64) - ref).max() / max(np.abs(ref).max(), 1e-30))


def read_layer(m, what, layer):
    pf, dev = _mods()
    md32 = pf.pf_model_desc.from_buffer_copy(m.md)
    md32.dtype = pf.PF_DTYPE_F32
    size, _ = pf.pf_layer_blob_layout(md32)
    buf = torch.empty(size, dtype=torch.uint8, device="cuda")
    m.ctx.pf_ctx_read_params(what, layer, buf.data_ptr(), size)
    m.ctx.pf_ctx_sync()
    return pf.unpack_layer_blob_f32(m.md, buf.cpu().numpy())[0]


def read_emb(m, what):
    pf, dev = _mods()
    md = m.md
    al = lambda x: (x + 255) // 256 * 256
    vp = (md.vocab + 63) // 64 * 64
    size = al(vp * md.d_model * 4) + al(md.seq_len * md.d_model * 4) + 2 * al(md.d_model * 4)
    buf = torch.empty(size, dtype=torch.uint8, device="cuda")
    m.ctx.pf_ctx_read_params(what, -1, buf.data_ptr(), size)
    m.ctx.pf_ctx_sync()
    out, total = pf.unpack_embedding_f32(md, buf.cpu().numpy())
    assert total == size
    return out


TRAIN_SHAPES = [
    (synth.ModelShape(2, 64, 4, 128, 24, 2, 50, True, "f32"), 1e-4),      # d_head 16, T = 48
    (synth.ModelShape(2, 128, 2, 256, 64, 2, 300, True, "bf16"), 2e-2),   # d_head 64, T = 128
    (synth.ModelShape(1, 256, 2, 512, 96, 2, 130, False, "bf16"), 2e-2),  # d_head 128, encoder, T = 192
]


@pytest.mark.parametrize("shape,tol", TRAIN_SHAPES, ids=lambda x: getattr(x, "dtype", None) and f"{x.dtype}-d{x.d_model}" or "")
def test_gradients_loss_and_adam(shape, tol):
    pf, dev = _mods()
    params = synth.make_model_params(shape, seed=31, std=0.08)
    P = ot.cast_params(params)
    adam = pf.pf_adam(1e-3, 0.9, 0.999, 1e-8, 2)
    m = dev.DeviceModel(shape, params, training=True, adam=adam)
    try:
        ids = np.stack([synth.make_token_ids(shape, seed=50 + i)[None] for i in range(2)])   # 2 replicas, g = 1
        d_in = dev.to_device(ids.astype(np.int32))
        m.set_io(d_in, 2, None, 0)
        nF = len(m.chain)
        assert nF == 2 * shape.n_layers + 4
        st = torch.cuda.Stream()
        # replica 0: forward chunk, then the backward cut in two (a bubble boundary in between)
        cut = shape.n_layers + 3
        m.ctx.pf_fill_chunk_fwd(m.chunk(0, cut), m.chain, stream=st.cuda_stream)
        m.ctx.pf_ctx_sync()
        m.ctx.pf_fill_chunk_bwd(m.chunk(cut, cut + 1), m.chain, stream=st.cuda_stream)
        m.ctx.pf_ctx_sync()
        m.ctx.pf_fill_chunk(m.chunk(cut + 1, nF), m.chain, stream=st.cuda_stream)
        loss, steps = m.ctx.pf_ctx_train_state()
        assert steps == 0                                       # accum = 2: no optimizer step yet
        ref_loss, G = ot.model_loss_and_grads(ids[0, 0], P, shape.n_heads, shape.causal, shape.eps, checkpoint=True)
        assert abs(loss - ref_loss) < tol * max(1.0, abs(ref_loss))
        for l in range(shape.n_layers):
            got = read_layer(m, 0, l)
            for k, ref in G["layers"][l].items():
                assert rel_err(got[k], ref) < tol, (l, k)
        ge = read_emb(m, 0)
        for k in ("tok_emb", "pos_emb", "lnf_g", "lnf_b"):
            assert rel_err(ge[k], G[k]) < tol, k
        assert not ge["tok_pad"].any()                          # padded vocabulary rows get no gradient
        # replica 1 through pf_fill_chunk in one go: triggers the optimizer step on the mean gradient
        ch = m.chunk(nF, 2 * nF)
        m.ctx.pf_fill_chunk(ch, m.chain, stream=st.cuda_stream)
        loss2, steps = m.ctx.pf_ctx_train_state()
        assert steps == 1
        ref_loss2, G2 = ot.model_loss_and_grads(ids[1, 0], P, shape.n_heads, shape.causal, shape.eps)
        assert abs(loss2 - ref_loss2) < tol * max(1.0, abs(ref_loss2))
        # Adam on the mean of the two microbatch gradients; compare the UPDATE (theta1 - theta0)
        for l in range(shape.n_layers):
            got = read_layer(m, 1, l)
            for k in G["layers"][l]:
                gmean = 0.5 * (G["layers"][l][k] + G2["layers"][l][k])
                th1, _, _ = ot.adam_step(P["layers"][l][k], 0.0, 0.0, gmean, 1, lr=1e-3)
                upd_ref = th1 - P["layers"][l][k]
                upd_got = got[k].astype(np.float64) - P["layers"][l][k]
                # the first Adam step is -lr * g/(|g| + eps): compare where the gradient is not tiny
                big = np.abs(gmean) > max(1e-3, 5 * tol) * np.abs(gmean).max()
                assert np.abs(upd_got - upd_ref)[big].max() < 0.05 * 1e-3, (l, k)
        # gradients were cleared by the step
        assert not any(np.any(v) for v in read_layer(m, 0, 0).values())
    finally:
        m.close()


def test_training_chunked_through_timeline():
    """A training chain planned onto bubbles and run by the Executor loop lowers nothing silently:
    optimizer steps happen and the loss is finite."""
    import ctypes as C
    pf, dev = _mods()
    shape = synth.ModelShape(2, 128, 2, 256, 64, 4, 300, True, "bf16")
    params = synth.make_model_params(shape, seed=3, std=0.05)
    m = dev.DeviceModel(shape, params, training=True, adam=pf.pf_adam(1e-3, 0.9, 0.999, 1e-8, 2))
    try:
        ids = np.stack([synth.make_token_ids(shape, seed=70 + i)[None] for i in range(4)])
        d_in = dev.to_device(ids.astype(np.int32))
        m.set_io(d_in, 4, None, 0)
        st, main = torch.cuda.Stream(), torch.cuda.Stream()
        m.ctx.pf_profile_chain(m.chain, 1, 2, st.cuda_stream)
        _, steps0 = m.ctx.pf_ctx_train_state()
        p, mm, stage, tf, tb = 3, 4, 1, 2_000_000, 4_000_000
        windows = pf.pf_schedule_1f1b(p, mm, stage, tf, tb, 1 << 34, True, 0)
        plan, n_plan, k = pf.pf_plan_bubbles(windows, m.chain, 800_000, 0, 0, raw=True)
        cursor = C.c_int32(0)
        done = 0
        for _ in range(4):
            s = pf.pf_timeline_run(m.ctx, None, None, p, mm, stage, tf, tb, windows, plan, n_plan, m.chain, cursor,
                                   st.cuda_stream, main.cuda_stream)
            done += s["replicas_done"]
        loss, steps = m.ctx.pf_ctx_train_state()
        assert done >= 2 and steps - steps0 >= done // 2 - 1
        assert np.isfinite(loss) and 0 < loss < 2 * np.log(shape.vocab)
    finally:
        m.close()


def test_profiling_leaves_training_state_alone():
    """pf_profile_chain runs every node of a training chain, optimizer nodes included, and still leaves parameters,
    moment estimates, gradient accumulators, step count and accumulated loss as they were; with microbatches
    accumulated it refuses to run."""
    pf, dev = _mods()
    shape = synth.ModelShape(2, 128, 2, 256, 64, 2, 300, True, "bf16")
    params = synth.make_model_params(shape, seed=3, std=0.05)
    m = dev.DeviceModel(shape, params, training=True, adam=pf.pf_adam(1e-2, 0.9, 0.999, 1e-8, 2))
    try:
        ids = np.stack([synth.make_token_ids(shape, seed=70 + i)[None] for i in range(2)])
        m.set_io(dev.to_device(ids.astype(np.int32)), 2, None, 0)
        st = torch.cuda.Stream()
        nF = len(m.chain)
        # one real optimizer step first (two microbatches), so the moments and the step count are not zero
        for r in range(2):
            m.ctx.pf_fill_chunk(pf.pf_chunk(0, 0, r * nF, (r + 1) * nF, 0, 0), m.chain, stream=st.cuda_stream)
        m.ctx.pf_ctx_sync()
        before = [[read_layer(m, what, l) for l in range(shape.n_layers)] + [read_emb(m, what)] for what in range(4)]
        m.ctx.pf_profile_chain(m.chain, 1, 3, st.cuda_stream)   # 4 passes: two dry optimizer steps
        assert all(n.dur_ns > 0 for n in m.chain)
        after = [[read_layer(m, what, l) for l in range(shape.n_layers)] + [read_emb(m, what)] for what in range(4)]
        for what in range(4):
            for a, b in zip(before[what], after[what]):
                for k in a:
                    assert np.array_equal(a[k], b[k]), (what, k)
        loss, steps = m.ctx.pf_ctx_train_state()
        assert steps == 1
        assert abs(loss - np.log(shape.vocab)) < 1.0     # the mean over the two real microbatches, not over six
        # one more microbatch is now accumulated towards a step of two: profiling must refuse
        m.ctx.pf_fill_chunk(pf.pf_chunk(0, 0, 2 * nF, 3 * nF, 0, 0), m.chain, stream=st.cuda_stream)
        m.ctx.pf_ctx_sync()
        with pytest.raises(pf.PipeFillError) as e:
            m.ctx.pf_profile_chain(m.chain, 0, 1, st.cuda_stream)
        assert e.value.code == pf.PF_ERR_STATE
    finally:
        m.close()


def test_main_stage_needs_a_checkpoint_slot_per_microbatch_in_flight():
    """A main context with fewer checkpoint slots (g) than the schedule keeps microbatches in flight would have
    forward j+g overwrite the checkpoints of microbatch j: refused, not computed wrongly."""
    import ctypes as C
    pf, dev = _mods()
    shape = synth.ModelShape(1, 128, 2, 256, 64, 1, 0, True, "bf16")
    params = synth.make_model_params(shape, seed=41, std=0.08)
    m = dev.DeviceModel(shape, params, g=1, training=True)
    try:
        x = dev.storage_tensor(synth.make_hidden(shape, seed=60), m.md)
        st, fs = torch.cuda.Stream(), torch.cuda.Stream()
        m.ctx.pf_main_stage_step(pf.PF_INSTR_FWD, 0, x.data_ptr(), st.cuda_stream)
        with pytest.raises(pf.PipeFillError) as e:
            m.ctx.pf_main_stage_step(pf.PF_INSTR_FWD, 1, x.data_ptr(), st.cuda_stream)   # slot 0 is still in use
        assert e.value.code == pf.PF_ERR_STATE
        m.ctx.pf_main_stage_step(pf.PF_INSTR_BWD, 0, x.data_ptr(), st.cuda_stream)
        with pytest.raises(pf.PipeFillError) as e:
            m.ctx.pf_main_stage_step(pf.PF_INSTR_BWD, 0, x.data_ptr(), st.cuda_stream)   # no forward to go back through
        assert e.value.code == pf.PF_ERR_STATE
        m.ctx.pf_ctx_sync()
        p, mm, stage = 3, 4, 1                       # stage 1 of 3 keeps min(p - stage, m) = 2 microbatches in flight
        windows = pf.pf_schedule_1f1b(p, mm, stage, 1_000_000, 2_000_000, 1 << 30, True, 0)
        with pytest.raises(pf.PipeFillError) as e:
            pf.pf_timeline_run(None, m.ctx, x.data_ptr(), p, mm, stage, 1_000_000, 2_000_000, windows, None, 0, None,
                               C.c_int32(0), fs.cuda_stream, st.cuda_stream)
        assert e.value.code == pf.PF_ERR_ARG
        stats = pf.pf_timeline_run(None, m.ctx, x.data_ptr(), p, mm, 2, 1_000_000, 2_000_000,
                                   pf.pf_schedule_1f1b(p, mm, 2, 1_000_000, 2_000_000, 1 << 30, True, 0), None, 0, None,
                                   C.c_int32(0), fs.cuda_stream, st.cuda_stream)        # last stage: one in flight
        assert stats["main_busy_ns"] > 0
    finally:
        m.close()


@pytest.mark.parametrize("dtype,tol", [("f32", 1e-4), ("bf16", 2e-2)])
def test_main_stage_forward_backward(dtype, tol):
    """Emulated main-job stage: forward of two microbatches, then their backwards (1F1B order keeps
    several microbatches in flight), against the checker's layer forward/backward."""
    pf, dev = _mods()
    shape = synth.ModelShape(2, 128, 2, 256, 64, 2, 0, True, dtype)
    params = synth.make_model_params(shape, seed=41, std=0.08)
    P = ot.cast_params(params)
    m = dev.DeviceModel(shape, params, g=2, training=True)
    try:
        xs = [synth.make_hidden(shape, seed=60 + i) for i in range(2)]
        dys = [synth.make_hidden(shape, seed=80 + i) * (1.0 if dtype == "f32" else 1.0) for i in range(2)]
        dxs = [dev.storage_tensor(x, m.md) for x in xs]
        ddy = [dev.storage_tensor(x, m.md) for x in dys]
        st = torch.cuda.Stream()
        for j in range(2):
            m.ctx.pf_main_stage_step(pf.PF_INSTR_FWD, j, dxs[j].data_ptr(), st.cuda_stream)
        for j in range(2):
            m.ctx.pf_main_stage_step(pf.PF_INSTR_BWD, j, ddy[j].data_ptr(), st.cuda_stream)
        m.ctx.pf_ctx_sync()
        Gsum = [None, None]
        for j in range(2):
            x = xs[j].astype(np.float64)
            caches = []
            for l in range(2):
                x, c = ot.layer_forward(x, P["layers"][l], shape.n_heads, True, shape.eps, keep=True)
                caches.append(c)
            dx = dys[j].astype(np.float64)
            for l in (1, 0):
                dx, G = ot.layer_backward(dx, caches[l], P["layers"][l], shape.n_heads)
                Gsum[l] = G if Gsum[l] is None else {k: Gsum[l][k] + G[k] for k in G}
        for l in range(2):
            got = read_layer(m, 0, l)
            for k, ref in Gsum[l].items():
                assert rel_err(got[k], ref) < tol, (l, k)
        with pytest.raises(pf.PipeFillError) as e:
            m.ctx.pf_main_stage_step(pf.PF_INSTR_BUBBLE, 0, dxs[0].data_ptr(), st.cuda_stream)
        assert e.value.code == pf.PF_ERR_ARG
    finally:
        m.close()


def test_main_stage_optimizer_update():
    """PF_INSTR_OPT of the emulated main stage: Adam on the mean of the accumulated microbatch gradients."""
    pf, dev = _mods()
    shape = synth.ModelShape(2, 128, 2, 256, 64, 2, 0, True, "f32")
    params = synth.make_model_params(shape, seed=43, std=0.08)
    P = ot.cast_params(params)
    m = dev.DeviceModel(shape, params, g=2, training=True, adam=pf.pf_adam(1e-3, 0.9, 0.999, 1e-8, 1))
    try:
        xs = [synth.make_hidden(shape, seed=160 + i) for i in range(2)]
        dys = [synth.make_hidden(shape, seed=180 + i) for i in range(2)]
        dxs = [dev.storage_tensor(x, m.md) for x in xs]
        ddy = [dev.storage_tensor(x, m.md) for x in dys]
        st = torch.cuda.Stream()
        for j in range(2):
            m.ctx.pf_main_stage_step(pf.PF_INSTR_FWD, j, dxs[j].data_ptr(), st.cuda_stream)
        for j in range(2):
            m.ctx.pf_main_stage_step(pf.PF_INSTR_BWD, j, ddy[j].data_ptr(), st.cuda_stream)
        m.ctx.pf_main_stage_step(pf.PF_INSTR_OPT, 2, None, st.cuda_stream)
        m.ctx.pf_ctx_sync()
        Gsum = [None, None]
        for j in range(2):
            x = xs[j].astype(np.float64)
            caches = []
            for l in range(2):
                x, c = ot.layer_forward(x, P["layers"][l], shape.n_heads, True, shape.eps, keep=True)
                caches.append(c)
            dx = dys[j].astype(np.float64)
            for l in (1, 0):
                dx, G = ot.layer_backward(dx, caches[l], P["layers"][l], shape.n_heads)
                Gsum[l] = G if Gsum[l] is None else {k: Gsum[l][k] + G[k] for k in G}
        for l in range(2):
            got, m1, v1 = read_layer(m, 1, l), read_layer(m, 2, l), read_layer(m, 3, l)
            for k in Gsum[l]:
                gmean = 0.5 * Gsum[l][k]
                th1, mo, vo = ot.adam_step(P["layers"][l][k], 0.0, 0.0, gmean, 1, lr=1e-3)
                assert rel_err(m1[k], mo) < 1e-4 and rel_err(v1[k], vo) < 2e-4, (l, k)
                big = np.abs(gmean) > 1e-3 * np.abs(gmean).max()
                upd = got[k].astype(np.float64) - P["layers"][l][k]
                assert np.abs(upd - (th1 - P["layers"][l][k]))[big].max() < 0.05 * 1e-3, (l, k)
            assert not any(np.any(v) for v in read_layer(m, 0, l).values())      # accumulators cleared
        _, steps = m.ctx.pf_ctx_train_state()
        assert steps == 1
        with pytest.raises(pf.PipeFillError) as e:
            m.ctx.pf_main_stage_step(pf.PF_INSTR_OPT, 0, None, st.cuda_stream)
        assert e.value.code == pf.PF_ERR_ARG
    finally:
        m.close()


def _moments(m, n_layers):
    """The stage's optimizer state as the library strings it: per layer, first then second moments."""
    pf, dev = _mods()
    md32 = pf.pf_model_desc.from_buffer_copy(m.md)
    md32.dtype = pf.PF_DTYPE_F32
    size, _ = pf.pf_layer_blob_layout(md32)
    out = []
    for l in range(n_layers):
        for what in (2, 3):
            buf = torch.empty(size, dtype=torch.uint8, device="cuda")
            m.ctx.pf_ctx_read_params(what, l, buf.data_ptr(), size)
            m.ctx.pf_ctx_sync()
            out.append(buf.cpu().numpy())
    return np.concatenate(out)


def test_main_stage_offload_round_trip():
    """Optimizer-state offload of the emulated main stage: slices leave with the forwards, what has left is
    overwritten on the device during the windows, everything is back for the optimizer update.  The bytes
    that reach the host are exactly the state of the iteration before, and the training run is the same as
    one without offload (up to the summation order of the gradient atomics)."""
    import ctypes as C
    pf, dev = _mods()
    shape = synth.ModelShape(2, 128, 2, 256, 64, 2, 0, True, "bf16")
    params = synth.make_model_params(shape, seed=47, std=0.08)
    p, mm, stage, tf, tb = 4, 4, 1, 3_000_000, 6_000_000
    windows = pf.pf_schedule_1f1b(p, mm, stage, tf, tb, 1 << 30, True, 0)
    runs = {}
    for mode in ("plain", "offload"):
        m = dev.DeviceModel(shape, params, g=mm, training=True, adam=pf.pf_adam(1e-3, 0.9, 0.999, 1e-8, 1))
        try:
            io = dev.storage_tensor(synth.make_hidden(shape, seed=190), m.md)
            S = m.ctx.pf_main_opt_state_bytes()
            md32 = pf.pf_model_desc.from_buffer_copy(m.md)
            md32.dtype = pf.PF_DTYPE_F32
            assert S == 2 * 2 * pf.pf_layer_blob_layout(md32)[0]
            host = torch.zeros(S, dtype=torch.uint8, pin_memory=True)
            slices = []
            if mode == "offload":
                # 0.4 S per forward (so a slice straddles the two layers), everything may come back
                per = int(0.4 * S) // 256 * 256
                d2h = -(-per * 10**9 // tf)
                slices, extra = pf.pf_offload_plan(p, mm, stage, tf, 10**9, S, d2h, 10**12)
                assert slices[0] == slices[1] == per and sum(slices) == S // 256 * 256 and slices[3] == 0
                assert extra == [sum(slices)] * 3 + [0]
            m.ctx.pf_ctx_set_main_offload(2_000_000, host.data_ptr(), S, slices, scrub=True)
            st, main = torch.cuda.Stream(), torch.cuda.Stream()
            cursor = C.c_int32(0)
            states, stats = [], []
            for _ in range(3):
                stats.append(pf.pf_timeline_run(None, m.ctx, io.data_ptr(), p, mm, stage, tf, tb, windows, None, 0, None,
                                                cursor, st.cuda_stream, main.cuda_stream))
                states.append(_moments(m, 2))
                if mode == "offload" and len(states) >= 2:
                    n = sum(slices)
                    # what reached the host during this iteration is the state the iteration before left behind
                    assert np.array_equal(host.numpy()[:n], states[-2][:n])
            _, steps = m.ctx.pf_ctx_train_state()
            assert steps == 3
            assert all(s["offloaded_bytes"] == sum(slices) for s in stats)
            assert all(s["iter_ns"] >= 2_000_000 for s in stats)
            runs[mode] = (states, [read_layer(m, 1, l) for l in range(2)])
        finally:
            m.close()
    a, b = runs["plain"], runs["offload"]
    for it in range(3):
        fa, fb = a[0][it].view(np.float32), b[0][it].view(np.float32)
        assert np.isfinite(fb).all()
        assert rel_err(fb, fa) < 1e-3, it
    for l in range(2):
        for k in a[1][l]:
            assert np.isfinite(b[1][l][k]).all()
            assert np.abs(b[1][l][k] - a[1][l][k]).max() < 2e-4, (l, k)      # three steps of at most lr = 1e-3 each


def test_main_offload_argument_errors():
    pf, dev = _mods()
    shape = synth.ModelShape(1, 64, 2, 128, 64, 1, 0, True, "bf16")
    m = dev.DeviceModel(shape, synth.make_model_params(shape, seed=5, std=0.05), training=True)
    try:
        S = m.ctx.pf_main_opt_state_bytes()
        host = torch.zeros(S, dtype=torch.uint8, pin_memory=True)
        for args, code in [((0, host.data_ptr(), S, [S + 256]), pf.PF_ERR_ARG), ((0, host.data_ptr(), S, [6]), pf.PF_ERR_ARG),
                           ((0, host.data_ptr(), 100, [256]), pf.PF_ERR_CAPACITY), ((0, None, S, [256]), pf.PF_ERR_ARG),
                           ((-1, host.data_ptr(), S, [256]), pf.PF_ERR_ARG)]:
            with pytest.raises(pf.PipeFillError) as e:
                m.ctx.pf_ctx_set_main_offload(*args)
            assert e.value.code == code, args
        # a slice count that does not match the timeline's m is refused by the timeline
        import ctypes as C
        m.ctx.pf_ctx_set_main_offload(0, host.data_ptr(), S, [256, 256])
        io = dev.storage_tensor(synth.make_hidden(shape, seed=1), m.md)
        st, main = torch.cuda.Stream(), torch.cuda.Stream()
        windows = pf.pf_schedule_1f1b(2, 3, 0, 10**6, 10**6, 1 << 30, True, 0)
        with pytest.raises(pf.PipeFillError) as e:
            pf.pf_timeline_run(None, m.ctx, io.data_ptr(), 2, 3, 0, 10**6, 10**6, windows, None, 0, None, C.c_int32(0),
                               st.cuda_stream, main.cuda_stream)
        assert e.value.code == pf.PF_ERR_ARG
        m.ctx.pf_ctx_set_main_offload(-1)          # phase off again
    finally:
        m.close()


# the MFMA kernels (bf16, d_head 64 / 128) walk tiles of 64 rows in blocks of 128: one row, one tile, one row more
# than a tile, a ragged multiple of the block; the other cases run on the generic kernels
ATT_BWD = [("bf16", 2, 200, 3, 64), ("bf16", 1, 321, 2, 128), ("bf16", 2, 64, 2, 64), ("bf16", 1, 130, 2, 16),
           ("f32", 2, 100, 2, 32), ("f32", 1, 70, 1, 64), ("bf16", 1, 1, 1, 64), ("bf16", 1, 65, 1, 128),
           ("bf16", 1, 129, 2, 64),
           # sizes at which the causal kernels hand the blocks of every other group of 32 units out in reverse order
           ("bf16", 2, 1024, 16, 64), ("bf16", 1, 2048, 16, 128)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype,B,S,h,dh", ATT_BWD)
def test_attention_backward_kernel(dtype, B, S, h, dh, causal):
    pf, dev = _mods()
    md = pf.pf_model_desc()
    md.dtype = pf.PF_DTYPE_BF16 if dtype == "bf16" else pf.PF_DTYPE_F32
    d = h * dh
    rng = np.random.default_rng(S * 7 + dh)
    rnd = lambda *s: (synth.round_to_bf16(rng.standard_normal(s).astype(np.float32)) if dtype == "bf16"
                      else rng.standard_normal(s).astype(np.float32))
    qkv, dout = rnd(B, S, 3 * d), rnd(B, S, d)
    dq_, do_ = dev.storage_tensor(qkv, md), dev.storage_tensor(dout, md)
    out = dev.empty_storage((B, S, d), md)
    dqkv = dev.empty_storage((B, S, 3 * d), md)
    lse = torch.empty((B, h, S), dtype=torch.float32, device="cuda")
    dsum = torch.empty((B, h, S), dtype=torch.float32, device="cuda")
    pf.pf_op_attention(md.dtype, dq_.data_ptr(), out.data_ptr(), B, S, h, dh, causal, lse.data_ptr())
    pf.pf_op_attention_bwd(md.dtype, dq_.data_ptr(), out.data_ptr(), do_.data_ptr(), lse.data_ptr(), dsum.data_ptr(),
                           dqkv.data_ptr(), B, S, h, dh, causal)
    torch.cuda.synchronize()
    q64 = qkv.astype(np.float64)
    q, k, v = (ot.split_heads(q64[..., i * d:(i + 1) * d], h) for i in range(3))
    A = ot.attention_probs(q, k, causal)
    do = ot.split_heads(dout.astype(np.float64), h)
    dA = do @ v.transpose(0, 1, 3, 2)
    dv = A.transpose(0, 1, 3, 2) @ do
    ds = A * (dA - (dA * A).sum(-1, keepdims=True))
    dq = ds @ k / np.sqrt(dh)
    dk = ds.transpose(0, 1, 3, 2) @ q / np.sqrt(dh)
    got = dev.read_storage(dqkv, md)
    tol = 2e-2 if dtype == "bf16" else 1e-4
    for i, ref in enumerate((dq, dk, dv)):
        assert rel_err(got[..., i * d:(i + 1) * d], ot.merge_heads(ref)) < tol, "qkv"[i]


# d covers every workgroup shape of the kernel: 1 wave (<= 512), 2 waves (<= 1024), 4 waves with 1, 2 and 4
# column groups per thread (<= 2048, <= 4096, <= 8192); rows cover fewer rows than workgroups, a ragged
# multiple, and more rows than the 512 partial rows
LN_BWD = [("f32", 5, 64), ("f32", 70, 520), ("bf16", 3, 256), ("bf16", 700, 768), ("bf16", 1500, 1024),
          ("bf16", 130, 1536), ("bf16", 600, 2048), ("bf16", 90, 2560), ("bf16", 520, 4096), ("bf16", 33, 4104),
          ("bf16", 64, 8192)]


@pytest.mark.parametrize("with_resid", [False, True])
@pytest.mark.parametrize("dtype,rows,d", LN_BWD)
def test_layernorm_backward_kernel(dtype, rows, d, with_resid):
    pf, dev = _mods()
    md = pf.pf_model_desc()
    md.dtype = pf.PF_DTYPE_BF16 if dtype == "bf16" else pf.PF_DTYPE_F32
    rng = np.random.default_rng(rows * 31 + d)
    rnd = lambda *s: (synth.round_to_bf16(rng.standard_normal(s).astype(np.float32)) if dtype == "bf16"
                      else rng.standard_normal(s).astype(np.float32))
    x, dy, res = rnd(rows, d) * 1.5 + 0.3, rnd(rows, d), rnd(rows, d)
    if dtype == "bf16":
        x = synth.round_to_bf16(x.astype(np.float32))
    g = (1.0 + 0.1 * rnd(d)).astype(np.float32)
    if dtype == "bf16":
        g = synth.round_to_bf16(g)
    b = np.zeros(d, np.float32)
    dx_, ddy, dg_, dres = (dev.storage_tensor(a, md) for a in (x, dy, g, res))
    db_ = dev.storage_tensor(b, md)
    y = dev.empty_storage((rows, d), md)
    mean = torch.empty(rows, dtype=torch.float32, device="cuda")
    rstd = torch.empty(rows, dtype=torch.float32, device="cuda")
    pf.pf_op_layernorm(md.dtype, dx_.data_ptr(), dg_.data_ptr(), db_.data_ptr(), y.data_ptr(), rows, d, 1e-5,
                       mean.data_ptr(), rstd.data_ptr())
    dxo = dev.empty_storage((rows, d), md)
    # dg / db are accumulated into: start from a known value
    acc_g = torch.full((d,), 2.0, dtype=torch.float32, device="cuda")
    acc_b = torch.full((d,), -1.0, dtype=torch.float32, device="cuda")
    partial = torch.empty(512 * 2 * d, dtype=torch.float32, device="cuda")
    pf.pf_op_layernorm_bwd(md.dtype, ddy.data_ptr(), dx_.data_ptr(), dg_.data_ptr(), mean.data_ptr(), rstd.data_ptr(),
                           dres.data_ptr() if with_resid else None, dxo.data_ptr(), acc_g.data_ptr(), acc_b.data_ptr(),
                           partial.data_ptr(), rows, d)
    torch.cuda.synchronize()
    x64 = x.astype(np.float64)
    _, xhat, rs = ot.layer_norm(x64, g.astype(np.float64), b.astype(np.float64), 1e-5)
    dx_ref, dg_ref, db_ref = ot.layer_norm_backward(dy.astype(np.float64), xhat, rs, g.astype(np.float64))
    if with_resid:
        dx_ref = dx_ref + res
    tol = 2e-2 if dtype == "bf16" else 1e-4
    assert rel_err(dev.read_storage(dxo, md), dx_ref) < tol
    assert rel_err(acc_g.cpu().numpy() - 2.0, dg_ref) < (1e-3 if dtype == "bf16" else 1e-4)
    assert rel_err(acc_b.cpu().numpy() + 1.0, db_ref) < (1e-3 if dtype == "bf16" else 1e-4)


@pytest.mark.parametrize("dtype,R,Cn", [("bf16", 64, 64), ("bf16", 200, 136), ("bf16", 8, 8), ("bf16", 1000, 3072),
                                         ("bf16", 37, 50), ("bf16", 129, 72), ("f32", 100, 36), ("f32", 64, 200)])
def test_transpose_kernel(dtype, R, Cn):
    """Byte work: exact.  Shapes with both sides a multiple of 8 take the vectorised kernel (tiles inside, on the
    edge and ragged in both directions), the others the element-wise one.  With an accumulator the column sums
    come along (fp32 atomics: compared within fp32 rounding of a sum of R terms)."""
    pf, dev = _mods()
    rng = np.random.default_rng(R * 13 + Cn)
    if dtype == "bf16":
        vals = synth.round_to_bf16(rng.standard_normal((R, Cn)).astype(np.float32))
        a = (vals.view(np.uint32) >> 16).astype(np.uint16)
        code = pf.PF_DTYPE_BF16
    else:
        vals = a = rng.standard_normal((R, Cn)).astype(np.float32)
        code = pf.PF_DTYPE_F32
    src = dev.to_device(a)
    for with_sum in (False, True):
        dst = torch.zeros((Cn, R), dtype=src.dtype, device="cuda")
        acc = torch.full((Cn,), 3.0, dtype=torch.float32, device="cuda")
        pf.pf_op_transpose(code, src.data_ptr(), dst.data_ptr(), R, Cn, acc.data_ptr() if with_sum else None)
        torch.cuda.synchronize()
        got = dst.cpu().numpy()
        assert np.array_equal(got.view(a.dtype) if got.dtype != a.dtype else got, a.T)
        if with_sum:
            ref = vals.astype(np.float64).sum(axis=0)
            scale = np.abs(vals.astype(np.float64)).sum(axis=0).max()
            assert np.abs(acc.cpu().numpy() - 3.0 - ref).max() < 1e-6 * scale + 1e-6
        else:
            assert bool((acc == 3.0).all())


# (M, N, K): whole tiles, ragged edges in both directions (multiples of 8 only), one K step, K split over
# workgroups (small M x N with long K), more tiles than resident workgroups
GEMM_TN = [(128, 128, 64), (256, 384, 512), (200, 136, 192), (8, 8, 64), (72, 1000, 320), (256, 256, 4096),
           (128, 128, 8192), (1536, 1280, 256)]


@pytest.mark.parametrize("with_colsum", [False, True])
@pytest.mark.parametrize("M,N,K", GEMM_TN)
def test_gemm_tn_kernel(M, N, K, with_colsum):
    """Weight-gradient GEMM on K-major operands against the plain float64 product; C and the column sums are
    accumulated into, so both start from known non-zero values."""
    pf, dev = _mods()
    rng = np.random.default_rng(M * 3 + N * 5 + K)
    A = synth.round_to_bf16(rng.standard_normal((K, M)).astype(np.float32))
    Bm = synth.round_to_bf16((rng.standard_normal((K, N)) * 0.5).astype(np.float32))
    md = pf.pf_model_desc()
    md.dtype = pf.PF_DTYPE_BF16
    dA, dB = dev.storage_tensor(A, md), dev.storage_tensor(Bm, md)
    C0 = rng.standard_normal((M, N)).astype(np.float32)
    dC = dev.to_device(C0)
    acc = torch.full((M,), 0.5, dtype=torch.float32, device="cuda")
    for rep in range(2):       # twice: accumulation, and the second call finds LDS and C as the first left them
        pf.pf_op_gemm_tn(pf.PF_DTYPE_BF16, dA.data_ptr(), dB.data_ptr(), dC.data_ptr(), M, N, K,
                         acc.data_ptr() if with_colsum else None)
    torch.cuda.synchronize()
    ref = C0.astype(np.float64) + 2.0 * (A.astype(np.float64).T @ Bm.astype(np.float64))
    scale = np.abs(A.astype(np.float64)).T @ np.abs(Bm.astype(np.float64))
    got = dC.cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= 5e-5 * scale.max() + 1e-5        # fp32 accumulation of K exact bf16 products
    if with_colsum:
        cref = 0.5 + 2.0 * A.astype(np.float64).sum(axis=0)
        assert np.abs(acc.cpu().numpy() - cref).max() <= 5e-5 * np.abs(A).sum(axis=0).max() + 1e-5
    else:
        assert bool((acc == 0.5).all())


# Tokens that are no whole number of K steps: less than one step, one to ten steps and a rest, slices of K whose last one ends in
# a rest; ragged edges.  slices: how many the launch takes.
GEMM_TN_EIGHTS = [(128, 128, 8, 1), (200, 136, 72, 1), (72, 1000, 200, 2), (136, 2000, 200, 1), (256, 384, 600, 4), (8, 8, 328, 2), (512, 1280, 1000, 2),
                  (1536, 2120, 4040, 2)]


@pytest.mark.parametrize("with_colsum", [False, True])
@pytest.mark.parametrize("M,N,K,slices", GEMM_TN_EIGHTS)
def test_gemm_tn_kernel_ends_inside_a_step(M, N, K, slices, with_colsum):
    """As test_gemm_tn_kernel, with LDS left full of NaN: rows past the last token must not come from there, nor from what follows
    the operands in memory (NaN as well)."""
    import ctypes as ct
    pf, dev = _mods()
    assert pf.lib.pf_gemm_tn_slices(ct.c_int64(M), ct.c_int64(N), ct.c_int64(K)) == slices
    f = pf.lib.pf_gemm_tn_eights
    f.restype, f.argtypes = ct.c_int32, [ct.c_void_p] * 4 + [ct.c_int64] * 3 + [ct.c_void_p]
    rng = np.random.default_rng(M + 2 * N + K)
    A = synth.round_to_bf16(rng.standard_normal((K, M)).astype(np.float32))
    B = synth.round_to_bf16((rng.standard_normal((K, N)) * 0.5).astype(np.float32))

    def on_gpu(a):      # 64 rows of NaN behind it
        t = torch.full((K + 64, a.shape[1]), float("nan"), dtype=torch.bfloat16, device="cuda")
        t[:K] = torch.from_numpy(a).cuda().to(torch.bfloat16)
        return t
    dA, dB = on_gpu(A), on_gpu(B)
    C0 = rng.standard_normal((M, N)).astype(np.float32)
    dC = dev.to_device(C0)
    acc = torch.full((M,), 0.5, dtype=torch.float32, device="cuda")
    bad = torch.full((1024, 2048), float("nan"), dtype=torch.bfloat16, device="cuda")
    sink = torch.zeros(2048, 2048, device="cuda")
    for _ in range(2):
        pf.pf_op_gemm_tn(pf.PF_DTYPE_BF16, bad.data_ptr(), bad.data_ptr(), sink.data_ptr(), 2048, 2048, 1024)
        assert f(dA.data_ptr(), dB.data_ptr(), dC.data_ptr(), acc.data_ptr() if with_colsum else None, M, N, K, None) == 0
    torch.cuda.synchronize()
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    scale = np.abs(A64).T @ np.abs(B64)
    assert np.abs(dC.cpu().numpy() - C0 - 2.0 * (A64.T @ B64)).max() <= 5e-5 * scale.max() + 1e-5      # as in test_gemm_tn_kernel
    if with_colsum:
        assert np.abs(acc.cpu().numpy() - 0.5 - 2.0 * A64.sum(axis=0)).max() <= 5e-5 * np.abs(A64).sum(axis=0).max() + 1e-5
    else:
        assert bool((acc == 0.5).all())


@pytest.mark.parametrize("M,N,K", [((1 << 23) + 8, 8, 128), (8, (1 << 23) + 8, 64)])
def test_gemm_tn_results_of_eight_million_rows_or_columns(M, N, K):
    """Rows of an operand long enough that 64 of them pass 2^31 bytes: C and the column sums at both ends of the long side and in
    its middle, against float64.  Each call adds to known values, twice."""
    pf, dev = _mods()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M % 1000 + N)
    A = torch.randn(K, M, device="cuda", generator=gen).to(torch.bfloat16)
    B = torch.randn(K, N, device="cuda", generator=gen).to(torch.bfloat16)
    C = torch.full((M, N), 0.25, device="cuda")
    cs = torch.full((M,), 0.5, device="cuda")
    for _ in range(2):
        pf.pf_op_gemm_tn(pf.PF_DTYPE_BF16, A.data_ptr(), B.data_ptr(), C.data_ptr(), M, N, K, cs.data_ptr())
    torch.cuda.synchronize()
    long = max(M, N)
    for first in (0, long // 2 - 100, long - 300):
        a = A[:, first:first + 300].double() if M > N else A.double()
        b = B[:, first:first + 300].double() if N > M else B.double()
        got = C[first:first + 300] if M > N else C[:, first:first + 300]
        scale = float((a.abs().t() @ b.abs()).max())
        assert float((got.double() - 0.25 - 2 * (a.t() @ b)).abs().max()) <= 5e-5 * scale      # as in test_gemm_tn_kernel
        s = cs[first:first + 300] if M > N else cs
        assert float((s.double() - 0.5 - 2 * a.sum(0)).abs().max()) <= 5e-5 * float(a.abs().sum(0).max())


def test_gemm_tn_argument_errors():
    pf, dev = _mods()
    t = torch.zeros(1 << 16, dtype=torch.int16, device="cuda")
    c = torch.zeros(1 << 16, dtype=torch.float32, device="cuda")
    for M, N, K, dt in [(12, 8, 64, pf.PF_DTYPE_BF16), (8, 20, 64, pf.PF_DTYPE_BF16), (8, 8, 96, pf.PF_DTYPE_BF16),
                        (8, 8, 64, pf.PF_DTYPE_F32), (0, 8, 64, pf.PF_DTYPE_BF16)]:
        with pytest.raises(pf.PipeFillError) as e:
            pf.pf_op_gemm_tn(dt, t.data_ptr(), t.data_ptr(), c.data_ptr(), M, N, K)
        assert e.value.code == pf.PF_ERR_ARG
    with pytest.raises(pf.PipeFillError):
        pf.pf_op_gemm_tn(pf.PF_DTYPE_BF16, t.data_ptr() + 2, t.data_ptr(), c.data_ptr(), 8, 8, 64)


def test_doubling_probe_against_the_emulated_stage():
    """Sec. 4.2, bubble characterisation: the probe with the stage's forward / backward kernels really running and
    the other stages simulated from the measured t_f / t_b.  The estimates are powers of two times the first wait;
    against the closed-form windows of the same schedule: no estimate is harmless beyond what the stage's idle time
    allows (each at most its own window plus the slack of the later ones, the sum at most the idle total), and the
    long fwd-bwd window is found to within the probe's factor of two, where the host simulation of the same probe,
    fed the measured times, puts it up to one doubling."""
    pf, dev = _mods()
    shape = synth.ModelShape(3, 1024, 16, 4096, 1024, 4, 0, True, "bf16")     # t_f about 1 ms, t_b about 3 ms
    params = synth.make_model_params(shape, seed=47)
    p, mm, stage = 4, 6, 1
    m = dev.DeviceModel(shape, params, g=min(p - stage, mm), training=True)
    try:
        x = dev.storage_tensor(synth.make_hidden(shape, seed=61), m.md)
        st = torch.cuda.Stream()
        import time
        # t_f, t_b as the probe itself sees an instruction: launch to the end of a host synchronisation, so that the
        # simulated neighbours are as fast as the real stage and the schedule is balanced
        tfs, tbs = [], []
        for _ in range(7):
            torch.cuda.synchronize()
            t0 = time.perf_counter_ns()
            m.ctx.pf_main_stage_step(pf.PF_INSTR_FWD, 0, x.data_ptr(), st.cuda_stream)
            st.synchronize()
            t1 = time.perf_counter_ns()
            m.ctx.pf_main_stage_step(pf.PF_INSTR_BWD, 0, x.data_ptr(), st.cuda_stream)
            st.synchronize()
            t2 = time.perf_counter_ns()
            tfs.append(t1 - t0)
            tbs.append(t2 - t1)
        tf, tb = sorted(tfs)[3], sorted(tbs)[3]
        assert tf > 100_000 and tb > tf
        first = tf // 4
        tol = 30_000                                           # 3 %: kernel and host-synchronisation noise
        est, base = pf.pf_probe_bubbles_live(m.ctx, x.data_ptr(), p, mm, stage, tf, tb, first, tol, st.cuda_stream)
        windows = pf.pf_schedule_1f1b(p, mm, stage, tf, tb, 1 << 30, True, 0)
        durs = [w["dur"] for w in windows]
        assert len(est) == len(durs)
        ideal = (mm + p - 1) * (tf + tb)
        assert abs(base - ideal) < 0.08 * ideal                # the undisturbed period is the schedule's iteration time
        slack = 0.06 * ideal                                   # what the tolerance lets through, plus timing noise
        assert sum(est) <= sum(durs) + slack
        for k, e in enumerate(est):
            assert e == 0 or (e % first == 0 and (e // first) & (e // first - 1) == 0)      # first * 2^i
            assert e <= sum(durs[k:]) + slack, (k, est, durs)
        # the long first window (the fwd-bwd bubble) is found to within the probe's factor of two, and the host
        # simulation of the same probe on the measured times agrees on it up to one doubling; the later, short
        # windows share what slack the first estimate left, which run-to-run noise distributes differently
        assert est[0] > durs[0] // 2 - slack
        host = pf.pf_probe_bubbles(p, mm, stage, tf, tb, first, tol)
        assert est[0] in (host[0], 2 * host[0], host[0] // 2), (est, host)
    finally:
        m.close()
