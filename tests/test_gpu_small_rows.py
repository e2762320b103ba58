"""The five-launch layers (few activation rows) and the one-launch prefix
hand-off, at the edges of their tiles, against the fp64 oracle and exact copies.

Tolerance of the denoise cases: every product's inputs are rounded to bf16
(relative 2^-9 each); over two layers and two steps with amplified gates the
error measured on the eight-launch layers is 0.1-2e-3, so 4e-3 per rollout.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import Inputs, assert_bf16, device_view_i16, make_expert, path_env, run, run_env, torch_cuda

pytestmark = pytest.mark.gpu
REL, ABS = 4e-3, 4e-2

SHAPES = {
    # contraction of 8 steps (no 32-step turns), an action width that is no multiple of 8, two heads per 128 columns
    "w256": synth.Dims(n_layers=2, width=256, n_heads=4, n_kv_heads=1, head_dim=64, mlp_dim=512, action_dim=7, horizon=10),
    # Dh 128, contractions of 16 and 40 steps
    "w512": synth.Dims(n_layers=2, width=512, n_heads=10, n_kv_heads=1, head_dim=128, mlp_dim=1280, action_dim=24, horizon=17),
    # narrow, with a wide MLP: gate/up on the rings past 48 and 272 rows; and widths whose contraction is 24 steps
    "w256f": synth.Dims(n_layers=2, width=256, n_heads=4, n_kv_heads=1, head_dim=64, mlp_dim=12288, action_dim=7, horizon=10),
    "w768": synth.Dims(n_layers=2, width=768, n_heads=4, n_kv_heads=1, head_dim=64, mlp_dim=3072, action_dim=14, horizon=16),
    "w1024": synth.Dims(n_layers=2, width=1024, n_heads=8, n_kv_heads=1, head_dim=256, mlp_dim=4096, action_dim=32, horizon=50),
}
LENS = [70, 0, 33, 1, 64, 31, 32, 69, 63, 65]


def _case(shape, batch, n_fixed=0, n_corr=0, prefix=70):
    lens = tuple(min(LENS[b % len(LENS)], prefix) for b in range(batch))
    wl = synth.Workload("small-%s-b%d" % (shape, batch), SHAPES[shape], prefix=prefix, batch=batch, n_steps=2,
                        n_fixed=n_fixed, dtype="bf16", prefix_len=lens, mod_gain=8.0)
    inp = Inputs(wl)
    corr = synth.normal_f32(wl.seed, "item", 1.0, (batch, n_corr, wl.dims.width)) if n_corr else None
    return wl, inp, corr


def _oracle(wl, inp, corr, t0=False):
    return oracle.denoise(oracle.Expert(wl.dims, inp.weights), inp.noise, inp.K, inp.V, inp.prefix_len, wl.n_steps,
                          committed=inp.committed, n_fixed=wl.n_fixed, corr=corr, committed_t0=t0)


# rows: 10, 30, 130, 510 | 17, 34 .. 289 | 50, 100, 200, 250, 300, 500 and with correction tokens 53, 159, 424
@pytest.mark.parametrize("shape,batch,n_fixed,n_corr,t0", [
    ("w256", 1, 0, 0, False), ("w256", 3, 4, 0, True), ("w256", 13, 0, 3, False), ("w256", 51, 2, 0, False),
    ("w256f", 4, 0, 0, False), ("w256f", 11, 2, 0, True), ("w256f", 27, 0, 3, False), ("w256f", 51, 0, 0, False),
    ("w768", 1, 0, 0, False), ("w768", 17, 3, 0, True), ("w768", 31, 0, 0, False),
    ("w512", 1, 0, 0, False), ("w512", 4, 3, 2, True), ("w512", 17, 0, 0, False),
    ("w1024", 1, 0, 0, False), ("w1024", 1, 10, 3, True), ("w1024", 2, 0, 0, False), ("w1024", 3, 7, 3, False),
    ("w1024", 4, 0, 0, False), ("w1024", 5, 7, 0, True), ("w1024", 6, 0, 0, False), ("w1024", 8, 5, 3, True),
    ("w1024", 10, 0, 0, False)])
def test_small_rows_match_oracle(shape, batch, n_fixed, n_corr, t0):
    wl, inp, corr = _case(shape, batch, n_fixed, n_corr)
    print("case", wl.name, n_fixed, n_corr, t0, flush=True)
    ae = make_expert(wl, inp.weights, max_batch=batch + 1, max_prefix=wl.prefix + 5, max_corr=n_corr)
    try:
        ae.set_committed_t0(t0)
        kw = dict(prefix_len=inp.prefix_len, committed=inp.committed, n_fixed=n_fixed, corr=corr)
        got = run(ae, inp.K, inp.V, inp.noise, wl.n_steps, **kw)
        assert_bf16(got, _oracle(wl, inp, corr, t0), wl.name, reg_rel=REL, reg_abs=ABS)
        assert np.array_equal(got, run(ae, inp.K, inp.V, inp.noise, wl.n_steps, **kw))
        if n_fixed:
            assert np.array_equal(got[:, :n_fixed], inp.committed.astype(np.float64))
    finally:
        ae.close()


# 1, 2, 4 and 8 key ranges, some without keys
@pytest.mark.parametrize("shape,batch,lens", [("w1024", 4, [300, 0, 33, 299]), ("w1024", 3, [1100, 0, 545]),
                                              ("w1024", 2, [700, 130]), ("w1024", 1, [700]), ("w512", 1, [1500])])
def test_small_rows_key_ranges(shape, batch, lens):
    wl = synth.Workload("ranges-%s-b%d" % (shape, batch), SHAPES[shape], prefix=lens[0], batch=batch, n_steps=2, n_fixed=0,
                        dtype="bf16", prefix_len=tuple(lens), mod_gain=8.0)
    inp = Inputs(wl)
    print("case", wl.name, lens, flush=True)
    ae = make_expert(wl, inp.weights)
    try:
        got = run(ae, inp.K, inp.V, inp.noise, wl.n_steps, prefix_len=inp.prefix_len)
        assert_bf16(got, _oracle(wl, inp, None), wl.name, reg_rel=REL, reg_abs=ABS)
    finally:
        ae.close()


# (rollouts, tokens): a long prefix for three rollouts goes to the eight-launch layers, for one rollout, and a short one, not
@pytest.mark.parametrize("batch,prefix,eight", [(3, 12800, True), (1, 12800, False), (3, 1600, False)])
def test_long_prefixes_take_the_faster_layers(batch, prefix, eight):
    d = synth.Dims(n_layers=1, width=512, n_heads=8, n_kv_heads=1, head_dim=256, mlp_dim=512, action_dim=7, horizon=50)
    lens = [prefix, prefix - 1, 77][:batch]
    wl = synth.Workload("long-b%d-p%d" % (batch, prefix), d, prefix=prefix, batch=batch, n_steps=2, n_fixed=0, dtype="bf16",
                        prefix_len=tuple(lens), mod_gain=8.0)
    inp = Inputs(wl)
    print("case", wl.name, flush=True)
    ae = make_expert(wl, inp.weights)
    try:
        got = run_env(ae, None, inp.K, inp.V, inp.noise, 2, prefix_len=lens)
        other = run_env(ae, "0", inp.K, inp.V, inp.noise, 2, prefix_len=lens)
        assert_bf16(got, _oracle(wl, inp, None), wl.name, reg_rel=REL, reg_abs=ABS)
        assert np.array_equal(got, other) == eight
    finally:
        ae.close()


def test_small_rows_after_longer_rows():
    """Own-key blocks keep what a longer call left behind their last key; it must not show."""
    wl, inp, corr = _case("w1024", 2, 0, 4)
    ae = make_expert(wl, inp.weights, max_corr=4)
    try:
        first = run(ae, inp.K, inp.V, inp.noise, wl.n_steps, prefix_len=inp.prefix_len)
        run(ae, inp.K, inp.V, inp.noise * np.float32(50), wl.n_steps, prefix_len=inp.prefix_len, corr=corr * np.float32(50))
        assert np.array_equal(first, run(ae, inp.K, inp.V, inp.noise, wl.n_steps, prefix_len=inp.prefix_len))
    finally:
        ae.close()


@pytest.mark.parametrize("shape,batch", [("w256", 3), ("w1024", 1)])
def test_single_launch_kernel_still_matches(shape, batch):
    """JPI_PERSIST=1 asks for the single-launch kernel, held to the same bars."""
    wl, inp, _ = _case(shape, batch)
    ae = make_expert(wl, inp.weights)
    try:
        got = run_env(ae, "1", inp.K, inp.V, inp.noise, wl.n_steps, prefix_len=inp.prefix_len)
        assert_bf16(got, _oracle(wl, inp, None), wl.name + "-single", reg_rel=REL, reg_abs=ABS)
    finally:
        ae.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Dh,B,P,Pmax", [(64, 1, 1, 40), (64, 3, 31, 31), (128, 2, 32, 45), (128, 1, 33, 33),
                                         (256, 2, 100, 131), (256, 3, 64, 64)])
def test_bind_prefix_copies(dtype, Dh, B, P, Pmax):
    """K, V and transposed V of every layer and rollout, exactly; then a hand-off in place gives the same V^T."""
    torch = torch_cuda()
    from paper_2607_12659_amd import jpi
    from paper_2607_12659_amd.expert import ActionExpert, to_device
    d = synth.Dims(n_layers=2, width=256, n_heads=4, n_kv_heads=1, head_dim=Dh, mlp_dim=512, action_dim=7, horizon=10)
    wl = synth.Workload("bind", d, prefix=P, batch=B, n_steps=1, n_fixed=0, dtype=dtype)
    K, V = synth.make_prefix(wl)
    ae = ActionExpert(d, dtype, B + 1, Pmax)
    try:
        ae.bind_prefix(to_device(K), to_device(V))
        torch.cuda.synchronize()
        _, kp, vp = jpi.jpi_prefix_buffers(ae.ctx)
        _, vt, ld = jpi.jpi_debug_prefix_vt(ae.ctx)
        w = 1 if dtype == "bf16" else 2  # 16-bit words per element

        def host(ptr, *shape):
            a = device_view_i16(ptr, shape[:-1] + (shape[-1] * w,)).cpu().numpy()
            return a.view(np.uint16 if dtype == "bf16" else np.float32)
        assert np.array_equal(host(kp, 2, B + 1, Pmax, Dh)[:, :B, :P], K)
        assert np.array_equal(host(vp, 2, B + 1, Pmax, Dh)[:, :B, :P], V)
        first = host(vt, 2, B + 1, Dh, ld)[:, :B, :, :P].copy()
        assert np.array_equal(first, V.transpose(0, 1, 3, 2))
        if P == Pmax:
            assert jpi.jpi_bind_prefix(ae.ctx, kp, vp, None, B, P) == jpi.JPI_OK
            torch.cuda.synchronize()
            assert np.array_equal(host(vt, 2, B + 1, Dh, ld)[:, :B, :, :P], first)
            assert np.array_equal(host(kp, 2, B + 1, Pmax, Dh)[:, :B, :P], K)
    finally:
        ae.close()


def test_bind_prefix_refuses_a_captured_stream():
    """The context notes batch and lengths on the host, which a replay would not do; the capture itself goes on."""
    torch = torch_cuda()
    from paper_2607_12659_amd import jpi
    from paper_2607_12659_amd.expert import to_device
    wl, inp, _ = _case("w256", 2)
    K, V = to_device(inp.K), to_device(inp.V)
    ae = make_expert(wl, inp.weights)
    try:
        want = run(ae, inp.K, inp.V, inp.noise, wl.n_steps, prefix_len=inp.prefix_len)
        t, graph, s = torch.zeros(4, device="cuda"), torch.cuda.CUDAGraph(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            t += 1
            st = jpi.jpi_bind_prefix(ae.ctx, K, V, [1, 2], 2, wl.prefix, s.cuda_stream)
        assert st == jpi.JPI_ERR_STATE
        graph.replay()
        torch.cuda.synchronize()
        assert t.tolist() == [1.0] * 4
        noise = to_device(np.ascontiguousarray(inp.noise, np.float32))
        out = ae.denoise(noise, wl.n_steps)  # the earlier binding holds
        ae.sync()
        assert np.array_equal(out.cpu().numpy().astype(np.float64), want)
    finally:
        ae.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_bind_prefix_from_any_element(dtype):
    """K and V that start one element past a 16-byte boundary give the same actions."""
    torch = torch_cuda()
    from paper_2607_12659_amd.expert import to_device
    d = synth.Dims(n_layers=2, width=256, n_heads=4, n_kv_heads=1, head_dim=64, mlp_dim=512, action_dim=7, horizon=10)
    wl = synth.Workload("bind", d, prefix=45, batch=2, n_steps=2, n_fixed=0, dtype=dtype)
    inp = Inputs(wl)
    ae = make_expert(wl, inp.weights)

    def moved(x):
        t = to_device(x)
        buf = torch.zeros(t.numel() + 1, dtype=t.dtype, device="cuda")
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)
    try:
        want = run(ae, inp.K, inp.V, inp.noise, 2)
        ae.bind_prefix(moved(inp.K), moved(inp.V))
        out = ae.denoise(to_device(np.ascontiguousarray(inp.noise, np.float32)), 2)
        ae.sync()
        assert np.array_equal(out.cpu().numpy().astype(np.float64), want)
    finally:
        ae.close()


def test_correction_inputs_from_any_element():
    """VLM state, compressed state and outputs that start off a 16-byte boundary."""
    torch = torch_cuda()
    import synth.correction as sc
    from gpu_util import Corr
    from paper_2607_12659_amd.expert import to_device
    wl = sc.CORR_WORKLOADS["corr40m-p816"].with_(batch=2, n_actions=5, vlm_tokens=130)
    x, acts = to_device(sc.make_vlm_state(wl)), to_device(np.ascontiguousarray(sc.make_actions(wl), np.float32))
    m = Corr(wl.dims, sc.make_corr_weights(wl), 2, 5, 130)

    def moved(t, copy=True):
        buf = torch.zeros(t.numel() + 1, dtype=t.dtype, device="cuda")
        if copy:
            buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)
    try:
        c = m.compress(x, 2, 130)
        item, conf = m.predict(c, acts, 2, 5)
        c2 = m.compress(x, 2, 130, out=moved(c, copy=False))
        item2, conf2 = m.predict(c2, moved(acts), 2, 5, item=moved(item, copy=False), conf=moved(conf, copy=False))
        assert torch.equal(c, c2) and torch.equal(item, item2) and torch.equal(conf, conf2)
        # an unaligned VLM state takes another product kernel: the same sums in another order
        c3 = m.compress(moved(x), 2, 130)
        assert float((c3 - c).norm() / c.norm()) <= 1e-3
    finally:
        m.close()


def test_correction_finalize_again_touches_nothing():
    """Finalizing without a new weight does no device work (calls in flight use the module's buffers): it can even be
    called while its stream is being captured.  A new weight is taken up by the next one."""
    torch = torch_cuda()
    import synth.correction as sc
    from gpu_util import Corr
    from paper_2607_12659_amd.expert import to_device
    wl = sc.CORR_WORKLOADS["corr-tiny"]
    w, x = sc.make_corr_weights(wl, std=0.08), to_device(sc.make_vlm_state(wl))
    m = Corr(wl.dims, w, wl.batch, 8, wl.vlm_tokens)
    try:
        first = m.compress(x, wl.batch, wl.vlm_tokens)
        t, graph, s = torch.zeros(4, device="cuda"), torch.cuda.CUDAGraph(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            t += 1
            st = m.jpi.jpi_corr_finalize_weights(m.ctx, s.cuda_stream)
        assert st == m.jpi.JPI_OK
        assert torch.equal(first, m.compress(x, wl.batch, wl.vlm_tokens))
        q = np.ascontiguousarray(-w["qformer.query"])
        assert m.jpi.jpi_corr_set_weight(m.ctx, "qformer.query", q, q.size, m.jpi.JPI_F32, 0) == m.jpi.JPI_OK
        assert m.jpi.jpi_corr_compress(m.ctx, x, wl.batch, wl.vlm_tokens, first.clone()) == m.jpi.JPI_ERR_STATE
        assert m.jpi.jpi_corr_finalize_weights(m.ctx) == m.jpi.JPI_OK
        other = Corr(wl.dims, {**w, "qformer.query": q}, wl.batch, 8, wl.vlm_tokens)
        got, want = m.compress(x, wl.batch, wl.vlm_tokens), other.compress(x, wl.batch, wl.vlm_tokens)
        assert torch.equal(got, want) and not torch.equal(got, first)
        other.close()
    finally:
        m.close()


# action rows 1, 75, 200 and 513 (past the five-launch layers); one token, a block's edge, several blocks; the tokens'
# product in one slice (few and very many tokens), four and two
@pytest.mark.parametrize("batch,n_actions,tokens", [(1, 1, 1), (3, 25, 33), (8, 25, 64), (2, 10, 130), (27, 19, 5),
                                                    (5, 3, 1003), (11, 2, 1499)])
def test_correction_rows_match_oracle(batch, n_actions, tokens):
    torch = torch_cuda()
    import synth.correction as sc
    from gpu_util import Corr
    from paper_2607_12659_amd.expert import to_device
    wl = sc.CORR_WORKLOADS["corr40m-p816"].with_(batch=batch, n_actions=n_actions, vlm_tokens=tokens)
    w = sc.make_corr_weights(wl)
    x, acts = sc.make_vlm_state(wl), sc.make_actions(wl)
    m = Corr(wl.dims, w, batch, n_actions, tokens + 7)
    try:
        print("case", batch, n_actions, tokens, flush=True)
        c = m.compress(to_device(x), batch, tokens)
        item, conf = m.predict(c, to_device(np.ascontiguousarray(acts, np.float32)), batch, n_actions)
        torch.cuda.synchronize()
        c, item = c.cpu().numpy().astype(np.float64), item.cpu().numpy().astype(np.float64)
        for b in sorted({0, batch // 2, batch - 1}):  # the oracle takes half a second a rollout
            c_o = oracle.correction.compress(wl.dims, w, x[b])
            i_o, f_o = oracle.correction.correct(wl.dims, w, c_o, acts[b])
            # measured on the eight-launch blocks: 7e-4 and 3.6e-3
            assert_bf16(c[b:b + 1], c_o[None], "state %d" % b, reg_rel=3e-3)
            assert_bf16(item[b:b + 1], i_o[None], "item %d" % b, reg_rel=1.5e-2)
            # each term of the confidence's dot product within the bf16 bar of the item
            assert abs(float(conf[b]) - f_o) <= 2e-2 * np.abs(oracle.widen(w["conf_head.w"])[0]).sum()
    finally:
        m.close()


@pytest.mark.parametrize("kappa", [1, 4, 16])
def test_small_rows_shift_cancels_the_activation(kappa):
    """These layers round u = h (1 + scale) and add the shift's part to the product, where the eight-launch layers round
    the sum: the error of a product is 2^-9 of r |h (1 + scale)|, not of the normalised value.  Here the shift of every
    norm takes away the part of h that all rows share, kappa times what is left.  Errors are taken of what the sublayers
    do to the actions: 4e-3 where every product's inputs are rounded to 2^-9 of themselves (as REL), kappa times that
    here (measured 3.1e-3, 6.3e-3 and 1.0e-2, against 2.3e-3, 2.3e-3 and 1.6e-3)."""
    d = synth.Dims(n_layers=2, width=512, n_heads=4, n_kv_heads=1, head_dim=64, mlp_dim=1024, action_dim=7, horizon=20)
    wl = synth.Workload("cancel", d, prefix=1, batch=3, n_steps=2, n_fixed=0, dtype="bf16", prefix_len=(0, 0, 0))
    inp = Inputs(wl)
    w = {k: v.copy() for k, v in inp.weights.items()}
    own = 1.0 / kappa  # rms of what differs between rows; the shared part has rms 1
    shared = synth.normal_f32(wl.seed, "shared", 1.0, (d.width,))
    w["action_in.w"] = synth.f32_to_bf16_bits(synth.normal_f32(wl.seed, "own", own / np.sqrt(7.0), (d.width, 7)))
    w["action_in.b"] = shared
    for l in range(2):
        for mod in ("attn_mod.b", "mlp_mod.b"):
            w["layers.%d.%s" % (l, mod)] = np.concatenate(
                [np.zeros(d.width), -shared / np.sqrt(1 + own * own), np.full(d.width, 0.5)]).astype(np.float32)
    print("case shift against activation", kappa, flush=True)
    ae = make_expert(wl, w)
    try:
        five = run_env(ae, None, inp.K, inp.V, inp.noise, 2, prefix_len=inp.prefix_len)
        eight = run_env(ae, "0", inp.K, inp.V, inp.noise, 2, prefix_len=inp.prefix_len)
    finally:
        ae.close()
    ref = oracle.denoise(oracle.Expert(d, w), inp.noise, inp.K, inp.V, inp.prefix_len, 2)
    for l in range(2):
        for mod in ("attn_mod", "mlp_mod"):  # no sublayer reaches the actions
            w["layers.%d.%s.b" % (l, mod)][2 * d.width:] = 0
            w["layers.%d.%s.w" % (l, mod)][2 * d.width:] = 0
    effect = np.linalg.norm(ref - oracle.denoise(oracle.Expert(d, w), inp.noise, inp.K, inp.V, inp.prefix_len, 2))
    err5, err8 = np.linalg.norm(five - ref) / effect, np.linalg.norm(eight - ref) / effect
    print("kappa %d, of the sublayers' effect: five-launch %.2e, eight-launch %.2e" % (kappa, err5, err8), flush=True)
    assert err8 <= REL and err5 <= kappa * REL


def _wide(B, lens, nH=1, Dh=256, horizon=20):
    """One layer, one step: a row's attention output reaches that row's action only."""
    d = synth.Dims(n_layers=1, width=512, n_heads=nH, n_kv_heads=1, head_dim=Dh, mlp_dim=512, action_dim=7, horizon=horizon)
    return synth.Workload("special", d, prefix=max(lens), batch=B, n_steps=1, n_fixed=0, dtype="bf16", prefix_len=tuple(lens),
                          mod_gain=8.0)


# key ranges of a 16-row tile by the rule: eight, four, two and one (short prefix, and many rollouts)
RANGES = [(1, [900]), (1, [500]), (1, [150]), (1, [20]), (25, [300])]


@pytest.mark.parametrize("B,lens", RANGES)
@pytest.mark.parametrize("what", ["query", "scale", "keys"])
def test_small_rows_keep_nan(B, lens, what):
    """A NaN in the query weights, in a modulation or in every prefix key makes every action of the rollout NaN
    (fmaxf drops a NaN score, so a row with nothing else has no maximum)."""
    wl = _wide(B, lens * B)
    inp = Inputs(wl)
    print("case NaN", what, B, lens, flush=True)
    ae = make_expert(wl, inp.weights)
    try:
        clean = run(ae, inp.K, inp.V, inp.noise, 1, prefix_len=inp.prefix_len)
        assert np.isfinite(clean).all()
        K = inp.K.copy()
        if what == "keys":
            K[:, 0] = 0x7fc0  # rollout 0
        else:
            name = "layers.0.q.w" if what == "query" else "layers.0.attn_mod.w"
            bad = inp.weights[name].copy()
            bad[0, 0] = 0x7fc0
            ae.load_weights({**inp.weights, name: bad})
        got = run(ae, K, inp.V, inp.noise, 1, prefix_len=inp.prefix_len)
    finally:
        ae.close()
    assert np.isnan(got[0]).all()
    if what == "keys":
        assert np.array_equal(got[1:], clean[1:])
    else:
        assert np.isnan(got).all()


@pytest.mark.parametrize("B,lens", RANGES)
@pytest.mark.parametrize("first,step", [(0, 1), (3, 1), (0, 2)])
def test_small_rows_infinite_scores(B, lens, first, step):
    """Prefix keys of infinite magnitude in one dimension (all, all but three, every other one): a row whose query is
    positive there gives them no weight, a negative one has no answer (NaN)."""
    wl = _wide(B, lens * B)
    inp = Inputs(wl)
    K = inp.K.copy()
    K[0, 0, first::step, 5] = 0xff80  # -inf, rollout 0
    print("case infinite scores", B, lens, first, step, flush=True)
    ae = make_expert(wl, inp.weights)
    try:
        got = run(ae, K, inp.V, inp.noise, 1, prefix_len=inp.prefix_len)
    finally:
        ae.close()
    with np.errstate(invalid="ignore"):
        ref = oracle.denoise(oracle.Expert(wl.dims, inp.weights), inp.noise, K, inp.V, inp.prefix_len, 1)
    bad = np.isnan(ref).any(axis=2)
    assert bad[0].any() and not bad[0].all() and not bad[1:].any()
    assert np.array_equal(np.isnan(got).all(axis=2), bad) and np.array_equal(np.isnan(got).any(axis=2), bad)
    ok = ~bad
    err = np.linalg.norm(got[ok] - ref[ok]) / np.linalg.norm(ref[ok])
    assert err <= REL, err


@pytest.mark.parametrize("B,lens", RANGES)
def test_small_rows_without_any_finite_score(B, lens):
    """Every score of every row overflows to -inf, its own keys' included: no answer, and none left from the call before."""
    wl = _wide(B, lens * B)
    inp = Inputs(wl)
    W, up, down = wl.dims.width, synth.f32_to_bf16_bits(np.float32([1e20]))[0], synth.f32_to_bf16_bits(np.float32([-1e20]))[0]
    w = {k: v.copy() for k, v in inp.weights.items()}
    # y = 1 in every column (scale -1, shift 1); q is 1e20 and k -1e20 in the dimension that rotates least
    w["layers.0.attn_mod.w"][:] = 0
    w["layers.0.attn_mod.b"][:] = np.repeat(np.float32([-1, 1, 1]), W)
    K = inp.K.copy()
    K[:], K[..., 127] = 0, down
    for name, v in (("q.w", up), ("k.w", down)):
        w["layers.0." + name][:] = 0
        w["layers.0." + name][127, 0] = v
    print("case no finite score", B, lens, flush=True)
    ae = make_expert(wl, inp.weights)
    try:
        assert np.isfinite(run(ae, inp.K, inp.V, inp.noise, 1, prefix_len=inp.prefix_len)).all()
        ae.load_weights(w)
        assert np.isnan(run(ae, K, inp.V, inp.noise, 1, prefix_len=inp.prefix_len)).all()
    finally:
        ae.close()


# what does not fit: the prefix's blocks (0.8 MB, allocated by the binding), the fragment-ordered weights (69 MB; the
# eight-launch layers' slices take 6.6 MB), the shift table of 100 steps (8.7 MB; their modulation table takes 6.2 MB)
@pytest.mark.parametrize("what,limit,steps", [("blocks", 1 << 19, 2), ("weights", 16 << 20, 2), ("shift table", 7 << 20, 100)])
def test_small_rows_without_memory(what, limit, steps):
    """The eight-launch layers run, with their results, where a buffer of the five-launch layers does not fit."""
    torch_cuda()
    from paper_2607_12659_amd import jpi
    from paper_2607_12659_amd.expert import to_device
    wl, inp, _ = _case("w1024", 4)
    K, V, noise = to_device(inp.K), to_device(inp.V), to_device(np.ascontiguousarray(inp.noise, np.float32))

    def denoise():
        out = ae.denoise(noise, steps)
        ae.sync()
        return out.cpu().numpy().astype(np.float64)

    print("case no memory for the", what, flush=True)
    ae = make_expert(wl, inp.weights, max_prefix=wl.prefix + 5)
    try:
        if what == "shift table":
            for env in ("0", None):  # every other buffer of either path is there
                run_env(ae, env, inp.K, inp.V, inp.noise, 2, prefix_len=inp.prefix_len)
        assert jpi.jpi_debug_set_alloc_limit(ae.ctx, limit) == jpi.JPI_OK
        ae.bind_prefix(K, V, inp.prefix_len)
        if what == "blocks":
            assert jpi.jpi_debug_set_alloc_limit(ae.ctx, 0) == jpi.JPI_OK
        got = denoise()
        assert np.array_equal(got, denoise())
        assert jpi.jpi_debug_set_alloc_limit(ae.ctx, 0) == jpi.JPI_OK
        with path_env("0"):
            eight = denoise()
        assert np.array_equal(got, eight)
        ae.bind_prefix(K, V, inp.prefix_len)  # the next binding has memory
        five = denoise()
        assert not np.array_equal(five, eight)
        if steps == 2:
            for out in (five, eight):
                assert_bf16(out, _oracle(wl, inp, None), wl.name, reg_rel=REL, reg_abs=ABS)
    finally:
        ae.close()
