"""Products and attention of more than 512 rows, at the edges of the ring tiles, of the key ranges and of the
grouped stores, against fp64 references of the same inputs."""
import numpy as np
import pytest

import oracle
import synth
import synth.vlm as synth_vlm
from gpu_util import Inputs, Vlm, assert_bf16, bf16_bits_to_f64, device_view_i16, make_expert, run, torch_cuda
from test_gpu_kernels import _attention, _bf16, _gemm

pytestmark = pytest.mark.gpu


# the tile the estimate picks on 256 units: 256 x 256, 128 x 256, 128 x 128, 128 x 64; row and column remainders
# of one and of all but one
@pytest.mark.parametrize("M,N,K,splitk", [(1126, 8192, 1024, 1), (1025, 8190, 128, 1), (816, 8100, 320, 1), (1409, 2049, 4096, 2),
                                          (1000, 2500, 4096, 1), (1025, 2431, 1024, 1), (1650, 1200, 1024, 1),
                                          (1537, 1217, 192, 1), (513, 2047, 2048, 4)])
def test_gemm_ring_tiles(M, N, K, splitk):
    from paper_2607_12659_amd import jpi
    rng = np.random.default_rng(M + N + K)
    A, W = _bf16(rng.normal(size=(M, K))), _bf16(rng.normal(size=(N, K)) * 0.02)
    got = _gemm(A, W, M, N, K, jpi.JPI_BF16, splitk)
    a, w = oracle.widen(A), oracle.widen(W)
    # fp32 sums of at most 4096 exact products: 1e-5 of the sum of their magnitudes, as for the other shapes
    assert np.all(np.abs(got - a @ w.T) <= 1e-5 * (np.abs(a) @ np.abs(w).T) + 1e-6)


# operands that start one element past a 16-byte boundary, at sizes that take each ring tile when aligned
@pytest.mark.parametrize("M,N,K,splitk", [(150, 1024, 4096, 4), (400, 2560, 1024, 1), (400, 8192, 1024, 1), (816, 2560, 2048, 1),
                                          (1126, 8192, 1024, 1)])
@pytest.mark.parametrize("a_off,w_off", [(1, 0), (0, 1), (3, 5)])
def test_gemm_unaligned_operands(M, N, K, splitk, a_off, w_off):
    torch = torch_cuda()
    from paper_2607_12659_amd import jpi
    from paper_2607_12659_amd.expert import to_device
    rng = np.random.default_rng(M + N + a_off + w_off)
    A, W = _bf16(rng.normal(size=(M, K))), _bf16(rng.normal(size=(N, K)) * 0.02)

    def at(x, off):
        buf = torch.zeros(x.size + 8, dtype=torch.int16, device="cuda")
        buf[off:off + x.size] = to_device(x).reshape(-1)
        return buf[off:off + x.size]
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    print("case unaligned", M, N, K, splitk, a_off, w_off, flush=True)
    st = jpi.jpi_debug_gemm(at(A, a_off), at(W, w_off), C, M, N, K, jpi.JPI_BF16, splitk)
    assert st == jpi.JPI_OK, jpi.jpi_last_error(None)
    torch.cuda.synchronize()
    a, w = oracle.widen(A), oracle.widen(W)
    assert np.all(np.abs(C.cpu().numpy().astype(np.float64) - a @ w.T) <= 1e-5 * (np.abs(a) @ np.abs(w).T) + 1e-6)


# merges of 3, 5, 6, 7, 9, 12 and 14 key ranges; a rollout with fewer keys leaves ranges empty
@pytest.mark.parametrize("B,P,Dh", [(2, 100, 64), (3, 333, 128), (2, 300, 256), (7, 816, 64), (2, 500, 128), (2, 700, 64),
                                    (2, 816, 256)])
def test_attention_range_counts(B, P, Dh):
    from paper_2607_12659_amd import jpi
    lens = [P, 0, 33, P - 1, 64, 1, 31][:B]
    got, ref, _ = _attention(jpi.JPI_BF16, B, 8, 50, P, Dh, lens, seed=B + P)
    # probabilities and the ranges' partial outputs are rounded to bf16 (relative 2^-9 each), values are N(0, 1)
    assert np.abs(got - ref).max() < 2e-2, np.abs(got - ref).max()
    assert np.sqrt(((got - ref) ** 2).mean()) < 4e-3


# 550, 527 and 550 action rows with even, odd and even horizons (V^T stores of 4, 1 and 2 tokens), ragged prefixes, one empty
@pytest.mark.parametrize("width,heads,Dh,horizon,batch,n_corr", [(256, 4, 64, 10, 55, 0), (512, 10, 128, 17, 31, 0),
                                                                 (1024, 8, 256, 50, 11, 0), (256, 4, 64, 16, 30, 4)])
def test_denoise_past_512_rows(width, heads, Dh, horizon, batch, n_corr):
    d = synth.Dims(n_layers=2, width=width, n_heads=heads, n_kv_heads=1, head_dim=Dh, mlp_dim=2 * width, action_dim=7,
                   horizon=horizon)
    lens = tuple([70, 0, 33, 1, 64, 31, 32, 69, 63, 65][b % 10] for b in range(batch))
    wl = synth.Workload("rows", d, prefix=70, batch=batch, n_steps=2, n_fixed=0, dtype="bf16", prefix_len=lens, mod_gain=8.0)
    inp = Inputs(wl)
    corr = synth.normal_f32(wl.seed, "item", 1.0, (batch, n_corr, width)) if n_corr else None
    print("case", width, horizon, batch, n_corr, flush=True)
    ae = make_expert(wl, inp.weights, max_batch=batch + 1, max_prefix=75, max_corr=n_corr)
    try:
        got = run(ae, inp.K, inp.V, inp.noise, 2, prefix_len=lens, corr=corr)
        ref = oracle.denoise(oracle.Expert(d, inp.weights), inp.noise, inp.K, inp.V, lens, 2, corr=corr)
        # bf16 inputs of every product over two layers and two steps: 0.1-2e-3 measured per rollout
        assert_bf16(got, ref, "rows", reg_rel=4e-3, reg_abs=4e-2)
    finally:
        ae.close()


# the last row kernel's passes over 1024 columns: one, two and four, the last one ragged; action widths around its groups of eight
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width,A", [(192, 8), (1024, 1), (1088, 9), (2112, 17)])
def test_last_row_kernel_widths(dtype, width, A):
    d = synth.Dims(n_layers=1, width=width, n_heads=1, n_kv_heads=1, head_dim=64, mlp_dim=64, action_dim=A, horizon=3)
    B = 2 if dtype == "f32" else 171  # 513 rows: past the five-launch layers
    lens = tuple([5, 0][b % 2] for b in range(B))
    wl = synth.Workload("head", d, prefix=5, batch=B, n_steps=2, n_fixed=1, dtype=dtype, prefix_len=lens)
    inp = Inputs(wl)
    print("case", dtype, width, A, flush=True)
    ae = make_expert(wl, inp.weights)
    try:
        got = run(ae, inp.K, inp.V, inp.noise, 2, prefix_len=lens, committed=inp.committed, n_fixed=1)
        pick = [0, 1, B - 1]  # rollouts are independent
        ref = oracle.denoise(oracle.Expert(d, inp.weights), inp.noise[pick], inp.K[:, pick], inp.V[:, pick],
                             [lens[b] for b in pick], 2, committed=inp.committed[pick], n_fixed=1)
        # fp32 sums of at most 2112 terms per product; bf16: every product's inputs rounded (2^-9 each)
        bar = 1e-5 if dtype == "f32" else 4e-3
        assert np.linalg.norm(got[pick] - ref) <= bar * np.linalg.norm(ref)
        assert np.array_equal(got[:, :1], inp.committed.astype(np.float64))
    finally:
        ae.close()


# several rollouts whose rows start at every place mod 4 in a row tile (QKV tiles cross rollouts)
@pytest.mark.parametrize("prefix", [44, 45, 46, 47])
def test_prefill_rows_cross_rollouts(prefix):
    torch = torch_cuda()
    from paper_2607_12659_amd import jpi
    from paper_2607_12659_amd.expert import to_device
    B, vd = 12, synth_vlm.VLM_TINY
    vwl = synth_vlm.VlmWorkload("vlm-rows", vd, prefix=prefix, batch=B)
    vw, emb = synth_vlm.make_vlm_weights(vwl), synth_vlm.make_embeddings(vwl)
    d = synth.Dims(n_layers=2, width=256, n_heads=4, n_kv_heads=1, head_dim=vd.head_dim, mlp_dim=512, action_dim=7, horizon=10)
    ewl = synth.Workload("expert", d, prefix=prefix, batch=B, n_steps=1, n_fixed=0, dtype="bf16")
    print("case", prefix, flush=True)
    vlm, ae = Vlm(vd, vw, B, prefix), make_expert(ewl, synth.make_weights(ewl))
    try:
        vlm.prefill(to_device(np.ascontiguousarray(emb, np.float32)), B, prefix, ae)
        torch.cuda.synchronize()
        _, kp, _ = jpi.jpi_prefix_buffers(ae.ctx)
        _, vt, ld = jpi.jpi_debug_prefix_vt(ae.ctx)
        K = bf16_bits_to_f64(device_view_i16(kp, (2, B, prefix, vd.head_dim)).cpu().numpy())
        V = bf16_bits_to_f64(device_view_i16(vt, (2, B, vd.head_dim, ld)).cpu().numpy())[..., :prefix]
        for b in range(B):
            K_o, V_o, _ = oracle.vlm_prefill(vd, vw, emb[b])
            for g, o in ((K[:, b], K_o), (V[:, b], np.swapaxes(V_o, 1, 2))):
                # bf16 storage and inputs over two layers, as in the single-rollout prefill
                assert np.linalg.norm(g - o) <= 1e-2 * np.linalg.norm(o), (b, np.linalg.norm(g - o) / np.linalg.norm(o))
    finally:
        ae.close()
        vlm.close()
