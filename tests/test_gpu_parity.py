"""GPU parity: the HIP path through the C ABI against the CPU oracle, element
by element, on the toy and one-layer workloads and on the edge cases."""
import dataclasses

import numpy as np
import pytest
import torch

import parity as P
from oracle import vidkv_oracle as O
from paper_2503_16257_amd import binding as vk
from paper_2503_16257_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _codec_all_heads(run: P.GpuRun, heads=None, scores=None, idx=None):
    w = run.w
    stats = {}
    heads = range(w.n_heads) if heads is None else heads
    sal_cache = {}
    for hd in heads:
        b = (hd // w.Hkv) % w.B
        if b not in sal_cache:
            sal_cache[b] = P.oracle_salient(w, b, None if scores is None else scores[b],
                                            None if idx is None else idx[b])
        P.check_keys_head(run, hd, synth.key_head(w, hd), stats)
        P.check_values_head(run, hd, synth.value_head(w, hd), sal_cache[b], stats)
    P.check_near_budget(stats)
    return stats


def _tails(w, layer, rows, dev=DEV):
    """Tail buffers [B, Hkv, rows, 128] of one layer, host and device."""
    Kt = np.stack([synth.tail_heads(w, layer, b, rows)[0] for b in range(w.B)])
    Vt = np.stack([synth.tail_heads(w, layer, b, rows)[1] for b in range(w.B)])
    return Kt, Vt, torch.from_numpy(Kt).to(dev), torch.from_numpy(Vt).to(dev)


@pytest.mark.parametrize("name", ["c1_toy", "c1_toy_na8"])
def test_toy_codec_and_attention(name):
    w = synth.WORKLOADS[name]
    print(f"[case] {name}", flush=True)
    run = P.GpuRun(w, DEV)
    scores = synth.saliency(w)
    _codec_all_heads(run, scores=scores)
    if name == "c1_toy_na8":
        assert run.key_record(0)["anom"].tolist() == synth.outlier_channels(w, 0).tolist()
    q = synth.query(w, 0)
    Kt, Vt, Ktd, Vtd = _tails(w, 0, w.T_tail)
    tl = torch.full((w.B,), w.T_tail, dtype=torch.int32, device=DEV)
    out = run.attention(0, torch.from_numpy(q).to(DEV), Ktd, Vtd, w.T_tail, tl).cpu().numpy()
    ref = P.oracle_attention(run, 0, 0, q[0], Kt[0], Vt[0])
    P.assert_out_close(out[0], ref, name)


def test_layer_codec_and_attention():
    w = synth.WORKLOADS["c2_layer"]
    print("[case] c2_layer", flush=True)
    run = P.GpuRun(w, DEV)
    _codec_all_heads(run)
    for hd in range(w.n_heads):
        assert set(synth.outlier_channels(w, hd).tolist()) <= set(run.key_record(hd)["anom"].tolist())
    q = synth.query(w, 0)
    out = run.attention(0, torch.from_numpy(q).to(DEV)).cpu().numpy()
    ref = P.oracle_attention(run, 0, 0, q[0])
    P.assert_out_close(out[0], ref, "c2_layer")


def test_index_list_equals_score_selection():
    """Passing the oracle's top-n list as indices gives the same buffer as passing scores."""
    w = synth.reduced(synth.WORKLOADS["c4_long"], 16)            # 3136 tokens, 156 protected
    print("[case] idx-vs-scores", flush=True)
    a = P.GpuRun(w, DEV)
    scores = synth.saliency(w)
    idx = np.stack([O.select_salient_tokens(scores[b], w.n_salient) for b in range(w.B)])
    b_ = P.GpuRun(w, DEV, salient_idx=torch.from_numpy(idx).to(DEV))
    assert np.array_equal(a.pv_np, b_.pv_np)
    _codec_all_heads(a, scores=scores)


@pytest.mark.parametrize("case", ["long_scores", "long_indices", "layer_no_protection", "serving_batch",
                                  "two_bit_rows_one_bit_keys"])
def test_fused_quantizer_equals_separate_calls(case):
    """vidkv_quantize_kv (with a side stream, below the size from which it uses one) writes the same bytes as
    the two separate calls, on the default and on a caller's stream, call after call."""
    kw = {}
    if case.startswith("long"):
        # 34 496 tokens, 1 724 protected: the selection is a chain of six launches, at 35 MB of keys in line
        w = synth.reduced(synth.WORKLOADS["c4_long"], 176)
    elif case == "layer_no_protection":
        w = synth.WORKLOADS["c2_layer"]
    elif case == "serving_batch":
        w = synth.reduced(synth.WORKLOADS["c5_serving"], 8, B=3)
    else:
        w = synth.reduced(synth.WORKLOADS["c4_long"], 16)
        kw = dict(salient_bits=2, use_fft=0)
    print(f"[case] fused-{case}", flush=True)
    idx = None
    if case == "long_indices":
        idx = torch.from_numpy(np.stack([
            np.sort(O.select_salient_tokens(synth.saliency(w)[b], w.n_salient)).astype(np.int32)
            for b in range(w.B)])).to(DEV)
    a = P.GpuRun(w, DEV, salient_idx=idx, **kw)
    b = P.GpuRun(w, DEV, salient_idx=idx, fused=True, **kw)
    assert torch.equal(a.pk, b.pk) and torch.equal(a.pv, b.pv)
    side = torch.cuda.Stream()                                     # default priority
    for rep in range(3):
        b.pk.fill_(0xA5)
        b.pv.fill_(0x5A)
        b.ws.fill_(rep)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            b.quantize(stream=side)
        torch.cuda.synchronize()
        assert torch.equal(a.pk, b.pk) and torch.equal(a.pv, b.pv), rep


def test_score_ties_and_negative_scores():
    w = synth.reduced(synth.WORKLOADS["c4_long"], 8)             # 1568 tokens, 78 protected
    print("[case] score ties", flush=True)
    rng = np.random.default_rng(5)
    scores = rng.integers(-3, 4, size=(w.B, w.T)).astype(np.float32)     # heavy ties, both signs
    scores[0, 5] = -0.0
    run = P.GpuRun(w, DEV, saliency=torch.from_numpy(scores).to(DEV))
    _codec_all_heads(run, scores=scores)


@pytest.mark.parametrize("n_a", [0, 8, 32, 128])
def test_anomalous_channel_counts(n_a):
    w = dataclasses.replace(synth.reduced(synth.WORKLOADS["c2_layer"], 8), n_anom=n_a)
    print(f"[case] n_a={n_a}", flush=True)
    run = P.GpuRun(w, DEV)
    _codec_all_heads(run)
    q = synth.query(w, 0)
    out = run.attention(0, torch.from_numpy(q).to(DEV)).cpu().numpy()
    P.assert_out_close(out[0], P.oracle_attention(run, 0, 0, q[0]), f"n_a={n_a}")


@pytest.mark.parametrize("Hkv,Hq", [(1, 1), (2, 4), (1, 8), (3, 15)])
def test_gqa_ratios_batch_and_layers(Hkv, Hq):
    base = synth.reduced(synth.WORKLOADS["c5_serving"], 8, L=2, B=3)
    w = dataclasses.replace(base, Hkv=Hkv, Hq=Hq, frames=8, n_salient=20, T_tail=7)
    print(f"[case] gqa {Hkv}/{Hq}", flush=True)
    run = P.GpuRun(w, DEV)
    scores = synth.saliency(w)
    _codec_all_heads(run, scores=scores)
    for layer in range(w.L):
        q = synth.query(w, layer)
        Kt, Vt, Ktd, Vtd = _tails(w, layer, 9)
        tl_np = np.array([7, 0, 9], dtype=np.int32)
        tl = torch.from_numpy(tl_np).to(DEV)
        out = run.attention(layer, torch.from_numpy(q).to(DEV), Ktd, Vtd, 9, tl).cpu().numpy()
        for b in range(w.B):
            ref = P.oracle_attention(run, layer, b, q[b], Kt[b][:, :tl_np[b]], Vt[b][:, :tl_np[b]])
            P.assert_out_close(out[b], ref, f"gqa {Hkv}/{Hq} l{layer} b{b}")


def test_values_eight_times_larger_scale_the_error_with_them():
    """Pins the error model of the attention output: every term of the error is a relative
    error of a probability or of a value, so with V scaled by 8 the absolute error may grow 8
    times and no more (the probabilities entering the numerator and the denominator are the
    same rounded numbers, so no bias adds to it)."""
    w = synth.reduced(synth.WORKLOADS["c4_long"], 24)
    print("[case] values x8", flush=True)
    K = torch.from_numpy(np.stack([synth.key_head(w, hd) for hd in range(w.n_heads)])
                         .reshape(w.L, w.B, w.Hkv, w.T, 128)).to(DEV)
    V1 = np.stack([synth.value_head(w, hd) for hd in range(w.n_heads)]).reshape(w.L, w.B, w.Hkv, w.T, 128)
    q = synth.query(w, 0)
    errs = []
    for scale in (1.0, 8.0):
        V = torch.from_numpy((V1.astype(np.float32) * scale).astype(np.float16)).to(DEV)
        run = P.GpuRun(w, DEV, K=K, V=V)
        out = run.attention(0, torch.from_numpy(q).to(DEV)).cpu().numpy()
        ref = P.oracle_attention(run, 0, 0, q[0])
        err = np.abs(out[0].astype(np.float64) - ref).max()
        assert np.isfinite(out).all()
        assert err <= scale * P.ATOL_OUT, f"values x{scale}: max abs err {err:.3e}"
        errs.append(err)
    print(f"[step] max err {errs[0]:.2e} at x1, {errs[1]:.2e} at x8", flush=True)


def test_one_long_head_many_split_parts():
    """One KV head with a long sequence: the split count goes far above what the
    one-round merge takes, so the general merge kernel is the one checked here."""
    base = synth.reduced(synth.WORKLOADS["c4_long"], 496)
    w = dataclasses.replace(base, Hkv=1, Hq=7, T_tail=40)
    print("[case] one long head", flush=True)
    run = P.GpuRun(w, DEV)
    q = synth.query(w, 0)
    Kt, Vt, Ktd, Vtd = _tails(w, 0, 64)
    tl = torch.tensor([40], dtype=torch.int32, device=DEV)
    out = run.attention(0, torch.from_numpy(q).to(DEV), Ktd, Vtd, 64, tl).cpu().numpy()
    ref = P.oracle_attention(run, 0, 0, q[0], Kt[0][:, :40], Vt[0][:, :40])
    P.assert_out_close(out[0], ref, "one long head")


def test_large_residual_block_with_ragged_lengths():
    """A batch with a large residual block, which gets a launch of its own, with lengths from 0 to the capacity: sampled
    sequences against the oracle."""
    w = synth.reduced(synth.WORKLOADS["c5_serving"], 8, B=32)
    print("[case] large residual block, ragged", flush=True)
    run = P.GpuRun(w, DEV)
    cap = 256
    q = synth.query(w, 0)
    Kt, Vt, Ktd, Vtd = _tails(w, 0, cap)
    rng = np.random.default_rng(5)
    tl_np = rng.integers(0, cap + 1, size=w.B).astype(np.int32)
    tl_np[0], tl_np[1], tl_np[2] = 0, cap, 1
    tl = torch.from_numpy(tl_np).to(DEV)
    out = run.attention(0, torch.from_numpy(q).to(DEV), Ktd, Vtd, cap, tl).cpu().numpy()
    for b in (0, 1, 2, 17, 31):
        n = int(tl_np[b])
        ref = P.oracle_attention(run, 0, b, q[b], Kt[b][:, :n], Vt[b][:, :n])
        P.assert_out_close(out[b], ref, f"large residual block b{b} len {n}")


def test_no_quantized_tokens_is_plain_attention():
    w = dataclasses.replace(synth.WORKLOADS["c2_layer"], frames=0, n_salient=0, B=2)
    print("[case] Tq=0", flush=True)
    run = P.GpuRun(w, DEV, K=torch.zeros((1, 2, 4, 0, 128), dtype=torch.float16, device=DEV),
                   V=torch.zeros((1, 2, 4, 0, 128), dtype=torch.float16, device=DEV))
    q = synth.query(w, 0)
    Kt, Vt, Ktd, Vtd = _tails(w, 0, 70)
    tl_np = np.array([70, 0], dtype=np.int32)
    out = run.attention(0, torch.from_numpy(q).to(DEV), Ktd, Vtd, 70,
                        torch.from_numpy(tl_np).to(DEV)).cpu().numpy()
    ref0 = P.oracle_attention(run, 0, 0, q[0], Kt[0], Vt[0])
    P.assert_out_close(out[0], ref0, "tail only")
    assert not out[1].any()                                   # a sequence with no token gets zeros


def test_single_group_and_all_protected():
    # 32 tokens, all protected: every trit is 0 and the rows carry everything
    print("[case] single group", flush=True)
    K = torch.from_numpy(synth.key_head(synth.WORKLOADS["c1_toy"], 0)[:32].reshape(1, 1, 1, 32, 128).copy()).to(DEV)
    V = torch.from_numpy(synth.value_head(synth.WORKLOADS["c1_toy"], 0)[:32].reshape(1, 1, 1, 32, 128).copy()).to(DEV)
    p = vk.make_params(1, 1, 1, 1, 32, 64, 32, gamma=P.GAMMA)
    pk = vk.alloc_bytes(vk.packed_keys_bytes(p), DEV)
    pv = vk.alloc_bytes(vk.packed_values_bytes(p), DEV)
    ws = vk.alloc_bytes(max(vk.workspace_bytes(p, i) for i in range(3)), DEV)
    sal = torch.rand((1, 32), device=DEV)
    vk.quantize_keys(p, K, pk, ws)
    vk.quantize_values(p, V, pv, ws, saliency=sal)
    q = torch.from_numpy(synth.query(synth.WORKLOADS["c1_toy"], 0)).to(DEV)
    out = torch.empty((1, 1, 128), dtype=torch.float16, device=DEV)
    vk.decode_attention(p, 0, q, pk, pv, out, ws)
    torch.cuda.synchronize()
    from oracle import layout as LY
    pk_np, pv_np = pk.cpu().numpy(), pv.cpu().numpy()
    perm, recs = LY.key_head_views(pk_np, 1, 1, 1, 32, 64, 0)
    Kd = O.dequantize_keys_head(LY.unpack_key_head(perm, recs, 64))
    codes, s16 = LY.unpack_value_head(LY.value_head_records(pv_np, 1, 1, 1, 32, 0))
    assert not codes.any()
    sec = LY.value_sections(1, 1, 1, 32, 32)
    idx, mask, rank = LY.unpack_salient(pv_np, sec, 0, 32, 32)
    assert idx.tolist() == list(range(32)) and mask[0] == 0xFFFFFFFF and rank[0] == 0
    rows = LY.salient_rows(pv_np, sec, 0, 32)
    Vh = V.cpu().numpy()[0, 0, 0]
    assert np.array_equal(rows.view(np.uint16), Vh.view(np.uint16))
    ref = O.attention_single_query(q.cpu().numpy()[0, 0], Kd, Vh.astype(np.float64), float(p.softmax_scale))
    P.assert_out_close(out.cpu().numpy()[0, 0], ref, "single group")


def test_split_count_does_not_change_the_result():
    """Same cache read with different batch sizes (hence different split-T
    counts): per-sequence outputs agree to accumulation-order noise."""
    w1 = synth.reduced(synth.WORKLOADS["c2_layer"], 16)
    print("[case] split invariance", flush=True)
    run1 = P.GpuRun(w1, DEV)
    q = synth.query(w1, 0)
    out1 = run1.attention(0, torch.from_numpy(q).to(DEV)).cpu().numpy()
    B = 40
    w2 = dataclasses.replace(w1, B=B)
    K2 = run1.K.expand(1, B, 4, w1.T, 128).contiguous()
    V2 = run1.V.expand(1, B, 4, w1.T, 128).contiguous()
    run2 = P.GpuRun(w2, DEV, K=K2, V=V2)
    q2 = torch.from_numpy(q).to(DEV).expand(B, 28, 128).contiguous()
    out2 = run2.attention(0, q2).cpu().numpy()
    assert np.abs(out2[0].astype(np.float64) - out1[0]).max() <= 1e-3
    assert np.array_equal(out2[0], out2[B - 1])


def test_calib_copy():
    src = torch.randint(0, 255, (1 << 20,), dtype=torch.uint8, device=DEV)
    dst = torch.zeros_like(src)
    vk.calib_copy(dst, src)
    torch.cuda.synchronize()
    assert torch.equal(src, dst)
