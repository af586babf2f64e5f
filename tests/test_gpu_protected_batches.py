"""GPU parity of decode attention where protected value tokens come in runs around the batch
sizes of the kernel (16 fp16 rows, records of 32 rows at 2 bits, 64 tokens of a pair), and where
an index list names fewer tokens than it has entries."""
import dataclasses

import numpy as np
import pytest
import torch

import parity as P
from oracle import vidkv_oracle as O
from paper_2503_16257_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(idx, bits, t_capacity=0, n_a=16):
    w = dataclasses.replace(synth.reduced(synth.WORKLOADS["c4_long"], 8), Hkv=2, Hq=14, n_anom=n_a,
                            n_salient=len(idx))
    d = torch.from_numpy(np.asarray(idx, np.int32)[None]).to(DEV)
    return P.GpuRun(w, DEV, salient_idx=d, salient_bits=bits, t_capacity=t_capacity), w


@pytest.mark.parametrize("n_a", [16, 96])
@pytest.mark.parametrize("bits", [16, 2])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 95, 129, 700])
def test_runs_of_protected_tokens(n, bits, n_a):
    run, w = _run(list(range(45, 45 + n)) + [w for w in (1200, 1567) if w >= 45 + n], bits, n_a=n_a)
    q = synth.query(w, 0)
    out = run.attention(0, torch.from_numpy(q).to(DEV)).cpu().numpy()
    P.assert_out_close(out[0], P.oracle_attention(run, 0, 0, q[0]), f"{n} protected in a row, {bits} bits")


def _oracle(run, w, q, n):
    """The oracle's attention from the packed bytes, with the first n entries of IDX and their rows only."""
    K, V = [], []
    for h in range(w.Hkv):
        K.append(O.dequantize_keys_head(run.key_record(h)))
        v = run.value_record(h)
        V.append(O.ternary_dequant(v["codes"], v["s16"], v["idx"][:n], v["rows"][:n]))
    none = np.zeros((w.Hkv, 0, 128), np.float16)
    return O.decode_attention(q, np.stack(K), np.stack(V), none, none, float(run.p.softmax_scale))


@pytest.mark.parametrize("bits", [16, 2])
def test_dropped_entries_and_a_flush_behind_them(bits):
    """Entries outside the cache are dropped: the rows behind the last protected token are never
    written (here: stale bytes that are NaN as fp16), and a flushed group's rank counts all entries."""
    idx = list(range(3, 903, 100)) + [5000, 6000, 7000] * 9
    run, w = _run(idx, bits, t_capacity=1568 + 32)
    sec = P.LY.value_sections(w.L, w.B, w.Hkv, run.Tcap, w.n_salient, run.sal_bits)
    if bits == 16:
        rows = run.pv[sec["rows"]:sec["rows"] + w.n_heads * w.n_salient * 256].view(w.n_heads, w.n_salient, 256)
        rows[:, 9:] = 0xFF
    else:                                          # 36 entries: the second record holds none of the nine
        recs = run.pv[sec["rows"]:sec["rows"] + w.n_heads * 2 * P.LY.PREC].view(w.n_heads, 2, P.LY.PREC)
        recs[:, 1:] = 0xFF
    qn = synth.query(w, 0)
    q = torch.from_numpy(qn).to(DEV)
    a = run.attention(0, q)
    P.assert_out_close(a.cpu().numpy()[0], _oracle(run, w, qn[0], 9), f"{bits} bits")
    Kt = np.stack([synth.tail_heads(w, 0, b, 32)[0] for b in range(w.B)])
    Vt = np.stack([synth.tail_heads(w, 0, b, 32)[1] for b in range(w.B)])
    Kd, Vd = torch.from_numpy(Kt).to(DEV), torch.from_numpy(Vt).to(DEV)
    run.flush(0, Kd, Vd, 32, 32)
    run.advance(32)
    b = run.attention(0, q)
    P.assert_out_close(b.cpu().numpy()[0], _oracle(run, w, qn[0], 9), f"{bits} bits, flushed")
    # the same cache with exactly the nine tokens protected gives the same attention, before the
    # flush and behind it
    ref, _ = _run(idx[:9], bits, t_capacity=1568 + 32)
    if bits == 16:
        assert torch.equal(a, ref.attention(0, q))
    ref.flush(0, Kd, Vd, 32, 32)
    ref.advance(32)
    if bits == 16:
        assert torch.equal(b, ref.attention(0, q))
