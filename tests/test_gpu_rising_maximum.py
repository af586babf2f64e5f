"""GPU parity of decode attention where the running maximum is raised again and again behind a wave's first
pair of groups, with and without protected rows waiting in its list, and where it never is."""
import dataclasses

import numpy as np
import pytest
import torch

import parity as P
from oracle import vidkv_oracle as O
from paper_2503_16257_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
B, H, T = 128, 4, 1568                         # 512 workgroups: one per head, six or seven pairs a wave


@pytest.mark.parametrize("fft", [1, 0])
@pytest.mark.parametrize("rows", [0, 16, 2])
@pytest.mark.parametrize("n_a", [16, 24, 64, 128])
def test_scores_that_rise(n_a, rows, fft):
    """Query heads 2 h and 2 h + 1 are each other's negative: the keys' scores rise along the tokens for one, fall for the other."""
    print(f"[case] rising scores, n_a {n_a}, rows {rows}, fft {fft}", flush=True)
    w = dataclasses.replace(synth.reduced(synth.WORKLOADS["c4_long"], 8), B=B, Hkv=H, Hq=2 * H, n_anom=n_a, n_salient=300 if rows else 0)
    assert w.T == T
    g = torch.Generator(device=DEV)
    g.manual_seed(n_a)
    q = torch.randn((B, H, 1, 128), generator=g, device=DEV)
    q = torch.cat((q, -q), dim=2).to(torch.float16)
    K = torch.randn((1, B, H, T, 128), generator=g, device=DEV)
    # from -300 to 300 in the exp2 domain, where |q|^2 = 128
    K += torch.linspace(-300, 300, T, device=DEV)[:, None] * q[None, :, :, :1].float() * (128 ** 0.5 / (128 * 1.4427))
    V = torch.randn((1, B, H, T, 128), generator=g, device=DEV)
    run = P.GpuRun(w, DEV, K=K.to(torch.float16), V=V.to(torch.float16), salient_bits=rows, use_fft=fft,
                   saliency=torch.rand((B, T), generator=g, device=DEV) if rows else None)
    out = run.attention(0, q.reshape(B, 2 * H, 128).contiguous()).cpu().numpy()
    qn = q.reshape(B, 2 * H, 128).cpu().numpy()
    for b in (0, B - 1):
        P.assert_out_close(out[b], P.oracle_attention(run, 0, b, qn[b]), f"seq {b}")
    # the case is what it claims: within a wave's run of pairs the maximum rises by more than 8 at least three times
    s = O.dequantize_keys_head(run.key_record(0)) @ qn[0, 0].astype(np.float64) * float(run.p.softmax_scale) * np.log2(np.e)
    top = s[:1536].reshape(24, 64).max(axis=1)[:6]
    assert (np.diff(top) > 8).sum() >= 3, top
