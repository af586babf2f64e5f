"""GPU parity of the key codes where a sign, a midpoint or a rounding decides: zeros of both signs,
constant channels, values on the midpoint of Eq. 4, subnormals, and a wide range; with
anomalous-channel counts whose last tile of 16 is full, half full or absent."""
import dataclasses

import numpy as np
import pytest
import torch

import parity as P
from paper_2503_16257_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _keys(w, kind, n_a):
    g = np.random.default_rng(7)
    x = g.standard_normal((1, 1, w.Hkv, w.T, 128))
    if kind == "zeros":                                   # groups of zeros, and zeros between numbers
        # (of both signs, but for the 2-bit code: its zero point may be the one or the other)
        z = np.copysign(0.0, x) if n_a == 0 else np.zeros_like(x)
        x = np.where(g.random(x.shape) < 0.6, z, np.round(2 * x))
        x = np.where((x == 0) & (n_a > 0), 0.0, x)
        x[:, :, :, :64] = z[:, :, :, :64]
    elif kind == "constant":
        x[:] = x[:, :, :, :1]
    elif kind == "midpoints":                             # few values, so that many lie on a group's midpoint
        x = np.round(x).clip(-2, 2) * 0.5
    elif kind == "neighbours":                            # two adjacent fp16 numbers and their signs
        x = np.where(x < 0, -1.0, 1.0) * np.where(g.random(x.shape) < 0.5, 1.0, 1.0009765625)
        x[:, :, :, 32:96] = np.abs(x[:, :, :, 32:96])
        x[:, :, :, 96:160] = -np.abs(x[:, :, :, 96:160])
    elif kind == "subnormal":
        x = x * 2.0 ** -23
    elif kind == "wide":
        x = (x * 8000).clip(-30000, 30000)
    return x.astype(np.float16)


@pytest.mark.parametrize("n_a", [0, 8, 24, 64, 120, 128])
@pytest.mark.parametrize("kind", ["zeros", "constant", "midpoints", "neighbours", "subnormal", "wide"])
@pytest.mark.parametrize("fft", [1, 0])
def test_key_codes(fft, kind, n_a):
    w = dataclasses.replace(synth.reduced(synth.WORKLOADS["c4_long"], 8), Hkv=2, Hq=14, n_anom=n_a, n_salient=0)
    print(f"[case] key codes fft {fft} {kind} n_a {n_a}", flush=True)
    K = _keys(w, kind, n_a)
    run = P.GpuRun(w, DEV, K=torch.from_numpy(K).to(DEV), use_fft=fft)
    stats = {}
    for hd in range(w.Hkv):
        P.check_keys_head(run, hd, K[0, 0, hd], stats)


@pytest.mark.parametrize("fft", [1, 0])
@pytest.mark.parametrize("n_a", [0, 8, 24, 64, 128])
@pytest.mark.parametrize("heads", [5, 6])
def test_groups_shared_out_and_not(heads, n_a, fft):
    """49 groups a head: 5 heads are coded one group per workgroup, 6 heads one per wave; a flush of 2 groups likewise
    and, of 6 heads x 22 groups (264 workgroups with the values), one per wave."""
    import test_gpu_flush as F
    w = dataclasses.replace(synth.reduced(synth.WORKLOADS["c4_long"], 8), Hkv=heads, Hq=heads, n_anom=n_a, n_salient=0)
    n = 64 if heads == 5 else 704
    run = P.GpuRun(w, DEV, use_fft=fft, t_capacity=w.T + n)
    stats = {}
    for hd in range(heads):
        P.check_keys_head(run, hd, synth.key_head(w, hd), stats)
    Kt, Vt = synth.tail_heads(w, 0, 0, n)
    run.flush(0, torch.from_numpy(Kt[None]).to(DEV), torch.from_numpy(Vt[None]).to(DEV), n, n)
    run.advance(n)
    for h in range(heads):
        F._check_block(run, h, w.T // 32, Kt[h], Vt[h], stats)
    P.check_near_budget(stats)
