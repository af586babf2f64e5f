"""GPU parity of the key codes where a sign, a midpoint or a rounding decides: zeros of both signs,
constant channels, values on the midpoint of Eq. 4, subnormals, and a wide range; with
anomalous-channel counts whose last tile of 16 is full, half full or absent."""
import dataclasses

import numpy as np
import pytest
import torch

import parity as P
from paper_2503_16257_amd import binding as vk
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


@pytest.mark.parametrize("bits", [0x7E00, 0xFE01, 0x7D00], ids=["quiet", "negative", "signalling"])
@pytest.mark.parametrize("n_a", [0, 24, 64, 128])
@pytest.mark.parametrize("tokens", [[3], [0, 2], [0, 2, 16, 18], list(range(31))], ids=["one", "pair", "lane", "all but one"])
def test_a_nan_costs_nothing_but_its_own_code(tokens, n_a, bits):
    """NaN elements of a group (one lane's tokens 0 .. 3 and 16 .. 19 of a channel among them) against the same keys with the
    group's minimum in their place, whose code is 0: equal bytes, but for the NaN elements' own 1-bit codes.  Eq. 4 at 2 bits,
    and at 1 bit (a sum over 32 tokens, the DFT, passes a NaN on to its channel)."""
    H, T = 2, 96
    print(f"[case] NaN {bits:#x} at {len(tokens)} tokens, n_a {n_a}", flush=True)
    g = np.random.default_rng(11)
    clean = (g.standard_normal((1, 1, H, T, 128)) * (1 + g.random(128))).astype(np.float16)
    count = 0
    for ch in (1, 6, 64, 127):
        group = clean[0, 0, :, 32:64, ch]
        # (the channel's widest two numbers stand outside the group: which channels are 2-bit ones stays as it is)
        clean[0, 0, :, 0, ch], clean[0, 0, :, 1, ch] = -9.0, 9.0
        rest = np.delete(group, tokens, axis=1)
        group[:, tokens] = rest.min(axis=1, keepdims=True)
        count += H * len(tokens)
    bad = clean.copy()
    for ch in (1, 6, 64, 127):
        bad.view(np.uint16)[0, 0, :, 32:64, ch][:, tokens] = bits
    p = vk.make_params(1, 1, H, H, T, n_a, 0, use_fft=0)
    packed = []
    for K in (clean, bad):
        pk = torch.zeros(vk.packed_keys_bytes(p), dtype=torch.uint8, device=DEV)
        vk.quantize_keys(p, torch.from_numpy(K).to(DEV), pk, vk.alloc_bytes(vk.workspace_bytes(p, 0), DEV))
        packed.append(pk.cpu().numpy())
    differ = int(np.unpackbits(packed[0] ^ packed[1]).sum())
    assert differ <= (0 if n_a == 128 else count), f"{differ} bits differ"
