"""The fp16 residual tokens' part of decode attention, at the edges of its blocks of 32 tokens and of the four waves
that share them, alone and beside packed tokens, against attention in float64.

Tolerance with residual tokens alone, per element: half an fp16 ulp of the result (2^-11 of it, 2^-25 where it is
subnormal); the softmax weights and their sum carry the scores' rounding, at most (128 + 2) 2^-24 of sum |q| |k| per score, the
probabilities' 2^-21 (two fp16 parts and exp2) and n 2^-24 for the sums over n tokens, each times the largest |v|."""
import dataclasses

import numpy as np
import pytest
import torch

import parity as P
from paper_2503_16257_amd import binding as vk
from paper_2503_16257_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _alone(q, Kt, Vt, lens):
    """Call without packed tokens: q [B, Hq, 128], Kt / Vt [B, H, cap, 128] fp16 tensors on the GPU."""
    B, H, cap, _ = Kt.shape
    p = vk.make_params(1, B, H, q.shape[1], 0, 16, 0)
    pk, pv = (torch.zeros(max(n, 256), dtype=torch.uint8, device=DEV) for n in (vk.packed_keys_bytes(p), vk.packed_values_bytes(p)))
    out = torch.full((B, q.shape[1], 128), float("nan"), dtype=torch.float16, device=DEV)
    vk.decode_attention(p, 0, q, pk, pv, out, vk.alloc_bytes(vk.workspace_bytes(p, 2), DEV), K_tail=Kt, V_tail=Vt,
                        tail_capacity=cap, tail_len=torch.tensor(lens, dtype=torch.int32, device=DEV))
    return out.cpu().numpy().astype(np.float64)


def _check(q, Kt, Vt, lens, what):
    got = _alone(q, Kt, Vt, lens)
    rep = q.shape[1] // Kt.shape[1]
    for b, n in enumerate(lens):
        for h in range(q.shape[1]):
            if n == 0:
                assert not got[b, h].any(), what
                continue
            k, v = (x[b, h // rep, :n].cpu().numpy().astype(np.float64) for x in (Kt, Vt))
            qq = q[b, h].cpu().numpy().astype(np.float64)
            s = k @ qq / np.sqrt(128.0)
            w = np.exp(s - s.max())
            ref = (w / w.sum()) @ v
            size = (np.abs(k) @ np.abs(qq)).max() / np.sqrt(128.0)
            tol = np.abs(ref) * 2.0 ** -11 + 2.0 ** -25 + np.abs(v).max() * (2 * 130 * size + 8 + n) * 2.0 ** -24
            err = np.abs(got[b, h] - ref)
            assert (err <= tol).all(), f"{what} seq {b} head {h} len {n}: {err.max():.2e}, {(err / tol).max():.2f} of the bound"


@pytest.mark.parametrize("cap", [1, 31, 32, 33, 128, 129, 300, 1100])
@pytest.mark.parametrize("heads,rep", [(1, 1), (2, 7), (3, 8)])
def test_blocks_and_waves(cap, heads, rep):
    print(f"[case] residual cap {cap} heads {heads} x {rep}", flush=True)
    lens = sorted({0, 1, cap} | {n for n in (31, 32, 33, 64, 97, 127, 128, 129, 256, 257, 1024) if n < cap})
    g = torch.Generator(device=DEV); g.manual_seed(cap * 64 + heads)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)
    q = rnd(len(lens), heads * rep, 128).to(torch.float16)
    Kt, Vt = rnd(len(lens), heads, cap, 128).to(torch.float16), rnd(len(lens), heads, cap, 128).to(torch.float16)
    _check(q, Kt, Vt, lens, f"cap {cap}")


@pytest.mark.parametrize("n,d", [(300, 8.0), (300, 20.0), (300, 25.4), (300, 33.0), (300, 36.3), (9000, 40.7), (9000, 43.6), (9000, 47.3),
                                 (9000, 50.2)])
def test_probabilities_far_below_the_largest(n, d):
    """One token with value 0 takes nearly all the weight, the others have 2^-d of it each and the largest values:
    what they add up to is still there."""
    at = 170
    Kt = torch.zeros((1, 1, n, 128), dtype=torch.float16, device=DEV)
    Kt[:, :, at, 0] = 8.0
    Vt = torch.full((1, 1, n, 128), 60000.0, dtype=torch.float16, device=DEV)
    Vt[:, :, at] = 0.0
    q = torch.zeros((1, 7, 128), dtype=torch.float16, device=DEV)
    q[:, :, 0] = d * np.log(2.0) * np.sqrt(128.0) / 8.0
    got = _alone(q, Kt, Vt, [n])
    d16 = float(q[0, 0, 0]) * 8.0 / np.sqrt(128.0) / np.log(2.0)
    ref = 60000.0 * (n - 1) * 2.0 ** -d16 / (1.0 + (n - 1) * 2.0 ** -d16)
    # (the scores differ by d: 2^-22 d and the exponentials' 2^-22 of a weight; half an fp16 ulp)
    assert np.abs(got / ref - 1.0).max() <= 2.0 ** -11 + (d + 4) * 2.0 ** -22 + 2.0 ** -25 / ref


@pytest.mark.parametrize("batch,cap", [(1, 100), (8, 300), (40, 513), (70, 130)])
def test_beside_packed_tokens(batch, cap):
    """Residual workgroups in the packed tokens' launch, one or several blocks a wave, and in one of their own."""
    w = dataclasses.replace(synth.reduced(synth.WORKLOADS["c5_serving"], 8, B=batch), Hkv=4, Hq=28)
    print(f"[case] {batch} sequences, residual capacity {cap}", flush=True)
    run = P.GpuRun(w, DEV)
    g = torch.Generator(device=DEV); g.manual_seed(cap)
    Kt, Vt = (torch.randn((batch, 4, cap, 128), generator=g, device=DEV).to(torch.float16) for _ in range(2))
    tl = torch.randint(0, cap + 1, (batch,), generator=g, device=DEV, dtype=torch.int32)
    tl[0] = cap
    q = synth.query(w, 0)
    out = run.attention(0, torch.from_numpy(q).to(DEV), Kt, Vt, cap, tl).cpu().numpy()
    for b in {0, batch // 2, batch - 1}:
        n = int(tl[b])
        ref = P.oracle_attention(run, 0, b, q[b], Kt[b, :, :n].cpu().numpy(), Vt[b, :, :n].cpu().numpy())
        P.assert_out_close(out[b], ref, f"seq {b} len {n}")
