"""GPU parity of decode attention for every anomalous-channel count, in both key codes and with
no, fp16 and 2-bit protected rows.  49 groups: the last pair of groups has one."""
import dataclasses

import numpy as np
import pytest
import torch

import parity as P
from paper_2503_16257_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_a", range(0, 129, 8))
def test_every_count(n_a):
    base = synth.reduced(synth.WORKLOADS["c4_long"], 8)
    w = dataclasses.replace(base, name=f"na{n_a}", Hkv=2, Hq=2 * (1 + n_a // 8 % 8), n_anom=n_a)
    K, V = torch.from_numpy(synth.keys(w)).to(DEV), torch.from_numpy(synth.values(w)).to(DEV)
    q = synth.query(w, 0)
    for use_fft in (1, 0):
        for n_s, bits in ((0, 16), (313, 16), (70, 2)):
            print(f"[case] n_a {n_a} fft {use_fft} n_s {n_s} bits {bits}", flush=True)
            run = P.GpuRun(dataclasses.replace(w, n_salient=n_s), DEV, use_fft=use_fft, salient_bits=bits,
                           K=K, V=V)
            out = run.attention(0, torch.from_numpy(q).to(DEV)).cpu().numpy()
            P.assert_out_close(out[0], P.oracle_attention(run, 0, 0, q[0]), f"n_a {n_a}")
