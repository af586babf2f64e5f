"""Decode attention keeps 32-bit accuracy for the anomalous-channel counts that are computed in
32 bits (every count but 0, 8, 16, 32, 64 and 128): inputs that show what 16-bit probabilities, scales
or queries lose, against the float64 oracle on the packed bytes.

Values alternate in sign where the scores are tested, so that the output is what the scores' differences
make of it: a score error e shows as e / (spread of the scores).

Tolerance: relative 2-norm of the whole output (all heads: one head's signed sum may happen to cancel).
Rounding the output to fp16 gives at most 2^-11 = 4.9e-4 of an element, about 2e-4 in the norm; p = exp2(t) carries a few 2^-24 of max(1, |t|), which a score spread
s turns into a few 2^-24 / s: below 1e-4 for the spreads here (4e-3 and more), about 2e-3 for the
subnormal scales' (1e-4).  Stated: 1e-3, and 8e-3 for the latter."""
import dataclasses

import numpy as np
import pytest
import torch

import parity as P
from paper_2503_16257_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _w(n_a, n_s=0):
    base = synth.reduced(synth.WORKLOADS["c4_long"], 8)          # 1568 tokens
    return dataclasses.replace(base, Hkv=2, Hq=14, n_anom=n_a, n_salient=n_s)


def _check(w, K, V, q, tol, what, idx=None, bits=16, fft=1):
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    run = P.GpuRun(w, DEV, K=dev(K), V=dev(V), salient_bits=bits, use_fft=fft,
                   salient_idx=None if idx is None else dev(idx[None].astype(np.int32)))
    got = run.attention(0, dev(q)).cpu().numpy()[0].astype(np.float64)
    ref = P.oracle_attention(run, 0, 0, q[0])
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"[err] {what}: {err:.3e}", flush=True)
    assert err <= tol, f"{what}: {err:.3e} > {tol}"


def _signed_values(w):
    V = np.full((1, 1, w.Hkv, w.T, 128), 60000.0, np.float16)
    V[:, :, :, 1::2] *= -1
    return V


@pytest.mark.parametrize("rows", ["none", "fp16", "2bit"])
@pytest.mark.parametrize("n_a", [24, 96, 120])
def test_probabilities_far_below_the_largest(n_a, rows):
    """One token whose value is 0 takes nearly all the weight; the output is what the others, each
    2^-d of it, add up to."""
    idx = None if rows == "none" else np.setdiff1d(np.arange(300, 1000), [777])
    w = _w(n_a, 0 if idx is None else len(idx))
    for d in (20.0, 24.6, 25.4, 28.0, 33.0):
        K = np.zeros((1, 1, w.Hkv, w.T, 128), np.float16)
        K[:, :, :, 777, 0] = 8.0
        V = np.full(K.shape, 60000.0, np.float16)
        V[:, :, :, 777] = 0.0
        q = np.zeros((1, w.Hq, 128), np.float16)
        q[:, :, 0] = d * np.log(2.0) * np.sqrt(128.0) / 8.0
        # a protected row's probability is held to 2^-22 of itself, and to 2^-43 of the largest
        tol = 1e-3 + (0.0 if rows == "none" else 2.0 ** (d - 43))
        _check(w, K, V, q, tol, f"n_a {n_a} {rows} 2^-{d}", idx=idx, bits=2 if rows == "2bit" else 16)


@pytest.mark.parametrize("fft", [1, 0])
@pytest.mark.parametrize("n_a", [24, 96, 120])
def test_small_queries(n_a, fft):
    """Query elements from 2^-24 to 2^-17 against large keys."""
    w, r = _w(n_a), np.random.default_rng(n_a)
    K = (1000.0 * r.standard_normal((1, 1, w.Hkv, w.T, 128))).astype(np.float16)
    q = (r.integers(-127, 128, (1, w.Hq, 128)) * 2.0 ** -24).astype(np.float16)
    _check(w, K, _signed_values(w), q, 1e-3, f"n_a {n_a} fft {fft}", fft=fft)


@pytest.mark.parametrize("n_a,fft,normal", [(24, 1, False), (96, 1, False), (96, 0, False), (24, 0, True), (96, 0, True)])
def test_subnormal_scales(n_a, fft, normal):
    """Keys of a few 2^-24: the codes' scale is the smallest fp16 number, and has no half."""
    w, r = _w(n_a), np.random.default_rng(n_a)
    K = np.zeros((1, 1, w.Hkv, w.T, 128))
    q = np.zeros((1, w.Hq, 128), np.float16)
    if normal:                                     # the 1-bit channels' scale; the others only take the places
        K[..., :n_a] = r.integers(0, 2, K.shape[:-1] + (n_a,)) * 4.0
        K[..., n_a:] = r.integers(0, 2, K.shape[:-1] + (128 - n_a,))
        q[..., n_a:] = 4000.0 * r.choice([-1.0, 1.0], (1, w.Hq, 128 - n_a))
    else:
        K[..., :n_a] = r.integers(0, 4, K.shape[:-1] + (n_a,))
        q[..., :n_a] = 4000.0 * r.choice([-1.0, 1.0], (1, w.Hq, n_a))
    _check(w, (K * 2.0 ** -24).astype(np.float16), _signed_values(w), q, 8e-3, f"n_a {n_a} fft {fft} normal {normal}", fft=fft)


@pytest.mark.parametrize("fft", [1, 0])
@pytest.mark.parametrize("n_a", [24, 96])
def test_queries_that_have_no_double(n_a, fft):
    """Elements beyond 2^15 in some heads and not in others, beside subnormal ones."""
    w, r = _w(n_a), np.random.default_rng(n_a)
    K = (2e-4 * r.standard_normal((1, 1, w.Hkv, w.T, 128))).astype(np.float16)
    q = r.standard_normal((1, w.Hq, 128)).astype(np.float16)
    q[:, ::3, 5::17] = 65504.0
    q[:, 1::3, 7::31] = -32768.0
    q[:, 2::3, 3::19] = 32752.0
    q[..., 9] = 2.0 ** -24
    _check(w, K, _signed_values(w), q, 1e-3, f"n_a {n_a} fft {fft}", fft=fft)


@pytest.mark.parametrize("fft", [1, 0])
@pytest.mark.parametrize("n_a", [8, 16, 32, 64, 128])
def test_small_queries_of_anomalous_channels(n_a, fft):
    """The other counts: the anomalous channels' queries keep all their bits too, where half of them is no fp16 number and the keys
    are large.  All channels of a token have one of four keys, so that what is lost adds up.  Tolerance: the probabilities are fp16
    numbers, at most 2^-11 of them off, and the scores spread by about 0.0018 n_a."""
    w, r = _w(n_a), np.random.default_rng(n_a)
    K = np.zeros((1, 1, w.Hkv, w.T, 128), np.float16)
    K[..., :n_a] = (r.integers(0, 4, (1, 1, w.Hkv, w.T, 1)) * 40000.0 - 60000.0).astype(np.float16)
    q = np.zeros((1, w.Hq, 128), np.float16)
    q[..., :n_a] = (r.integers(3, 6, (1, w.Hq, 1)) * 4 - 1) * 2.0 ** -24
    _check(w, K, _signed_values(w), q, 5e-4 + 2.0 ** -11 / (0.0018 * n_a), f"n_a {n_a} fft {fft}", fft=fft)


@pytest.mark.parametrize("fft", [1, 0])
@pytest.mark.parametrize("n_a", [16, 64, 128])
def test_queries_that_have_no_double_beside_others(n_a, fft):
    """The same counts with heads that have an element beyond 2^15 and heads that have none, anomalous or not.  Tolerance: fp16
    probabilities and a spread of the scores of 1 and more; the normal channels' q / 16 is exact here."""
    w, r = _w(n_a), np.random.default_rng(n_a)
    K = (2e-5 * r.standard_normal((1, 1, w.Hkv, w.T, 128))).astype(np.float16)
    K[..., 5::9] *= 4
    q = r.standard_normal((1, w.Hq, 128)).astype(np.float16)
    q[:, ::3, 5::9] = 65504.0
    q[:, 1::3, 7::9] = -32768.0
    q[:, 2::3, 3::9] = 32752.0
    _check(w, K, _signed_values(w), q, 2e-3, f"n_a {n_a} fft {fft}", fft=fft)
