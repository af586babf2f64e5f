"""Protected-token selection around the sizes where it changes: slabs of 4096 tokens, the longest
sequence one workgroup takes (32768), the first one that takes the chain of launches; from scores
(with ties) and from index lists, in a cache with room behind the tokens.  IDX, MASK and RANK
against the oracle, exactly."""
import numpy as np
import pytest
import torch

from oracle import layout as LY
from oracle import vidkv_oracle as O
from paper_2503_16257_amd import binding as vk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("T", [32, 4064, 4096, 4128, 28704, 32768, 32800])
def test_selection(T, fused):
    B, room = 3, 64
    rng = np.random.default_rng(T)
    K = torch.randn((1, B, 1, T, 128), device=DEV).to(torch.float16)
    V = torch.randn((1, B, 1, T, 128), device=DEV).to(torch.float16)
    for n_s in sorted({1, 7, T // 5, T - 1, T}):
        for kind in ("uniform", "ties", "signed", "index"):
            print(f"[case] T {T} n_s {n_s} {kind}", flush=True)
            p = vk.make_params(1, B, 1, 1, T, 16, n_s, t_capacity=T + room)
            if kind == "uniform":
                sc = rng.random((B, T), dtype=np.float32)
            elif kind == "ties":
                sc = rng.integers(0, 3, (B, T)).astype(np.float32)
            else:
                sc = (rng.standard_normal((B, T)) * 1e3).astype(np.float32)
                sc[0, ::3] = -0.0
                sc[0, 1::3] = 0.0
            idx = [O.select_salient_tokens(sc[b], n_s) for b in range(B)]
            pk, pv = vk.alloc_bytes(vk.packed_keys_bytes(p)), vk.alloc_bytes(vk.packed_values_bytes(p))
            pv.fill_(0x5A)
            ws = vk.alloc_bytes(vk.workspace_bytes(p, 3))
            ws.fill_(0xFF)
            kw = (dict(salient_idx=torch.from_numpy(np.stack(idx).astype(np.int32)).to(DEV)) if kind == "index"
                  else dict(saliency=torch.from_numpy(sc).to(DEV)))
            if fused:
                vk.quantize_kv(p, K, V, pk, pv, ws, **kw)
            else:
                vk.quantize_values(p, V, pv, ws, **kw)
            torch.cuda.synchronize()
            sec = LY.value_sections(1, B, 1, T + room, n_s)
            ngc, ng = (T + room) // 32, T // 32
            got = pv.cpu().numpy()
            for b in range(B):
                i = got[sec["idx"] + 4 * b * n_s:][:4 * n_s].view("<i4")
                np.testing.assert_array_equal(i, idx[b])
                m = got[sec["mask"] + 4 * b * ngc:][:4 * ngc].view("<u4")
                r = got[sec["rank"] + 4 * b * ngc:][:4 * ngc].view("<u4")
                flag = np.zeros(T, np.uint32)
                flag[idx[b]] = 1
                word = (flag.reshape(ng, 32) << np.arange(32, dtype=np.uint32)).sum(axis=1, dtype=np.uint32)
                np.testing.assert_array_equal(m[:ng], word)
                np.testing.assert_array_equal(r[:ng], np.concatenate([[0], np.cumsum(flag.reshape(ng, 32).sum(1))[:-1]]))
                # room behind the tokens: cleared for an index list, left alone for scores
                assert (m[ng:] == (0 if kind == "index" else 0x5A5A5A5A)).all()


@pytest.mark.parametrize("T", [1568, 32768])
def test_scores_that_differ_in_one_digit(T):
    """Infinities, and scores whose ordered keys differ only in the highest, a middle or the lowest bits."""
    rng = np.random.default_rng(T)
    for kind in ("infinite", "high", "middle", "low"):
        if kind == "infinite":
            sc = rng.choice(np.array([-np.inf, -1.0, 0.0, 1.0, np.inf], np.float32), (2, T))
        else:
            shift = {"high": 24, "middle": 12, "low": 0}[kind]
            sc = (np.uint32(0x3F000000) + (rng.integers(0, 16, (2, T)).astype(np.uint32) << np.uint32(shift))).view(np.float32)
        for n_s in (1, T // 3, T - 1):
            print(f"[case] T {T} n_s {n_s} {kind}", flush=True)
            p = vk.make_params(1, 2, 1, 1, T, 16, n_s)
            V = torch.zeros((1, 2, 1, T, 128), dtype=torch.float16, device=DEV)
            pv, ws = vk.alloc_bytes(vk.packed_values_bytes(p)), vk.alloc_bytes(vk.workspace_bytes(p, 1))
            vk.quantize_values(p, V, pv, ws, saliency=torch.from_numpy(sc).to(DEV))
            off = LY.value_sections(1, 2, 1, T, n_s)["idx"]
            got = pv[off:off + 8 * n_s].cpu().numpy().view("<i4").reshape(2, n_s)
            for b in range(2):
                np.testing.assert_array_equal(got[b], O.select_salient_tokens(sc[b], n_s))


def test_equal_scores_take_no_longer():
    """The longest sequence of one workgroup, all scores equal (padding) against scattered ones.  A
    histogram whose counters for one digit share a bank takes 2.4 times as long, one that spreads them 0.93."""
    T = 32768
    p = vk.make_params(1, 1, 1, 1, T, 16, T // 10)
    V = torch.zeros((1, 1, 1, T, 128), dtype=torch.float16, device=DEV)
    pv, ws = vk.alloc_bytes(vk.packed_values_bytes(p)), vk.alloc_bytes(vk.workspace_bytes(p, 1))
    scattered = torch.rand((1, T), device=DEV)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def best(sc):
        t = []
        for _ in range(7):
            e0.record()
            for _ in range(50):
                vk.quantize_values(p, V, pv, ws, saliency=sc, stages=1)
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1))
        return min(t)

    assert best(torch.full_like(scattered, 0.25)) < 1.5 * best(scattered)
