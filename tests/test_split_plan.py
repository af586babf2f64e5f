"""How a decode call is split: the workspace of a cache with room to grow stays the same while it
grows (CPU), and grids just below and above one round, with and without residual tokens in the
same launch, against the oracle (GPU)."""
import dataclasses

import numpy as np
import pytest
import torch

import parity as P
from paper_2503_16257_amd import binding as vk
from paper_2503_16257_amd import synth

DEV = "cuda:0"


@pytest.mark.parametrize("batch,heads", [(1, 1), (1, 4), (3, 5), (43, 4), (300, 1), (1100, 1)])
def test_workspace_does_not_depend_on_the_fill(batch, heads):
    cap = 32 * 700
    sizes = {vk.workspace_bytes(vk.make_params(1, batch, heads, heads, 32 * g, 16, 0, t_capacity=cap), 2)
             for g in list(range(1, 60)) + [100, 257, 699, 700]}
    assert len(sizes) == 1
    full = [vk.workspace_bytes(vk.make_params(1, batch, heads, heads, 32 * g, 16, 0), 2) for g in range(1, 700)]
    assert full == sorted(full) and full[-1] <= max(sizes)


@pytest.mark.parametrize("batch,heads,rep,tokens", [(51, 8, 8, 512), (128, 4, 7, 512), (128, 4, 7, 196000), (300, 1, 8, 6272),
                                                    (64, 8, 7, 25088), (1, 1, 8, 1000000)])
def test_more_splits_never_outgrow_the_array_of_the_call_without_a_workspace(batch, heads, rep, tokens):
    """Shapes whose partials fit the library's array at one round of workgroups and two pairs per
    wave keep fitting it: the finer splits are only taken where they fit too."""
    p = vk.make_params(1, batch, heads, heads * rep, tokens, 16, 0)
    assert vk.workspace_bytes(p, 2) <= vk.NOALLOC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads", [(1, 1), (9, 4), (31, 4), (43, 3), (129, 1), (130, 4)])
@pytest.mark.parametrize("cap", [1, 40, 256])
def test_grids_around_one_round(batch, heads, cap):
    w = dataclasses.replace(synth.reduced(synth.WORKLOADS["c3_stack"], 8, L=1, B=batch), Hkv=heads, Hq=2 * heads)
    print(f"[case] {batch} x {heads} heads, residual capacity {cap}", flush=True)
    K, V = synth.device_kv(w, DEV)
    run = P.GpuRun(w, DEV, K=K, V=V)
    g = torch.Generator(device=DEV); g.manual_seed(cap)
    shape = (batch, heads, cap, 128)
    Kt, Vt = (torch.randn(shape, generator=g, device=DEV).to(torch.float16) for _ in range(2))
    tl = torch.randint(0, cap + 1, (batch,), generator=g, device=DEV, dtype=torch.int32)
    tl[0], tl[-1] = cap, 0 if batch > 1 else cap
    q = synth.query(w, 0)
    out = run.attention(0, torch.from_numpy(q).to(DEV), Kt, Vt, cap, tl).cpu().numpy()
    for b in {0, batch // 2, batch - 1}:
        n = int(tl[b])
        ref = P.oracle_attention(run, 0, b, q[b], Kt[b, :, :n].cpu().numpy(), Vt[b, :, :n].cpu().numpy())
        P.assert_out_close(out[b], ref, f"seq {b}")


@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads,cap", [(1, 4, 0), (1, 4, 128), (2, 1, 40), (16, 4, 256)])
def test_a_workspace_for_the_coarsest_split_is_still_taken(batch, heads, cap):
    """The size for one round of workgroups and two pairs per wave, which the query once reported: such a
    buffer is accepted, nothing behind it is touched, and one byte less is refused."""
    w = dataclasses.replace(synth.reduced(synth.WORKLOADS["c3_stack"], 32, L=1, B=batch), Hkv=heads, Hq=7 * heads)
    run = P.GpuRun(w, DEV)
    bh, npairs, cus = batch * heads, (w.T // 32 + 1) // 2, torch.cuda.get_device_properties(0).multi_processor_count
    splits = max(1, min(-(-2 * cus // bh), (npairs + 7) // 8))
    size = -(-(splits + 8) * batch * w.Hq * 130 * 4 // 256) * 256 + 256
    assert size <= vk.workspace_bytes(run.p, 2)
    if bh <= 4:
        assert size < vk.workspace_bytes(run.p, 2)
    big = torch.full((size + 4096,), 0xCC, dtype=torch.uint8, device=DEV)
    Kt = Vt = tl = None
    if cap:
        g = torch.Generator(device=DEV); g.manual_seed(cap)
        Kt, Vt = (torch.randn((batch, heads, cap, 128), generator=g, device=DEV).to(torch.float16) for _ in range(2))
        tl = torch.full((batch,), cap, dtype=torch.int32, device=DEV)
    q = synth.query(w, 0)
    qd = torch.from_numpy(q).to(DEV)
    out = torch.empty((batch, w.Hq, 128), dtype=torch.float16, device=DEV)
    kw = dict(K_tail=Kt, V_tail=Vt, tail_capacity=cap, tail_len=tl)
    vk.decode_attention(run.p, 0, qd, run.pk, run.pv, out, big[:size], **kw)
    torch.cuda.synchronize()
    assert (big[size:] == 0xCC).all()
    b = batch - 1
    ref = P.oracle_attention(run, 0, b, q[b], *((Kt[b].cpu().numpy(), Vt[b].cpu().numpy()) if cap else ()))
    P.assert_out_close(out[b].cpu().numpy(), ref, f"seq {b}")
    with pytest.raises(RuntimeError, match="too small"):
        vk.decode_attention(run.p, 0, qd, run.pk, run.pv, out, big[:size - 1], **kw)


@pytest.mark.gpu
def test_residual_tokens_do_not_hold_up_a_small_batch():
    """8 sequences x 4 KV heads of 1568 tokens: 128 residual tokens in the same launch, against none.  In
    one workgroup per head, 32 tokens after 32, the call took 1.9 times as long; in four 1.2 times."""
    from perf import cases

    def best(cap):
        st = cases.prepare(cases._case(kind="step", B=8, T=1568, cap=cap, tail=cap), 3)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t = []
        for _ in range(9):
            e0.record()
            for _ in range(50):
                cases.run(st)
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1))
        return min(t)

    assert best(128) < 1.5 * best(0)
