"""The key range pass in each of its forms (1024 or 256 threads a chunk of 512 tokens, alone or beside the token selection, plain or
streaming loads): the channel split against the ranges and their order as torch finds them, through vidkv_quantize_keys and
vidkv_quantize_kv, whose packed bytes agree."""
import pytest
import torch

from paper_2503_16257_amd import binding as vk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N_A = 48


def _perm(K):
    """[heads, 128]: the N_A channels of largest range (ties: the lower channel), ascending, then the others, ascending."""
    R = K.amax(1).float() - K.amin(1).float()
    top = R.sort(dim=1, descending=True, stable=True).indices[:, :N_A].sort(dim=1).values
    rest = torch.ones(R.shape, dtype=torch.bool, device=DEV).scatter_(1, top, False)
    return torch.cat([top, rest.nonzero()[:, 1].view(len(R), -1)], 1).to(torch.uint8)


def _check(L, B, H, T, select):
    print(f"[case] {L} x {B} x {H} x {T} {select}", flush=True)
    n_s = 0 if select == "none" else max(1, T // 10)
    g = torch.Generator(device=DEV); g.manual_seed(T * 7 + L * B * H)
    heads = L * B * H
    # each channel's range is set by one token of its own, wherever it lies, and a third of them come in ties
    K = torch.randint(-8, 9, (heads, T, 128), generator=g, device=DEV, dtype=torch.int8).to(torch.float16)
    at = torch.randint(0, T, (heads, 1, 128), generator=g, device=DEV)
    K.scatter_(1, at, (torch.randint(20, 110, (heads, 1, 128), generator=g, device=DEV) * 4).to(torch.float16))
    V = torch.empty_like(K).normal_(generator=g)
    ref = _perm(K)
    p = vk.make_params(L, B, H, H, T, N_A, n_s)
    sal = torch.rand((B, T), generator=g, device=DEV) if n_s else None
    kw = {}
    if n_s:
        kw = {"saliency": sal} if select == "scores" else {"salient_idx": sal.topk(n_s).indices.sort(dim=1).values.to(torch.int32).contiguous()}
    ws = vk.alloc_bytes(vk.workspace_bytes(p, 3), DEV)
    pk, pv, rk, rv = (torch.zeros(n, dtype=torch.uint8, device=DEV) for n in (vk.packed_keys_bytes(p), vk.packed_values_bytes(p)) * 2)
    K5, V5 = K.view(L, B, H, T, 128), V.view(L, B, H, T, 128)
    vk.quantize_kv(p, K5, V5, pk, pv, ws, **kw)
    ws.fill_(0x5A)
    vk.quantize_keys(p, K5, rk, ws)
    vk.quantize_values(p, V5, rv, ws, **kw)
    torch.cuda.synchronize()
    assert torch.equal(rk[:heads * 128].view(heads, 128), ref), "channel split of quantize_keys"
    assert torch.equal(pk, rk) and torch.equal(pv, rv), "quantize_kv and the separate calls"


@pytest.mark.parametrize("select", ["none", "scores", "list"])
@pytest.mark.parametrize("T", [32, 96, 128, 224, 256, 480, 512, 544, 960, 1056])
def test_lengths_and_head_counts(T, select):
    for L, B, H in ((1, 3, 1), (1, 16, 4), (5, 16, 4), (3, 64, 4), (7, 50, 4)):
        _check(L, B, H, T, select)


@pytest.mark.parametrize("L,B,H,T", [(1, 3, 4, 8224), (1, 20, 8, 3136), (1, 2, 8, 32768), (1, 4, 8, 12544)])
def test_long_sequences_beside_their_selection(L, B, H, T):
    for select in ("scores", "list"):
        _check(L, B, H, T, select)


@pytest.mark.parametrize("L,B,H,T", [(2, 64, 64, 96), (2, 64, 8, 544), (1, 64, 8, 1056), (1, 8, 4, 16416), (1, 2, 4, 65568), (1, 3, 4, 90016)])
def test_streaming_loads(L, B, H, T):
    """More than 128 MiB of keys (the last: 277 MB), and a little less."""
    for select in ("none", "scores"):
        _check(L, B, H, T, select)
        if T > 16000:
            _check(L, B, H, T // 64 * 32, select)
