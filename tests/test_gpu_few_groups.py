"""vidkv_quantize_kv of calls with few groups (two launches, ranks and channels found by every workgroup for itself) against
the separate calls, byte for byte over the whole packed buffers: both write the same bytes and leave the same ones."""
import pytest
import torch

from paper_2503_16257_amd import binding as vk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _both(L, B, H, T, n_a, n_s, scores=None, idx=None, bits=16, fft=1, cap=0, K=None, V=None):
    p = vk.make_params(L, B, H, H, T, n_a, n_s, gamma=0.7, use_fft=fft, salient_bits=bits, t_capacity=cap)
    g = torch.Generator(device=DEV); g.manual_seed(T * 131 + n_a + n_s)
    if K is None:
        K = (torch.randn((L, B, H, T, 128), generator=g, device=DEV) * (1 + torch.rand((L, B, H, 1, 128), generator=g, device=DEV))).to(torch.float16)
    if V is None:
        V = torch.randn((L, B, H, T, 128), generator=g, device=DEV).to(torch.float16)
    ws = vk.alloc_bytes(vk.workspace_bytes(p, 3), DEV)
    out = []
    for fused in (True, False):
        pk = torch.full((vk.packed_keys_bytes(p),), 0xA5, dtype=torch.uint8, device=DEV)
        pv = torch.full((vk.packed_values_bytes(p),), 0xA5, dtype=torch.uint8, device=DEV)
        ws.fill_(0x5A)
        if fused:
            vk.quantize_kv(p, K, V, pk, pv, ws, saliency=scores, salient_idx=idx)
        else:
            vk.quantize_keys(p, K, pk, ws)
            vk.quantize_values(p, V, pv, ws, saliency=scores, salient_idx=idx)
        out.append((pk, pv))
    torch.cuda.synchronize()
    for a, b, what in zip(out[0], out[1], ("keys", "values")):
        d = (a != b).nonzero().flatten()
        assert d.numel() == 0, f"{what}: {d.numel()} bytes differ, the first at {int(d[0])}"
    return p, out[0]


def _scores(B, T, kind):
    g = torch.Generator(device=DEV); g.manual_seed(T)
    if kind == "uniform":
        return torch.rand((B, T), generator=g, device=DEV)
    if kind == "signed":
        return torch.randn((B, T), generator=g, device=DEV)
    if kind == "ties":
        return torch.randint(0, 3, (B, T), generator=g, device=DEV).to(torch.float32) * 0.5 - 0.5
    s = torch.zeros((B, T), device=DEV)                  # all equal, both zeros
    s[:, ::2] = -0.0
    return s


@pytest.mark.parametrize("L,B,H,T", [(1, 1, 1, 32), (1, 1, 1, 96), (1, 3, 2, 256), (2, 2, 1, 544), (1, 1, 4, 2048),
                                     (1, 1, 1, 4128), (1, 1, 1, 8192), (1, 7, 1, 1152), (28, 1, 1, 288)])
@pytest.mark.parametrize("kind", ["uniform", "signed", "ties", "equal"])
def test_shapes_and_scores(L, B, H, T, kind):
    print(f"[case] {L} x {B} x {H} x {T} {kind}", flush=True)
    for n_s in sorted({1, T // 10 + 1, T // 2, T - 1, T}):
        _both(L, B, H, T, 16, n_s, scores=_scores(B, T, kind))


@pytest.mark.parametrize("n_a", [0, 8, 16, 24, 32, 64, 96, 120, 128])
@pytest.mark.parametrize("fft", [1, 0])
def test_channel_counts(n_a, fft):
    print(f"[case] n_a {n_a} fft {fft}", flush=True)
    _both(1, 2, 2, 1056, n_a, 100, scores=_scores(2, 1056, "uniform"), fft=fft)
    _both(1, 2, 2, 1056, n_a, 0, fft=fft)


@pytest.mark.parametrize("bits", [16, 2])
@pytest.mark.parametrize("cap", [0, 2048])
def test_rows_capacity_and_lists(bits, cap):
    T, B, n_s = 1248, 2, 201
    print(f"[case] bits {bits} capacity {cap}", flush=True)
    sc = _scores(B, T, "uniform")
    _, scored = _both(1, B, 1, T, 32, n_s, scores=sc, bits=bits, cap=cap)
    best = sc.argsort(dim=1, descending=True)[:, :n_s].to(torch.int32)
    p, listed = _both(1, B, 1, T, 32, n_s, idx=best[:, torch.randperm(n_s, device=DEV)].contiguous(), bits=bits, cap=cap)
    if not cap:                                          # (a list also clears the marks of the room behind the tokens)
        assert all(torch.equal(a, b) for a, b in zip(scored, listed))


def test_equal_channels_and_lists_with_repeats():
    T = 320
    K = torch.randn((1, 1, 2, T, 1), device=DEV).to(torch.float16).expand(1, 1, 2, T, 128).contiguous()
    _both(1, 1, 2, T, 64, 10, scores=_scores(1, T, "ties"), K=K)
    idx = torch.tensor([[5, 5, 319, -1, 320, 0, 0, 64]], dtype=torch.int32, device=DEV)
    _both(1, 1, 2, T, 16, 8, idx=idx)


def test_the_lines_between_few_and_many_groups():
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for heads in (2 * cus - 1, 2 * cus, 2 * cus + 1):        # 2 groups each
        print(f"[case] {heads} heads x 64", flush=True)
        for bits in (16, 2):
            _both(1, 1, heads, 64, 16, 9, scores=_scores(1, 64, "uniform"), bits=bits)
    for B, T in ((1, 8192), (1, 8224), (2, 8192), (1, 8160)):
        print(f"[case] {B} x {T}", flush=True)
        for bits in (16, 2):
            _both(1, B, 1, T, 16, 300, scores=_scores(B, T, "uniform"), bits=bits)
        _both(1, B, 1, T, 16, 300, idx=_scores(B, T, "uniform").argsort(dim=1)[:, :300].to(torch.int32).contiguous())


@pytest.mark.parametrize("n_s", [1, 31, 32, 33, 64, 700, 1055, 1056])
def test_two_bit_records_found_by_rank(n_s):
    print(f"[case] {n_s} of 1056 tokens at 2 bits", flush=True)
    _both(2, 2, 1, 1056, 16, n_s, scores=_scores(2, 1056, "ties"), bits=2)
    _both(1, 1, 4, 4128, 64, min(4 * n_s - 3, 4128), scores=_scores(1, 4128, "uniform"), bits=2)
