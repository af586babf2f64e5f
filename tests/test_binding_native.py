"""The native call layer takes plain arguments only and leaves every refusal to the Python path: the errors are
the same with and without it, and no exception of C++ leaves it (CPU: nothing here reaches a launch)."""
import ctypes as C

import pytest
import torch

from paper_2503_16257_amd import binding as vk


def _args(**kw):
    a = dict(q=torch.zeros((1, 2, 128), dtype=torch.float16), pk=torch.zeros(4096, dtype=torch.uint8),
             pv=torch.zeros(4096, dtype=torch.uint8), out=torch.zeros((1, 2, 128), dtype=torch.float16),
             ws=torch.zeros(4096, dtype=torch.uint8))
    a.update(kw)
    return a


def _calls(a):
    p = vk.make_params(1, 1, 1, 2, 32, 16, 0)
    return [lambda: vk.decode_attention(p, 0, a["q"], a["pk"], a["pv"], a["out"], a["ws"]),
            lambda: vk.decode_attention_noalloc(p, 0, a["q"], a["pk"], a["pv"], a["out"]),
            lambda: vk.flush_residual(p, 0, a["q"], a["q"], 32, 32, a["pk"], a["pv"])]


class _Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("bad", [torch.zeros((1, 2, 128), dtype=torch.float16), "text", 7, torch.zeros(4),
                                 torch.zeros((1, 2, 128), dtype=torch.float16).as_subclass(_Sub),
                                 torch.zeros((1, 2, 128), dtype=torch.float16, device="meta")])
def test_refusals_are_the_python_paths(bad):
    for call in _calls(_args(q=bad)):
        with pytest.raises(TypeError, match="expected a CUDA tensor"):
            call()


def test_under_vmap_the_call_is_refused_as_before():
    x = torch.zeros((3, 1, 2, 128), dtype=torch.float16)

    def f(q):
        for call in _calls(_args(q=q)):
            with pytest.raises((TypeError, RuntimeError)):
                call()
        return q

    torch.vmap(f)(x)


def test_odd_arguments_are_left_to_the_python_path():
    vk.lib()
    n = vk._native
    none14 = [None] * 14
    assert n.decode_attention(*none14) is None and n.decode_attention(1) is None
    assert n.decode_attention_noalloc(*[None] * 12) is None and n.flush_residual(*[None] * 10) is None
    p = vk.make_params(1, 1, 1, 2, 32, 16, 0)
    null = [p, 0, None, None, None, None, None, 0, None, None]
    # a NULL q passes the layer and is refused by the library; a number that is no int32, a foreign structure are not taken
    assert n.decode_attention_noalloc(*null, lambda s: 0, None) == vk.EINVAL
    assert n.decode_attention_noalloc(p, 1 << 40, *null[2:], lambda s: 0, None) is None
    assert n.decode_attention_noalloc(p, True, *null[2:], lambda s: 0, None) is None
    assert n.decode_attention_noalloc((C.c_int * 3)(), *null[1:], lambda s: 0, None) is None
    assert n.decode_attention_noalloc(*null, lambda s: "no handle", None) is None
    with pytest.raises(ZeroDivisionError):
        n.decode_attention_noalloc(*null, lambda s: 1 // 0, None)
