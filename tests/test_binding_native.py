"""The native call layer takes plain arguments only and leaves every refusal to the Python path: the errors are
the same with and without it, and no exception of C++ leaves it (nothing here reaches a launch)."""
import ctypes as C
import importlib
import os
import shutil
import sys
import types

import pytest
import torch

from paper_2503_16257_amd import binding as vk
from paper_2503_16257_amd import build as B

PARAM_BYTES, SIDE_BYTES = C.sizeof(vk.VidkvParams), C.sizeof(vk.VidkvSideStream)


class ForeignParams(C.Structure):
    _fields_ = [("words", C.c_int32 * (PARAM_BYTES // 4))]


class ForeignSide(C.Structure):
    _fields_ = [("words", C.c_void_p * (SIDE_BYTES // 8))]


FOREIGN_PARAMS = [bytes(PARAM_BYTES), bytearray(PARAM_BYTES), memoryview(bytes(PARAM_BYTES)), (C.c_int32 * (PARAM_BYTES // 4))(),
                  ForeignParams()]
FOREIGN_SIDES = [bytes(SIDE_BYTES), bytearray(SIDE_BYTES), (C.c_void_p * (SIDE_BYTES // 8))(), ForeignSide()]
REFUSED = (TypeError, C.ArgumentError)                 # what ctypes raises


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


@pytest.mark.parametrize("foreign", FOREIGN_PARAMS, ids=lambda f: type(f).__name__)
def test_a_buffer_of_the_size_of_the_parameters_is_refused(foreign):
    with pytest.raises(REFUSED):
        vk.decode_attention_noalloc(foreign, 0, None, None, None, None, stream=types.SimpleNamespace(cuda_stream=0))
    assert vk._native.decode_attention_noalloc(foreign, 0, *[None] * 5, 0, None, None, lambda s: 0, None) is None


def test_a_structure_derived_from_the_parameters_is_taken_where_it_adds_nothing():
    class Same(vk.VidkvParams):
        pass

    class Longer(vk.VidkvParams):
        _fields_ = [("more", C.c_int32)]

    vk.lib()
    args = (0, *[None] * 5, 0, None, None, lambda s: 0, None)
    assert vk._native.decode_attention_noalloc(Same(), *args) == vk.EINVAL
    assert vk._native.decode_attention_noalloc(Longer(), *args) is None
    # (the Python path takes it, as a pointer to its first part)
    with pytest.raises(vk.VidkvError):
        vk.decode_attention_noalloc(Longer(), 0, None, None, None, None, stream=types.SimpleNamespace(cuda_stream=0))


@pytest.mark.gpu
def test_foreign_structures_are_refused_with_tensors_in_place():
    """Parameters and side stream of each call, everything else in order (no launch: refused in front of the library)."""
    z = lambda n, t: torch.zeros(n, dtype=t, device="cuda:0")
    p = vk.make_params(1, 1, 1, 2, 32, 16, 0, t_capacity=64)
    q, tail, pk = z((1, 2, 128), torch.float16), z((1, 1, 32, 128), torch.float16), z(vk.packed_keys_bytes(p), torch.uint8)
    pv, ws = z(vk.packed_values_bytes(p), torch.uint8), z(vk.workspace_bytes(p, 2), torch.uint8)
    for f in FOREIGN_PARAMS:
        for call in (lambda: vk.decode_attention(f, 0, q, pk, pv, q, ws), lambda: vk.decode_attention_noalloc(f, 0, q, pk, pv, q),
                     lambda: vk.flush_residual(f, 0, tail, tail, 32, 32, pk, pv)):
            with pytest.raises(REFUSED):
                call()
    for f in FOREIGN_SIDES:
        with pytest.raises(REFUSED):
            vk.decode_attention(p, 0, q, pk, pv, q, ws, side=types.SimpleNamespace(c=f))


@pytest.mark.parametrize("layer", ["missing", "not loadable", "of another torch", "of older source"])
def test_without_the_layer_every_call_takes_the_python_path(layer, tmp_path, monkeypatch):
    """A package that holds the library and no native layer that fits: everything works as it did before there was one."""
    name = "vidkv_copy_" + layer.replace(" ", "_")
    d = tmp_path / name
    d.mkdir()
    here = os.path.dirname(vk.__file__)
    shutil.copy(os.path.join(here, "binding.py"), d)
    (d / "__init__.py").write_text("")
    os.symlink(vk.LIB_PATH, d / "libvidkv.so")
    if layer == "not loadable":
        (d / "vidkv_marshal.so").write_bytes(b"no shared object")
    elif layer != "missing":
        tag = 'built_for = "cpython-00 torch 0.0"\n' if layer == "of another torch" else ""
        (d / "vidkv_marshal.py").write_text(tag + "def bind(*a):\n    raise RuntimeError('taken')\n")
    monkeypatch.syspath_prepend(str(tmp_path))
    try:
        v = importlib.import_module(name + ".binding")
        p = v.make_params(1, 1, 1, 2, 32, 16, 0)
        assert v.packed_keys_bytes(p) == vk.packed_keys_bytes(vk.make_params(1, 1, 1, 2, 32, 16, 0)) > 0
        assert v._native is None
        s = types.SimpleNamespace(cuda_stream=0)
        with pytest.raises(v.VidkvError, match="invalid argument"):
            v.decode_attention_noalloc(p, 0, None, None, None, None, stream=s)
        cpu = torch.zeros((1, 2, 128), dtype=torch.float16)
        for call in (lambda: v.decode_attention(p, 0, cpu, None, None, None, cpu, stream=s),
                     lambda: v.decode_attention_noalloc(p, 0, cpu, None, None, None, stream=s),
                     lambda: v.flush_residual(p, 0, cpu, cpu, 32, 32, cpu, cpu, stream=s)):
            with pytest.raises(TypeError, match="expected a CUDA tensor"):
                call()
    finally:
        for m in [m for m in sys.modules if m == name or m.startswith(name + ".")]:
            del sys.modules[m]


def test_the_layer_built_here_is_used():
    vk.lib()
    assert vk._native is not None and vk._native.built_for == vk.native_tag()


def test_the_library_is_built_where_the_layer_cannot_be(tmp_path, monkeypatch, capsys):
    """No torch or Python headers, no g++: the library alone, and no layer of an older build beside it."""
    stale = tmp_path / "vidkv_marshal.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(B, "MARSHAL", str(stale))
    monkeypatch.setattr(B, "OBJ", str(tmp_path))
    monkeypatch.setattr(B, "_compile", lambda src: str(tmp_path / src))
    ran = []

    def run(cmd, **kw):
        ran.append(cmd)
        if cmd[0] == "g++":
            raise FileNotFoundError("g++")
        return types.SimpleNamespace(returncode=0, stderr="")

    monkeypatch.setattr(B.subprocess, "run", run)
    assert B.build(verbose=False) == B.LIB
    assert [c[0] for c in ran].count("g++") == 1 and len(ran) == 2 and not stale.exists()
    assert "vidkv_marshal.so" in capsys.readouterr().err


_DTYPE = {"q": torch.float16, "pk": torch.uint8, "pv": torch.uint8, "Kt": torch.float16, "Vt": torch.float16,
          "tl": torch.int32, "out": torch.float16, "ws": torch.uint8}
_OF_CALL = {"decode_attention": ["q", "pk", "pv", "Kt", "Vt", "tl", "out", "ws"],
            "decode_attention_noalloc": ["q", "pk", "pv", "Kt", "Vt", "tl", "out"],
            "flush_residual": ["Kt", "Vt", "pk", "pv"]}


@pytest.mark.gpu
@pytest.mark.parametrize("call,name", [(c, n) for c, names in _OF_CALL.items() for n in names])
def test_device_tensors_that_do_not_fit_are_refused(call, name):
    """One tensor of a call that would pass is of another type, not contiguous, or not on the device (raised in front of
    any launch); the call itself passes, and leaves what the Python path leaves."""
    p = vk.make_params(1, 1, 1, 2, 32, 16, 0, t_capacity=64)
    size = {"pk": (vk.packed_keys_bytes(p),), "pv": (vk.packed_values_bytes(p),), "ws": (vk.workspace_bytes(p, 2),), "tl": (1,),
            "q": (1, 2, 128), "out": (1, 2, 128), "Kt": (1, 1, 32, 128), "Vt": (1, 1, 32, 128)}
    good = {n: torch.zeros(size[n], dtype=t, device="cuda:0") for n, t in _DTYPE.items()}

    def run(t):
        if call == "flush_residual":
            vk.flush_residual(p, 0, t["Kt"], t["Vt"], 32, 32, t["pk"], t["pv"])
        else:
            ws = (t["ws"],) if call == "decode_attention" else ()
            getattr(vk, call)(p, 0, t["q"], t["pk"], t["pv"], t["out"], *ws, K_tail=t["Kt"], V_tail=t["Vt"], tail_capacity=32,
                              tail_len=t["tl"])

    other = {torch.float16: (torch.bfloat16, torch.float32), torch.uint8: (torch.int8, torch.float16),
             torch.int32: (torch.int64, torch.float32)}[_DTYPE[name]]
    for t in other:
        with pytest.raises(TypeError, match="expected dtype"):
            run({**good, name: torch.zeros(size[name], dtype=t, device="cuda:0")})
    # (one element is contiguous whatever its stride: two, every other one of four)
    strided = torch.zeros(size[name][:-1] + (2 * max(size[name][-1], 2),), dtype=_DTYPE[name], device="cuda:0")[..., ::2]
    with pytest.raises(ValueError, match="must be contiguous"):
        run({**good, name: strided})
    with pytest.raises(TypeError, match="expected a CUDA tensor"):
        run({**good, name: good[name].cpu()})
    run(good)
    native, vk._native = vk._native, None
    try:
        again = {n: torch.zeros_like(t) for n, t in good.items()}
        run(again)
    finally:
        vk._native = native
    assert all(torch.equal(good[n], again[n]) for n in ("pk", "pv", "out"))
