"""The extension module behind the binding's hot calls, on functions that record what they are called with: arguments arrive as through ctypes, and
what is not in a hot loop's form is left to ctypes (None, and no call)."""
import ctypes as C

import pytest

from paper_2103_15195_amd import binding as B

vp, i32, u32, u64, f32 = C.c_void_p, C.c_int32, C.c_uint32, C.c_uint64, C.c_float
FORMS = [(i32, vp, i32, u32, u64, vp, vp, vp, vp)] * 2 + [(i32, vp, i32, vp, i32, f32, vp, vp), (i32, vp, u32, u64, vp, vp, vp, vp), (i32, vp, vp, i32, f32, vp, vp)]


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


class Broken:
    def data_ptr(self):
        raise RuntimeError("gone")


@pytest.fixture
def calls():
    seen, keep = [], []
    for f in FORMS:
        keep.append(C.CFUNCTYPE(*f)(lambda *a: seen.append(a) or -len(seen)))
    fast = B._fastcall().Calls(C.Array, *[C.cast(k, vp).value for k in keep])
    return fast, seen, keep


def stream():
    return 0x7000


def test_arguments_arrive(calls):
    fast, seen, _ = calls
    a, b = B.ptr_array([Tensor(16), Tensor(32)]), (vp * 3)(1, 2, 3)
    at, bt = C.addressof(a), C.addressof(b)
    raw = B._fastcall().RawStream(lambda d: 0x100 + d, lambda: 3)
    big = 2 ** 64 - 1
    assert fast.compress(0xFFFF000000000010, 2, 2 ** 32 + 5, 2 ** 64 + 7, a, None, Tensor(big - 15), stream) == -1
    assert seen[-1] == (0xFFFF000000000010, 2, 5, 7, at, None, big - 15, 0x7000)
    assert fast.compress_static(8, True, 0, 1, a, Tensor(64), Tensor(128), raw) == -2
    assert seen[-1] == (8, 1, 0, 1, at, 64, 128, 0x103)
    assert fast.decompress(8, -1, b, 0.1, a, stream) == -3
    assert seen[-1] == (8, -1, bt, 3, C.c_float(0.1).value, at, 0x7000)
    assert fast.compress_groups(0, 1, 2, a, None, b, stream) == -4
    assert seen[-1] == (None, 1, 2, at, None, bt, 0x7000)
    assert fast.compress_groups(8, 1, 2, a, b, b, stream) == -5 and seen[-1][4] == bt
    assert fast.decompress_groups(8, b, 3, float("inf"), a, stream) == -6
    assert seen[-1] == (8, bt, 3, float("inf"), at, 0x7000)


def test_other_forms_are_left_to_ctypes(calls):
    fast, seen, _ = calls
    a, t = (vp * 1)(1), Tensor(16)
    good = {"compress": (8, 0, 0, 0, a, t, t, stream), "decompress": (8, 0, a, 1.0, a, stream), "compress_groups": (8, 0, 0, a, a, a, stream),
            "decompress_groups": (8, a, 1, 1.0, a, stream)}

    def fails():
        raise RuntimeError("no device")
    for name, args in good.items():
        f = getattr(fast, name)
        assert f(*args[:-1]) is None and f(*args, 1) is None
        for i, arg in enumerate(args):
            for bad in {"int": [1.5, "1", None], "float": [1, "1", None], "c_void_p_Array_1": [[t], (1,), t, b"x"],
                        "Tensor": [Broken(), 5, a], "function": [None, fails, lambda: None]}[type(arg).__name__]:
                assert f(*args[:i], bad, *args[i + 1:]) is None, (name, i, bad)
    assert not seen
    with pytest.raises(TypeError):
        B._fastcall().Calls(C.Array, 1, 2, 3)


@pytest.fixture
def no_module(monkeypatch):
    """The package without its extension module."""
    import sys

    import paper_2103_15195_amd as package
    monkeypatch.setitem(sys.modules, package.__name__ + "._fastcall", None)
    monkeypatch.delattr(package, "_fastcall", raising=False)


def test_the_binding_does_without_the_module(no_module, monkeypatch):
    with pytest.raises(ImportError):
        B._fastcall()
    monkeypatch.setattr(B, "_lib", None)
    with pytest.warns(UserWarning, match="ctypes"):
        fast = B.lib().fast
    args = (8, 0, 0, 0, None, None, None, None)
    assert [getattr(fast, name)(*args) for name in ("compress", "compress_static", "decompress", "compress_groups", "decompress_groups")] == [None] * 5
    assert B.mc_partition([3, 4, 5], 2) == [0, 2, 3]


def test_the_stream_is_found_without_the_module(no_module, monkeypatch):
    import torch
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: None)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 0x100 + d, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(B, "_raw_stream", None)
    assert B._current_stream() == 0x103


@pytest.mark.parametrize("compiler", ["/nowhere/to/be/found", "false"])
def test_the_library_is_built_where_the_module_cannot_be(monkeypatch, tmp_path, compiler):
    from paper_2103_15195_amd import build as hip_build
    ran = []
    run = hip_build._run
    monkeypatch.setattr(hip_build, "_run", lambda cmd, verbose: ran.append(cmd[0]) if "hipcc" in cmd[0] else run(cmd, verbose))
    monkeypatch.setattr(hip_build, "FASTCALL", str(tmp_path / "_fastcall.tag.so"))
    monkeypatch.setenv("CXX", compiler)
    monkeypatch.setenv("HIPCC", "hipcc")
    with pytest.warns(UserWarning, match="ctypes"):
        assert hip_build.build() == hip_build.LIB
    assert ran == ["hipcc"]


def test_the_module_is_this_interpreters(monkeypatch, tmp_path):
    import importlib.machinery
    import os

    from paper_2103_15195_amd import build as hip_build
    assert B._fastcall().__file__ == hip_build.FASTCALL
    tag = os.path.basename(hip_build.FASTCALL)[len("_fastcall"):]
    assert tag == importlib.machinery.EXTENSION_SUFFIXES[0] != ".so"
    (tmp_path / "_fastcall.so").write_text("of another interpreter")
    monkeypatch.setattr(hip_build, "FASTCALL", str(tmp_path / ("_fastcall" + tag)))
    assert hip_build.build_fastcall()
    assert os.listdir(tmp_path) == ["_fastcall" + tag]
