"""CPU checks of the compiled marshalling (csrc/lutgemm_binding.cpp): every argument arrives where the C interface has it, and
what it does not take itself ends as the ctypes functions end it."""
import ctypes
import os
import shutil
import subprocess
import sys
import sysconfig

import numpy as np
import pytest

import paper_2206_09557_amd as L
from paper_2206_09557_amd import lutgemm as M

pytestmark = pytest.mark.skipif("LUTGEMM_LIB" in os.environ, reason="a host-only build has no device calls")

BIG = (1 << 63) + 5      # an address beyond the signed range
LAYER = [ctypes.c_void_p] * 5 + [ctypes.c_int] * 3 + [ctypes.c_int64] * 2
SCRATCH = [ctypes.c_uint, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]


class Buffer:
    def __init__(self, address):
        self.address = address

    def data_ptr(self):
        return self.address


@pytest.fixture
def caught():
    """Calls of the entry points end in Python functions that keep their arguments and return code[0]."""
    calls, code = [], [0]
    types = {"lutgemm_gemv": LAYER + SCRATCH, "lutgemm_gemm": LAYER + [ctypes.c_int] + SCRATCH,
             "lutgemm_gemm_mfma": LAYER + [ctypes.c_int] + SCRATCH,
             "lutgemm_gemm_dequant_mfma": LAYER + [ctypes.c_int] + SCRATCH,
             "lutgemm_gemv_static": LAYER + [ctypes.c_uint, ctypes.c_void_p],
             "lutgemm_gemv_group": [ctypes.c_void_p] * 7 + [ctypes.c_int] * 4 + SCRATCH}
    assert set(types) == set(M._DEVICE_CALLS)

    def catcher(name):
        def f(*args):
            if name == "lutgemm_gemv_group":      # the arrays live as long as the call
                count = args[7]
                read = [None if a is None else list((ctypes.c_uint64 * count).from_address(a)) for a in args[:7]]
                args = tuple(read) + args[7:]
            calls.append((name, args))
            return code[0]
        return ctypes.CFUNCTYPE(ctypes.c_int, *types[name])(f)

    L.lib()
    keep = {name: catcher(name) for name in types}
    M._binding.load({name: ctypes.cast(f, ctypes.c_void_p).value for name, f in keep.items()})
    yield calls, code
    M._binding.load({name: ctypes.cast(getattr(L.lib(), name), ctypes.c_void_p).value for name in types})


def test_is_what_the_package_exports():
    assert M._binding is not None and L.lutgemm_gemv is M._binding.lutgemm_gemv


@pytest.mark.parametrize("name,batch,scratch", [("lutgemm_gemv", (), True), ("lutgemm_gemv_static", (), False), ("lutgemm_gemm", (7,), True),
                                                ("lutgemm_gemm_mfma", (8,), True), ("lutgemm_gemm_dequant_mfma", (9,), True)])
def test_arguments_arrive(caught, name, batch, scratch):
    calls, code = caught
    ws = (Buffer(1 << 50), 1 << 40) if scratch else ()
    args = (Buffer(16), 32, Buffer(BIG), None, Buffer(64), 3, 128, 8, (1 << 40) + 1, -3, *batch, 0xfffffffe, *ws)
    seen = (16, 32, BIG, None, 64, 3, 128, 8, (1 << 40) + 1, -3, *batch, 0xfffffffe, *((1 << 50, 1 << 40) if scratch else ()))
    f = getattr(L, name)
    assert f(*args) is None and f(*args, 0) is None and f(*args, 4096) is None
    assert calls == [(name, seen + (s,)) for s in (None, None, 4096)]
    code[0] = L.LUTGEMM_EUNSUPPORTED
    with pytest.raises(L.LutGemmError) as e:
        f(*args)
    assert e.value.code == L.LUTGEMM_EUNSUPPORTED and name in str(e.value)


@pytest.mark.parametrize("z", [None, [4, Buffer(5)], (4, 5)])
def test_group_arguments_arrive(caught, z):
    calls, _ = caught
    L.lutgemm_gemv_group([Buffer(1), 2], (3, 4), [5, Buffer(6)], z, [7, 8], [9, 10], (11, 12), 2, 64, 8, 1, Buffer(13), 14, 15)
    assert calls == [("lutgemm_gemv_group", ([1, 2], [3, 4], [5, 6], None if z is None else [4, 5], [7, 8], [9, 10], [11, 12], 2, 2, 64, 8,
                                             1, 13, 14, 15))]


def test_the_rest_ends_as_with_ctypes(caught):
    # None of these reaches the functions put in place above: the ctypes function decides (here: y is missing, or it raises).
    calls, _ = caught
    good = dict(x=16, bits=16, alpha=16, z=None, y=None, q=3, g=128, mu=8, m=16, n=128, flags=0, workspace=16, workspace_bytes=100)
    by_ctypes = M._binding.lutgemm_gemv

    def outcome(f, *a, **k):
        try:
            return f(*a, **k)
        except Exception as e:
            return type(e), str(e), getattr(e, "code", None)

    array = np.zeros(8, dtype=np.uint8)
    for change in (dict(), dict(q=np.int64(3)), dict(q=3.0), dict(q=1 << 40), dict(q=True), dict(x="text"), dict(x=array), dict(flags=-1),
                   dict(m="1"), dict(workspace_bytes=-1), dict(x=-1), dict(z=Buffer("none"))):
        k = {**good, **change}
        if not change:
            got = outcome(by_ctypes, **k)                      # keywords
        else:
            got = outcome(by_ctypes, *k.values())
        assert not calls, change
        assert isinstance(got, tuple), (change, got)
    assert outcome(by_ctypes, 1)[0] is TypeError
    assert outcome(by_ctypes, **good)[2] == L.LUTGEMM_EINVAL
    assert outcome(by_ctypes, *{**good, "q": np.int64(3)}.values())[2] == L.LUTGEMM_EINVAL
    assert outcome(by_ctypes, *{**good, "q": 3.0}.values())[0] is ctypes.ArgumentError
    assert outcome(by_ctypes, *{**good, "x": "text"}.values())[:2] == (TypeError, "cannot take the address of <class 'str'>")


def test_is_built_for_this_python_alone():
    assert M._binding.__file__.endswith(sysconfig.get_config_var("EXT_SUFFIX"))


def _import_of_a_copy(tmp_path, code):
    """Output of `code` in a package `lutgemm_copy` of the Python files, in a process of its own."""
    pkg = tmp_path / "lutgemm_copy"
    pkg.mkdir(exist_ok=True)
    for name in ("__init__.py", "lutgemm.py", "build.py"):
        shutil.copy(os.path.join(os.path.dirname(M.__file__), name), pkg / name)
    return subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True, check=True)


def test_one_that_does_not_load_is_reported(tmp_path):
    code = "from lutgemm_copy import lutgemm as M; print(M._binding, type(M.lutgemm_gemv).__name__)"
    absent = _import_of_a_copy(tmp_path, code)
    assert absent.stdout.split() == ["None", "function"] and "marshalling" not in absent.stderr
    (tmp_path / "lutgemm_copy" / ("_binding" + sysconfig.get_config_var("EXT_SUFFIX"))).write_bytes(b"no shared object")
    broken = _import_of_a_copy(tmp_path, code)
    assert broken.stdout.split() == ["None", "function"] and "marshalling of the device calls does not load" in broken.stderr


def test_a_python_without_headers_builds_none(tmp_path, monkeypatch, capsys):
    from paper_2206_09557_amd import build
    built = tmp_path / "_binding.so"
    built.write_bytes(b"of before")
    monkeypatch.setattr(build, "PKG", str(tmp_path))
    monkeypatch.setattr(build, "BINDING", str(built))
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_binding() is None
    assert "ctypes" in capsys.readouterr().out and not built.exists()
