"""The binding needs torch only where a call brings a tensor, and its native modules are used only with the library they belong
to; without them every call goes through ctypes."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.exists(os.path.join(ROOT, "paper_2605_11093_amd", "_dmi_python.so"))

# observe_into on a stand-in for the library's entry point: how often it was called natively, how often through ctypes
CALLS = """
import ctypes as C, numpy as np
INTO = C.CFUNCTYPE(C.c_int32, C.c_uint32, *[C.c_void_p] * 3, C.c_uint64, C.c_uint64, C.c_uint32, C.c_void_p, C.c_uint64, C.c_void_p,
                   C.c_void_p)
native, general = [], []
entry = INTO(lambda *a: native.append(a) or 0)
def call(torch, times=2):
    x, out = torch.zeros(3, 8, dtype=torch.float16), torch.zeros(64, dtype=torch.uint8)
    for _ in range(times):
        B.observe_into(1, x, np.zeros((1, 5), dtype=np.uint32), out, seq=0, step_id=0)
"""


def _run(code, path=()):
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([*path, ROOT]))
    p = subprocess.run([sys.executable, "-c", CALLS + textwrap.dedent(code)], env=env, cwd=ROOT, timeout=240,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    assert p.returncode == 0, p.stdout.decode(errors="replace")[-4000:]


def test_importing_the_package_does_not_import_torch():
    _run("""
        import sys
        import paper_2605_11093_amd as dmi
        from paper_2605_11093_amd import binding as B
        assert "gfx950" in dmi.version() and "torch" not in sys.modules
    """)


@pytest.mark.parametrize("error", ["OSError", "ImportError", "RuntimeError"])
def test_a_torch_that_cannot_be_imported(tmp_path, error):
    (tmp_path / "torch").mkdir()
    (tmp_path / "torch" / "__init__.py").write_text(f"raise {error}('libtorch is not there')\n")
    _run("""
        import sys
        from paper_2605_11093_amd import binding as B
        assert "gfx950" in B.version() and B.record_bytes(4, 4, 256, 1, 0) == 2176
        try:
            import torch
        except Exception:
            pass
        assert "torch" not in sys.modules
    """, [str(tmp_path)])


@pytest.mark.skipif(not NATIVE, reason="the native module has not been built")
@pytest.mark.parametrize("first", ["torch", "binding", "library"])
def test_the_first_call_with_a_tensor_is_native(first):
    _run(f"""
        import sys
        if {first == "torch"}:
            import torch
        from paper_2605_11093_amd import binding as B
        if {first == "library"}:
            B.lib()
        import torch
        B.lib()
        assert B._native_ok and ("paper_2605_11093_amd._dmi_python_torch" in sys.modules) == {first != "library"}
        B._native.bind_into(C.cast(entry, C.c_void_p).value)
        B._into_raw = lambda: lambda *a: general.append(a) or 0
        call(torch)
        assert len(native) == 2 and not general and "paper_2605_11093_amd._dmi_python_torch" in sys.modules
    """)


@pytest.mark.skipif(not NATIVE, reason="the native module has not been built")
def test_a_reader_that_cannot_be_loaded():
    _run("""
        import sys
        import paper_2605_11093_amd.build
        sys.modules["paper_2605_11093_amd._dmi_python_torch"] = None        # (an import of it fails)
        from paper_2605_11093_amd import binding as B
        import torch
        B.lib()
        B._native.bind_into(C.cast(entry, C.c_void_p).value)
        B._into_raw = lambda: lambda *a: general.append(a) or 0
        call(torch)
        assert not native and len(general) == 2
    """)


@pytest.mark.skipif(not NATIVE, reason="the native module has not been built")
def test_native_modules_of_another_library():
    _run("""
        from paper_2605_11093_amd import binding as B
        import torch
        B._native.HEADER_DIGEST ^= 1
        B.lib()
        assert not B._native_ok
        B._into_raw = lambda: lambda *a: general.append(a) or 0
        call(torch)
        assert len(general) == 2

        class Ring:
            _h = C.c_void_p(0x1000)
        p = B.PreparedObserve(Ring, 1, torch.zeros(3, 8, dtype=torch.float16), [[0, 0, 0, 1, 1]])
        p._fn = lambda *a: general.append(a) or 0
        assert p(5, 6) == 0 and general[-1][-2:] == (5, 6)
    """)


def test_a_native_module_of_other_sources():
    _run("""
        import sys, types
        import paper_2605_11093_amd.build                   # (the package, and what builds that module, import all the same)
        for k in [k for k in sys.modules if k.startswith("paper_2605")]:
            del sys.modules[k]
        sys.modules["paper_2605_11093_amd._dmi_python"] = types.ModuleType("_dmi_python")
        from paper_2605_11093_amd import binding as B
        assert B._native is None and "gfx950" in B.version()
    """)


def test_a_prepared_observe_can_be_copied():
    _run("""
        import copy
        from paper_2605_11093_amd import binding as B
        import torch
        B.lib()

        class Ring:
            _h = C.c_void_p(0x1000)
        p = B.PreparedObserve(Ring, 1, torch.zeros(3, 8, dtype=torch.float16), [[0, 0, 0, 1, 1]])
        q = copy.copy(p)
        assert q._ra is p._ra and type(q) is B.PreparedObserve
        q._fn = lambda *a: general.append(a) or 0
        assert q(5, 6) == 0 and general[-1][-2:] == (5, 6)
    """)
