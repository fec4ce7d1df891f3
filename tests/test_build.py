"""CPU: what the library's build and import do without, shown with a library of one small source."""
import os
import subprocess
import sys
import sysconfig

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("missing", ["torch", "compiler", "headers"])
def test_the_library_is_built_without_the_native_calls(missing, tmp_path, monkeypatch, capsys):
    from paper_2510_02822_amd import build as b

    def no_torch():
        raise ImportError("No module named 'torch'")

    commands = {"torch": no_torch, "compiler": lambda: [str(tmp_path / "no-such-compiler")],
                "headers": lambda: ["g++", "-x", "c++", "-include", "no_such_header.h", "-c", str(tmp_path / "one.hip"), "-o", str(tmp_path / "x.o")]}
    (tmp_path / "one.hip").write_text("extern \"C\" int one() { return 1; }\n")
    (tmp_path / "_calls.so").write_text("of other sources")
    monkeypatch.setattr(b, "CSRC", str(tmp_path))
    monkeypatch.setattr(b, "LIB", str(tmp_path / "one.so"))
    monkeypatch.setattr(b, "CALLS", str(tmp_path / "_calls.so"))
    monkeypatch.setattr(b, "UNITS", [("one.hip", "one.o", [])])
    monkeypatch.setattr(b, "_calls_command", commands[missing])
    assert b.build() == str(tmp_path / "one.so") and os.path.exists(tmp_path / "one.so")
    assert not os.path.exists(tmp_path / "_calls.so") and "native calls were not built" in capsys.readouterr().err
    # what the library itself needs still ends the build, and says which command it was
    (tmp_path / "one.hip").write_text("#error not this\n")
    with pytest.raises(RuntimeError, match="hipcc failed"):
        b.build()


@pytest.mark.parametrize("before", ["import sys; sys.modules['torch'] = None", "import torch; torch.__version__ = 'another'",
                                    "import sys; sys.modules['paper_2510_02822_amd._calls'] = None"])
def test_imported_without_the_native_calls(before):
    """No torch, another torch than the native calls were built for, no native calls: the package is there, with Python's functions."""
    program = before + """
import types
import paper_2510_02822_amd as fq
from paper_2510_02822_amd import build
assert fq.binding._calls is None and fq.Layer.__mro__ == (fq.Layer, object)
assert type(fq.flexiq_mixed_gemm) is types.FunctionType and not hasattr(fq.flexiq_mixed_gemm, '__wrapped__')
if fq.binding.os.path.exists(fq.binding.LIB_PATH):
    fq.load()
"""
    subprocess.check_call([sys.executable, "-c", program], cwd=ROOT)


def test_native_calls_are_for_this_python_and_this_torch():
    import torch
    import paper_2510_02822_amd as fq
    from paper_2510_02822_amd import build
    assert build.CALLS.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and os.path.samefile(fq.binding._calls.__file__, build.CALLS)
    assert fq.binding._calls.built_for == torch.__version__
