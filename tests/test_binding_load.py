"""Loading of the extension with the Python callables: a missing one, one that does not load, one that appears later.
Each case runs in a process of its own on a copy of the package's Python files."""
import os
import shutil
import subprocess
import sys

import pytest

import paper_2412_20386_amd as ptq
from paper_2412_20386_amd import build as hip_build

PACKAGE = os.path.dirname(os.path.abspath(ptq.__file__))
PRELUDE = """
import os, shutil, sys
sys.path.insert(0, os.getcwd())
import paper_2412_20386_amd as ptq
from paper_2412_20386_amd import quantize_pts as early
assert os.path.dirname(os.path.dirname(os.path.abspath(ptq.__file__))) == os.getcwd()
def message(call):
    try:
        call()
    except Exception as err:
        return type(err).__name__ + ": " + str(err)
"""


def _run(tmp_path, code, extension=None):
    if not (os.path.exists(ptq.binding.LIB_PATH) and os.path.exists(ptq.binding.CALLS_PATH)):
        hip_build.build()
    copy = tmp_path / "paper_2412_20386_amd"
    copy.mkdir()
    for name in os.listdir(PACKAGE):
        if name.endswith(".py"):
            shutil.copy(os.path.join(PACKAGE, name), copy)
    if extension is not None:
        (copy / os.path.basename(ptq.binding.CALLS_PATH)).write_bytes(extension)
    env = dict(os.environ, PTQ4VM_LIB=ptq.binding.LIB_PATH, GOOD=ptq.binding.CALLS_PATH)
    res = subprocess.run([sys.executable, "-c", PRELUDE + code], cwd=tmp_path, env=env, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr


@pytest.mark.parametrize("extension", [None, b"", b"\x7fELF cut short", b"not a library"])
def test_import_without_a_usable_extension(tmp_path, extension):
    """The package imports (its build module is the remedy), and a call says what to do."""
    _run(tmp_path, """
from paper_2412_20386_amd import build
for call in (early, ptq.quantize_pts, ptq.binding.w8a8_linear):
    text = message(lambda: call())
    assert "python -m paper_2412_20386_amd.build" in text and text.split(":")[0] in ("ImportError", "FileNotFoundError"), text
""", extension)


def test_extension_that_appears_after_the_import(tmp_path):
    """It is bound once, by the first call, and then stands in the package itself."""
    _run(tmp_path, """
assert "python -m" in message(lambda: early())
stand_in = ptq.w8a8_linear
shutil.copy(os.environ["GOOD"], ptq.binding.CALLS_PATH)
assert "missing required argument" in message(lambda: early())
binds = []
bind = ptq.binding._bind_calls
ptq.binding._bind_calls = lambda: (binds.append(1), bind())
for name in ptq.binding.HOT_CALLS:
    call = getattr(ptq.binding._calls, name)
    assert getattr(ptq, name) is call and getattr(ptq.binding, name) is call
for call in (early, stand_in):
    assert "missing required argument" in message(lambda: call())
assert not binds
""")


def test_extension_without_one_of_the_callables(tmp_path):
    """An extension of other sources is refused as a whole."""
    _run(tmp_path, """
shutil.copy(os.environ["GOOD"], ptq.binding.CALLS_PATH)
ptq.binding.HOT_CALLS += ("brand_new_call",)
text = message(lambda: early())
assert text.startswith("ImportError") and "brand_new_call" in text and "python -m" in text, text
""")
