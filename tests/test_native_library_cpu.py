"""Which files the PyTorch layers run on: the native functions beside libsk.so go through that libsk.so, wherever the package lies."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = "paper_2601_15473_amd"


def _copy(to):
    shutil.copytree(os.path.join(ROOT, PACKAGE), os.path.join(to, PACKAGE), ignore=shutil.ignore_patterns("csrc", "__pycache__"))
    return str(to)


def _run(where, code):
    """The last line that `code` prints in a fresh interpreter whose package lies in `where`."""
    env = {k: v for k, v in os.environ.items() if k not in ("PYTHONPATH", "LD_LIBRARY_PATH")}
    r = subprocess.run([sys.executable, "-c", code], cwd=where, env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return r.stdout.strip().splitlines()[-1]


MAPPED = """
mapped = sorted({l.split()[-1] for l in open('/proc/self/maps') if l.rstrip().endswith(('/libsk.so', '/_sktorch.so'))})
"""


def test_a_copied_package_runs_its_own_library(tmp_path):
    where = _copy(tmp_path)
    got = _run(where, "from paper_2601_15473_amd import nn\n" + MAPPED + "print(nn._native is not None, *mapped)")
    lib = os.path.join(where, PACKAGE, "lib")
    assert got == f"True {lib}/_sktorch.so {lib}/libsk.so"


def test_native_functions_refuse_another_packages_library(tmp_path):
    """Two packages in one process: the loader has one libsk.so by name, and the second's native functions would run on the first's."""
    second = os.path.join(_copy(tmp_path), PACKAGE, "lib", "_sktorch.so")
    got = _run(ROOT, f"""
import importlib.util
from paper_2601_15473_amd import nn
spec = importlib.util.spec_from_file_location("_sktorch", {second!r})
try:
    importlib.util.module_from_spec(spec)
    print("loaded")
except ImportError as e:
    print(e)
""")
    assert "libsk.so" in got and ROOT in got, got


@pytest.mark.parametrize("torch_is", ["this one", "another"])
def test_layers_without_their_native_functions(tmp_path, torch_is):
    """Missing, or built for another PyTorch: a warning, and the Python functions serve every call (here: their refusal of CPU tensors)."""
    where = _copy(tmp_path)
    if torch_is == "this one":
        os.remove(os.path.join(where, PACKAGE, "lib", "_sktorch.so"))
    got = _run(where, f"""
import warnings, torch
if {torch_is == "another"}:
    torch.__version__ = torch.torch_version.TorchVersion("2.9.1")
with warnings.catch_warnings(record=True) as said:
    warnings.simplefilter("always")
    from paper_2601_15473_amd import nn
nn.release_workspaces()
try:
    nn.sklinear(torch.zeros(4, 32), torch.zeros(32, 16), torch.zeros(16, 48), None, 1, 16)
except RuntimeError as e:
    print(nn._native, [w.category.__name__ for w in said if "native functions" in str(w.message)], "GPU only" in str(e))
""")
    assert got == "None ['RuntimeWarning'] True"


def test_build_without_pytorch(tmp_path):
    """libsk.so alone, as its callers without PyTorch need it (the compiler steps replaced: what is asked for is looked at)."""
    got = _run(ROOT, f"""
import sys
sys.modules["torch"] = None
from paper_2601_15473_amd import build as b
done = []
b.OUT = {str(tmp_path / "libsk.so")!r}
b._compile = lambda src, obj: done.append(src)
b.subprocess.run = lambda cmd, **kw: done.append(cmd[-1]) or __import__("types").SimpleNamespace(returncode=0, stderr="")
b.build(verbose=False)
print(len(done) == len(b.SOURCES) + 1, done[-1] == b.OUT)
""")
    assert got == "True True"
