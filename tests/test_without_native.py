"""The package without its _native extension (not built, or built against
another torch): it imports, says so, and its functions take the Python path."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import importlib.abc, sys, warnings
class Blocked(importlib.abc.MetaPathFinder):
    def find_spec(self, name, path=None, target=None):
        if name == "paper_2006_12838_amd._native":
            raise ImportError("undefined symbol")
sys.meta_path.insert(0, Blocked())
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    import paper_2006_12838_amd as P
assert any("_native" in str(x.message) and x.category is RuntimeWarning for x in w), w
import torch
n, V0, phi = torch.rand(5, 3), torch.rand(5), torch.rand(4, 4, 4)
for call in (lambda: P.offset(n, V0), lambda: P.offset(tuple(n.unbind(-1)), V0), lambda: P.volume(n, V0),
             lambda: P.curvature(phi)):
    try:
        call()
    except ValueError as e:            # the library's own check: tensors on a GPU
        assert "GPU" in str(e), e
    else:
        raise AssertionError("accepted CPU tensors")
print("ok")
"""


def test_imports_and_takes_the_python_path():
    r = subprocess.run([sys.executable, "-c", PROGRAM], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stderr
