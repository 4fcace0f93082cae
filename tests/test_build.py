"""Building without torch: the library, the plain-C caller and the binding need none."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import sys
sys.modules["torch"] = None  # import torch raises ImportError
sys.path.insert(0, {root!r})
from paper_2608_20818_amd import build as b
done = []
b.build = lambda: done.append("library")
b.build_c_caller = lambda: done.append("caller")
import __graft_entry__ as g
g.build()
assert done == ["library", "caller"], done
import paper_2608_20818_amd as prm
assert prm.schedule_is_refresh(4, 2) == 1
assert prm._Tensors([(2, 3)], prm.F32, True).pointers([1]) is None
print("built")
"""


def test_build_without_torch():
    r = subprocess.run([sys.executable, "-c", CODE.format(root=ROOT)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "built" in r.stdout, r.stderr[-2000:]
    assert "no torch" in r.stderr


def test_build_without_headers(tmp_path, monkeypatch, capsys):
    import sysconfig

    from paper_2608_20818_amd import build as b
    paths = dict(sysconfig.get_paths(), include=str(tmp_path))
    monkeypatch.setattr(sysconfig, "get_paths", lambda *a, **k: paths)
    assert b.build_marshal() == ""
    assert "Python.h" in capsys.readouterr().err
