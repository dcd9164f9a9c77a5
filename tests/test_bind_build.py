"""The compiled tensor marshalling belongs to one torch: one that was built for
another is not loaded, and where there is none it is compiled on first use."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2604_27210_amd import _native as N
from paper_2604_27210_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_another_torch_has_its_own(monkeypatch):
    import torch
    N.bind()
    here = build.bind_path()
    assert os.path.exists(here) and torch.__version__ in here
    monkeypatch.setattr(torch, "__version__", "0.0.1")
    assert build.bind_path() != here and not os.path.exists(build.bind_path())
    monkeypatch.setattr(N, "_bind", None)

    def no_compiler(*a, **k):
        raise FileNotFoundError("g++")

    monkeypatch.setattr(build.subprocess, "run", no_compiler)
    with pytest.raises(N.FastvolError, match="no tensor marshalling for torch here .*0.0.1.*g[+][+]"):
        N.bind()
    assert N._bind is None


def test_a_library_alone_is_enough(tmp_path):
    """The sources without their builds, FASTVOL_LIBRARY naming the library."""
    shutil.copytree(os.path.join(ROOT, "paper_2604_27210_amd"), str(tmp_path / "paper_2604_27210_amd"),
                    ignore=shutil.ignore_patterns("_build", "__pycache__"))
    shutil.copytree(os.path.join(ROOT, "include"), str(tmp_path / "include"))
    code = ("import torch, paper_2604_27210_amd as fv\n"
            "v = torch.ones(4, dtype=torch.float64)\n"
            "try:\n"
            "    fv.price('bs', v, v, 1.0, 0.0, 0.2)\n"
            "except ValueError as e:\n"
            "    print('refused:', e)\n")
    env = dict(os.environ, FASTVOL_LIBRARY=N.LIB_PATH)
    res = subprocess.run([sys.executable, "-c", code], cwd=str(tmp_path), env=env, capture_output=True, text=True)
    assert "refused: fs must be on the GPU" in res.stdout, res.stderr[-2000:]
    assert len(os.listdir(str(tmp_path / "paper_2604_27210_amd" / "_build"))) == 1
