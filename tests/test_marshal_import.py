"""The package without its extension _marshal, or with one of another torch
build: it imports, and the extension is not used (CPU only, in a process of
its own)."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1906_05936_amd")

LOADED = "import paper_1906_05936_amd._lib as l; print(l._marshal is not None)"


def run(script, cwd):
    r = subprocess.run([sys.executable, "-c", script], cwd=cwd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return r.stdout.strip()


@pytest.fixture
def copy(tmp_path):
    """A copy of the package without the extension."""
    if not os.path.exists(os.path.join(PKG, "liblsgd.so")):
        pytest.skip("liblsgd.so is not built")
    d = tmp_path / "paper_1906_05936_amd"
    d.mkdir()
    for name in os.listdir(PKG):
        if name.endswith(".py"):
            shutil.copy(os.path.join(PKG, name), d / name)
    os.symlink(os.path.join(PKG, "liblsgd.so"), d / "liblsgd.so")
    return tmp_path


def test_import_without_the_extension(copy):
    assert run(LOADED, copy) == "False"


def test_extension_of_another_torch_build_is_not_used(copy):
    assert run(LOADED, ROOT) == "True"
    other = "import torch; torch.version.git_version = 'another'\n" + LOADED
    assert run(other, ROOT) == "False"
