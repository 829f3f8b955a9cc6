"""How the binding finds its native part: importing the package needs neither a compiler nor the built file, a file of other
sources or another torch is not loaded, and where none can be had the general path serves every call."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = "paper_2505_07291_amd"


@pytest.fixture
def tree(tmp_path):
    """A copy of the package with the library, without the native part, and a PATH without compilers."""
    shutil.copytree(os.path.join(ROOT, PKG), tmp_path / PKG, ignore=shutil.ignore_patterns("_fastcall*", "__pycache__"))
    shutil.copytree(os.path.join(ROOT, "include"), tmp_path / "include")
    (tmp_path / "bin").mkdir()

    def go(code):
        env = dict(os.environ, PATH=str(tmp_path / "bin"), PYTHONPATH=str(tmp_path), PYTHONDONTWRITEBYTECODE="1")
        r = subprocess.run([sys.executable, "-W", "always", "-c", code], env=env, cwd=tmp_path, capture_output=True, text=True,
                           timeout=300)
        assert r.returncode == 0, r.stderr[-3000:]
        return r.stdout, r.stderr
    return tmp_path, go


USE = """
import paper_2505_07291_amd as grpo
from paper_2505_07291_amd import binding
assert binding.__file__.startswith(%r), binding.__file__
import threading
threads = [threading.Thread(target=grpo.grpo_workspace_bytes, args=(1,)) for _ in range(4)]  # one of them loads
[t.start() for t in threads], [t.join() for t in threads]
assert grpo.grpo_workspace_bytes(1) > 0
print("native" if binding._fast.__class__.__name__ == "module" else binding._fast.total_rewards(1, 2, 3, 4))
grpo.lib()
"""


def test_import_and_calls_without_a_native_part(tree):
    path, go = tree
    out, err = go("import paper_2505_07291_amd, sys; print(paper_2505_07291_amd.GRPO_BF16)")
    assert out == "1\n" and "Warning" not in err
    out, err = go(USE % str(path))
    assert out == "None\n" and err.count("RuntimeWarning") == 1 and "general Python path" in err


def test_a_file_that_does_not_load_is_not_fatal(tree):
    path, go = tree
    name, _ = go("from paper_2505_07291_amd import build; print(build.fastcall_path())")
    with open(name.strip(), "w") as f:
        f.write("no shared object")
    out, err = go(USE % str(path))
    assert out == "None\n" and err.count("RuntimeWarning") == 1


def test_a_native_part_of_other_sources_is_not_loaded(tree):
    import paper_2505_07291_amd.build as build
    path, go = tree
    built = build.fastcall_path()
    if not os.path.exists(built):
        build.build_fastcall()
    shutil.copy(built, path / PKG / os.path.basename(built))
    shutil.copy(built, path / PKG / "_fastcall.so")  # the name without sources
    out, err = go(USE % str(path))
    assert out == "native\n" and "Warning" not in err
    with open(path / "include" / "grpo.h", "a") as f:
        f.write("/* an argument more */\n")
    out, err = go(USE % str(path))
    assert out == "None\n" and err.count("RuntimeWarning") == 1
    stale, _ = go("from paper_2505_07291_amd import build; print(build.is_stale())")
    assert stale == "True\n"
