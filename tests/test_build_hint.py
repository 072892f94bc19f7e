"""Importing the package with one of its built libraries missing names the build."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = "paper_2609_03844_amd"


@pytest.mark.parametrize("missing", ["libsbw.so", "_binding.so"])
def test_missing_library_names_the_build(tmp_path, missing):
    kept = {"libsbw.so", "_binding.so"} - {missing}
    copy = tmp_path / PACKAGE
    copy.mkdir()
    for name in ["__init__.py", "_build.py", *kept]:
        if os.path.exists(os.path.join(ROOT, PACKAGE, name)):
            shutil.copy(os.path.join(ROOT, PACKAGE, name), copy)
    r = subprocess.run([sys.executable, "-c", f"import {PACKAGE}"], cwd=tmp_path, capture_output=True,
                       text=True, timeout=300)
    last = r.stderr.strip().splitlines()[-1]
    assert r.returncode != 0 and last.startswith("ImportError") and missing in last
    # the file that the message names can be run while the package cannot be imported
    named = last.split("python ")[-1].strip()
    assert "__graft_entry__.build()" in last and os.path.samefile(named, copy / "_build.py")
    probe = ("import importlib.util as u; s = u.spec_from_file_location('b', %r); "
             "m = u.module_from_spec(s); s.loader.exec_module(m); print(m.LIBRARY)" % named)
    r = subprocess.run([sys.executable, "-c", probe], cwd=tmp_path, capture_output=True, text=True, timeout=60)
    assert r.stdout.strip() == str(copy / "libsbw.so")
