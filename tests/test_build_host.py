"""The library is built again when a header has changed, not only a source.  CPU only, with a stand-in for the compiler."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("changed", (None, "paper_2506_01352_amd/csrc/tahq_select.hpp", "paper_2506_01352_amd/csrc/tahq.hip", "include/tahq.h"))
def test_a_changed_header_makes_the_library_old(tmp_path, changed):
    for folder in ("paper_2506_01352_amd/csrc", "include"):
        shutil.copytree(os.path.join(ROOT, folder), tmp_path / folder)
    shutil.copy(os.path.join(ROOT, "paper_2506_01352_amd", "build.py"), tmp_path / "paper_2506_01352_amd")
    compiler = tmp_path / "compiler"
    compiler.write_text('#!/bin/sh\nwhile [ "$1" != "-o" ]; do shift; done\necho built > "$2"\n')
    compiler.chmod(0o755)
    for path in tmp_path.rglob("*"):
        os.utime(path, (1000, 1000))
    library = tmp_path / "paper_2506_01352_amd" / "libtahq.so"
    library.write_text("old")
    os.utime(library, (2000, 2000))
    if changed:
        os.utime(tmp_path / changed, (3000, 3000))
    subprocess.run([sys.executable, "-c", "import build; build.build(force=False)"], check=True, cwd=tmp_path / "paper_2506_01352_amd",
                   env=dict(os.environ, HIPCC=str(compiler)))
    assert library.read_text().strip() == ("built" if changed else "old")
