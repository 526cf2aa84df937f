"""What a compile leaves in the tree: objects and the temporary files of an
interrupted compiler stay out of the package folder's tracked names."""
import os
import stat
import subprocess

import pytest

from paper_2304_07006_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# stands for the compiler: writes its temporary file beside the output as clang does, then fails
FAKE = """#!/bin/sh
while [ $# -gt 0 ]; do
  if [ "$1" = -o ]; then out=$2; fi
  shift
done
: > "${out%.o}-0123abcd.o.tmp"
exit 1
"""


def test_a_failed_compile_leaves_nothing_beside_the_library(tmp_path, monkeypatch):
    cc = tmp_path / "cc"
    cc.write_text(FAKE)
    cc.chmod(cc.stat().st_mode | stat.S_IXUSR)
    out = tmp_path / "pkg"
    out.mkdir()
    monkeypatch.setattr(build, "HIPCC", str(cc))
    with pytest.raises(RuntimeError):
        build.build(out=str(out / "libxtc.so"))
    assert os.listdir(out) == ["_build"]


def test_build_artefacts_are_not_tracked():
    if not os.path.isdir(os.path.join(ROOT, ".git")):
        pytest.skip("not a git checkout")
    names = subprocess.run(["git", "ls-files"], cwd=ROOT, capture_output=True, text=True, check=True).stdout.split()
    bad = [n for n in names if n.endswith((".o", ".so", ".tmp")) or "_build/" in n]
    assert not bad, bad
