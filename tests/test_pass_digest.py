"""The digest that tells whether a stored pass-kernel profile belongs to the
sources: it follows every file the pass kernels are compiled from, as the
compiler lists them, and none of the host's."""
import os
import shutil
import subprocess

import pytest

from paper_2606_31098_amd import build


def test_digest_covers_what_the_compiler_reads():
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("needs a C++ preprocessor")
    read = set()
    for f in os.listdir(build.CSRC):
        if f.startswith("pilot_pass") and f.endswith(".hip"):
            # quoted includes only: -MM leaves out system headers, -MG the missing ones
            out = subprocess.run([cxx, "-x", "c++", "-std=c++17", "-E", "-MM", "-MG", os.path.join(build.CSRC, f)],
                                 capture_output=True, text=True, check=True).stdout
            read |= {os.path.basename(w) for w in out.replace("\\\n", " ").split() if w.startswith(build.CSRC)}
    assert "pilot_step.inc" in read and len(read) > 8
    assert read == set(build.pass_kernel_sources())


def test_digest_changes_with_every_source(tmp_path, monkeypatch):
    csrc = str(tmp_path / "csrc")
    shutil.copytree(build.CSRC, csrc)
    monkeypatch.setattr(build, "CSRC", csrc)
    before = build.pass_kernel_digest()
    for f in build.pass_kernel_sources():
        with open(os.path.join(csrc, f), "a") as fh:
            fh.write("// another line\n")
        after = build.pass_kernel_digest()
        assert after != before, f
        before = after
    with open(os.path.join(csrc, "pilot_runtime.cpp"), "a") as fh:
        fh.write("// another line\n")
    assert build.pass_kernel_digest() == before
