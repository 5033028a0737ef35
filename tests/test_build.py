"""What a build leaves behind, without compiling the kernels: the C compiler is given in any number of words, and the library and the
module of its calls are replaced together or not at all; without Python's headers there is no such module.  No GPU needed."""
import subprocess

import pytest

from paper_2605_22428_amd import build


@pytest.fixture
def tree(tmp_path, monkeypatch):
    """Built files of an earlier build, and a library that compiles at once."""
    def library(cmd, **kw):
        if cmd[0] != "hipcc-of-the-test":
            return run(cmd, **kw)
        open(cmd[cmd.index("-o") + 1], "w").write("new library")
        return subprocess.CompletedProcess(cmd, 0, stdout="")

    run = subprocess.run
    monkeypatch.setattr(build.subprocess, "run", library)
    monkeypatch.setenv("HIPCC", "hipcc-of-the-test")
    for name in ("LIB", "CALLS"):
        at = tmp_path / name
        at.write_text("old")
        monkeypatch.setattr(build, name, str(at))
    return tmp_path


@pytest.mark.parametrize("cc", [None, "gcc -m64", "gcc -O1 -DNAME='a b'"])
def test_compiler_of_several_words(tree, monkeypatch, cc):
    monkeypatch.delenv("CC", raising=False) if cc is None else monkeypatch.setenv("CC", cc)
    build.build()
    assert (tree / "LIB").read_text() == "new library" and (tree / "CALLS").read_bytes()[:4] == b"\x7fELF"
    assert sorted(f.name for f in tree.iterdir()) == ["CALLS", "LIB"]


def test_a_failure_leaves_both_files_as_they_were(tree, monkeypatch):
    monkeypatch.setenv("CC", "false")
    with pytest.raises(subprocess.CalledProcessError):
        build.build()
    assert sorted((f.name, f.read_text()) for f in tree.iterdir()) == [("CALLS", "old"), ("LIB", "old")]


def test_without_pythons_headers_there_is_no_module(tree, monkeypatch):
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tree)})
    build.build()
    assert sorted(f.name for f in tree.iterdir()) == ["LIB"]
