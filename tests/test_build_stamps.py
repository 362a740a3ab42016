"""An object is rebuilt when any file its translation unit includes has changed (host only: nothing is compiled)."""
import shutil
import subprocess

import pytest

from paper_2309_07235_amd import build


@pytest.fixture
def tree(tmp_path, monkeypatch):
    """A copy of csrc/ and include/ that may be edited, with the instantiation units generated as a build does."""
    csrc = tmp_path / "pkg" / "csrc"
    shutil.copytree(build.CSRC, csrc)
    shutil.copytree(build.HERE.parent / "include", tmp_path / "include")
    monkeypatch.setattr(build, "CSRC", csrc)
    inst = tmp_path / "pkg" / "_build" / "gemm_inst_f64_16x16_16x16.hip"
    inst.parent.mkdir()
    text = (csrc / "gemm_inst.hip.in").read_text()
    for key, val in (("@T@", "double"), ("@TM@", "16"), ("@TN@", "16"), ("@WM@", "16"), ("@WN@", "16")):
        text = text.replace(key, val)
    inst.write_text(text)
    return tmp_path, sorted(csrc.glob("*.hip")) + [inst]


def test_every_included_file_is_in_the_stamp(tree):
    """The compiler's own list of what a unit includes, against the files whose edit changes its stamp."""
    root, units = tree
    for unit in units:
        make = subprocess.run([build.HIPCC, *build.FLAGS, "-I", str(build.CSRC), "-MM", "--cuda-host-only", str(unit)],
                              capture_output=True, text=True, check=True).stdout
        included = [w for w in make.replace("\\\n", " ").split() if w.startswith(str(root))]
        assert len(included) > 1, make
        before = build._stamp(unit)
        assert build._stamp(unit) == before
        for path in sorted({build.Path(w).resolve() for w in included}):
            text = path.read_text()
            path.write_text(text + "\n// edited\n")
            assert build._stamp(unit) != before, f"{unit.name} is not rebuilt after an edit of {path.name}"
            path.write_text(text)
        assert build._stamp(unit) == before


def test_an_include_that_is_not_there_is_an_error(tree):
    _, units = tree
    units[0].write_text('#include "no_such_header.hpp"\n')
    with pytest.raises(RuntimeError, match="no_such_header"):
        build._stamp(units[0])
