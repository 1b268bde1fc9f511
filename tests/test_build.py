"""The library builds and works on machines that cannot build the extension module beside it."""
import os
import subprocess
import sys

import pytest

from paper_2305_13525_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def no_library(monkeypatch, tmp_path):
    """build() with a stand-in for the HIP compiler that does nothing, and the module's file in a folder of its own."""
    monkeypatch.setattr(build, "HIPCC", "true")
    monkeypatch.setattr(build, "CALLS", str(tmp_path / os.path.basename(build.CALLS)))
    return tmp_path


@pytest.mark.parametrize("missing", ["compiler", "headers"])
def test_builds_without(no_library, monkeypatch, missing):
    if missing == "compiler":
        monkeypatch.setenv("CC", str(no_library / "no-such-compiler"))
    else:
        monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(no_library)})
    with open(build.CALLS, "w") as f:
        f.write("of an older build")
    with pytest.warns(UserWarning, match="_calls was not built"):
        assert build.build() == build.LIB
    assert os.listdir(no_library) == []


def test_module_is_named_for_its_interpreter(no_library):
    """No file that another interpreter would load is left, nor one of an older build."""
    (no_library / "_calls.so").write_text("of an older build")
    if not build.build_calls():
        pytest.skip("no C compiler or headers")
    tag = build.sysconfig.get_config_var("EXT_SUFFIX")
    assert os.listdir(no_library) == ["_calls" + tag] and tag != ".so"


def test_the_library_itself_has_to_build(no_library, monkeypatch):
    monkeypatch.setattr(build, "HIPCC", "false")
    with pytest.raises(RuntimeError):
        build.build()


def test_works_without_the_module():
    code = """
import sys
sys.modules["paper_2305_13525_amd._calls"] = None
import paper_2305_13525_amd as axo
from paper_2305_13525_amd import binding
p = axo.Problem.make((1, 1, 1), (0, 0, 0), 0, 32, 48)
for name in binding._QUICK:
    assert getattr(axo, name) is binding._WRAPPERS[name], name
assert axo.axo_fc_fwd(p, 1 << 32, 32, 2 << 32, 48, None, 0, 3 << 32, 48) == 0
"""
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True, timeout=120)
