"""The host side's build beside the C-ABI library's (host only; the compiler is not run)."""
import types

import pytest

from paper_2204_07143_amd import build


@pytest.fixture
def compiler(monkeypatch, tmp_path):
    """Records the compiler's calls; the built file and the record of what it was built against go to a folder of the test's own."""
    calls, lib = [], tmp_path / "na2d_torch.so"

    def run(cmd, **_):
        calls.append(cmd)
        lib.touch()
        return types.SimpleNamespace(returncode=0, stdout="", stderr="")
    monkeypatch.setattr(build, "HOST_LIB", str(lib))
    monkeypatch.setattr(build, "HOST_STAMP", str(tmp_path / "against"))
    monkeypatch.setattr(build, "subprocess", types.SimpleNamespace(run=run))
    return calls


@pytest.mark.parametrize("missing", ["torch", "compiler"])
def test_the_c_library_does_not_need_torch(monkeypatch, capfd, compiler, missing):
    if missing == "torch":
        monkeypatch.setattr(build.importlib.util, "find_spec", lambda name: None)
    else:
        monkeypatch.setenv("CXX", "no-such-compiler")
    build._build_host(force=True)
    assert not compiler and "not built" in capfd.readouterr().err


def test_rebuilt_against_another_torch(monkeypatch, compiler):
    for expected in 1, 1:   # built once
        build._build_host(force=False)
        assert len(compiler) == expected
    monkeypatch.setattr(build.importlib.metadata, "version", lambda name: "0.1")
    build._build_host(force=False)
    assert len(compiler) == 2
    build._build_host(force=False)
    assert len(compiler) == 2
