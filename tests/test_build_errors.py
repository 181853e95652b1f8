"""What the build reports when a compiler run fails (the compiler is replaced by a stand-in)."""
import subprocess

import pytest

from paper_2505_16162_amd import build


@pytest.fixture
def compiler(tmp_path, monkeypatch):
    """run(fails): a compiler that writes its output file, or fails with a message if fails(command)."""
    lib = tmp_path / "lib.so"
    monkeypatch.setattr(build, "LIB", str(lib))

    def use(fails):
        def run(cmd, **kw):
            if fails(cmd):
                return subprocess.CompletedProcess(cmd, 1, "", "kernel.hip:7:3: error: no such thing")
            open(cmd[cmd.index("-o") + 1], "w").write("")
            return subprocess.CompletedProcess(cmd, 0, "", "")
        monkeypatch.setattr(build.subprocess, "run", run)
        return lib
    return use


@pytest.mark.parametrize("to_assembly", [False, True])
def test_the_compilers_message_is_reported(compiler, to_assembly):
    lib = compiler(lambda cmd: ("-S" in cmd) == to_assembly)
    with pytest.raises(RuntimeError, match="kernel.hip:7:3: error: no such thing"):
        build.build_library()
    assert not lib.exists()


def test_an_assembly_text_without_the_kernels_is_refused(compiler):
    lib = compiler(lambda cmd: False)
    with pytest.raises(RuntimeError, match="kernels not found in the assembly text"):
        build.build_library()
    assert not lib.exists()
