"""How the compiled files are named and get into place."""
import os
import subprocess
import sysconfig

import pytest

from paper_2605_10670_amd import build


def test_module_carries_the_interpreter_s_tag():
    assert build.MARSHAL.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and os.path.exists(build.MARSHAL)


@pytest.mark.parametrize("fails", [False, True])
def test_outputs_move_into_place_whole(tmp_path, monkeypatch, fails):
    """No moment at which the module's own name holds half a file, and nothing left behind."""
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "module.so"))
    (tmp_path / "module.so").write_bytes(b"old")

    def compiler(cmd, check):
        out = cmd[cmd.index("-o") + 1]
        assert out != build.MARSHAL and os.path.dirname(out) == str(tmp_path)
        with open(out, "wb") as f:
            f.write(b"ne")
            f.flush()
            assert (tmp_path / "module.so").read_bytes() == b"old"
            f.write(b"w")
        if fails:
            raise subprocess.CalledProcessError(1, cmd)
    monkeypatch.setattr(build.subprocess, "run", compiler)
    if fails:
        with pytest.raises(subprocess.CalledProcessError):
            build.build_marshal()
    else:
        build.build_marshal()
    assert (tmp_path / "module.so").read_bytes() == (b"old" if fails else b"new")
    assert os.listdir(tmp_path) == ["module.so"]
