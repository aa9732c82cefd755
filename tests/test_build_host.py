"""CPU test of the build script: flags given to it reach every compilation and the
link, and a source that does not compile stops the build."""
import importlib.util
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _script():
    spec = importlib.util.spec_from_file_location("lbm_build", os.path.join(ROOT, "paper_1611_03329_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("fails", [False, True])
def test_extra_flags_reach_compilation_and_link(monkeypatch, fails):
    build = _script()
    compiled, linked = [], []

    class Job:
        def __init__(self, cmd):
            compiled.append(cmd)
            self.returncode = 1 if fails and len(compiled) == 2 else 0

        def wait(self):
            return self.returncode

    monkeypatch.setattr(subprocess, "Popen", Job)
    monkeypatch.setattr(subprocess, "run", lambda cmd, check: linked.append(cmd))
    monkeypatch.setattr(os, "replace", lambda a, b: None)
    if fails:
        with pytest.raises(subprocess.CalledProcessError):
            build.build(("-lextra",))
        assert not linked
    else:
        build.build(("-lextra",))
        assert len(linked) == 1 and "-lextra" in linked[0]
    assert len(compiled) == len(build.SRCS) and all("-lextra" in cmd for cmd in compiled)
