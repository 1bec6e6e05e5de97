"""The server scheduler's choice between a request's two workspace sizes (CPU only): the larger
one never keeps another request out of an idle slot (tests/native/srv_room.cpp, built with the
address and undefined-behaviour sanitizers)."""
import os
import subprocess

from tests.test_host_sanitized import ASAN, CSRC, ENV, NATIVE, ROOT, _build, pytestmark  # noqa: F401


def test_larger_workspace_displaces_nothing(tmp_path):
    exe = _build(str(tmp_path / "srv_room"), "g++", [os.path.join(NATIVE, "srv_room.cpp")],
                 ASAN + ["-I", CSRC, "-I", os.path.join(ROOT, "include")])
    r = subprocess.run([exe], capture_output=True, text=True, env=ENV, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    assert "srv_room: all passed" in r.stdout
