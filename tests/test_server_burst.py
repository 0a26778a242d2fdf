"""The request server's choice of a launch's kind for the requests of a burst,
compiled for the CPU against the stub HIP runtime."""
import os

from tests import test_server_host as host


def test_requests_of_a_burst_share_a_kind(tmp_path, monkeypatch):
    monkeypatch.setattr(host, "SRC", os.path.join(host.ROOT, "tests", "cpp", "test_server_burst.cpp"))
    r = host.build_and_run(tmp_path, "server_burst", "g++", ["-Wno-unknown-pragmas", "-Wno-subobject-linkage"])
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
