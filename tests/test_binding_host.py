"""The binding without its native argument checks: the host-side calls need
neither the module nor a torch with GPU support, and the build goes on without
Python's or torch's headers."""
import os
import subprocess
import sys

import pytest

from paper_2609_38169_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST_CALLS = """
import sys
import numpy as np
import torch
if hasattr(torch._C, "_cuda_getCurrentRawStream"):
    del torch._C._cuda_getCurrentRawStream          # as in a torch without GPU support
sys.modules["paper_2609_38169_amd._stepq_args"] = None
from paper_2609_38169_amd import stepq
S = np.random.default_rng(0).standard_normal((2, 8, 64)).astype(np.float32)
r, c = stepq.stepq_setup_fit(S)
assert r.shape == (2, 8) and c.shape == (2, 64)
assert stepq.stepq_pool_bytes(3, 2, 1, 8, 64, np.full((2, 8), 8, np.uint8))[0] > 0
launches, order = stepq.stepq_pool_plan(3, 2, 1, 8, 64, np.full((2, 8), 8, np.uint8))
assert len(launches) == 1
print("host calls ok")
"""


def test_host_calls_without_the_module_or_a_gpu_torch():
    r = subprocess.run([sys.executable, "-c", HOST_CALLS], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "host calls ok" in r.stdout, r.stderr[-2000:]


def test_module_is_skipped_without_headers(monkeypatch, tmp_path):
    assert B.args_command(str(tmp_path / "m.so"), B.CSRC)[0] == "g++"
    monkeypatch.setattr(B.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert B.args_command(str(tmp_path / "m.so"), B.CSRC) is None


@pytest.mark.parametrize("headers,present,name,built", [
    (True, False, "libstepq.so", True), (True, True, "libstepq.so", True), (False, False, "libstepq.so", False),
    (False, True, "libstepq.so", False), (True, False, "other.so", True), (True, True, "other.so", False),
    (False, False, "other.so", False)])
def test_build_makes_the_module_where_it_can(monkeypatch, tmp_path, headers, present, name, built):
    """The commands of a build, recorded instead of run: the library always,
    the module for the package's own library or where there is none yet."""
    monkeypatch.setattr(B, "LIB", str(tmp_path / "libstepq.so"))
    monkeypatch.setattr(B, "ARGS_MODULE", str(tmp_path / "_stepq_args.so"))
    monkeypatch.setattr(B, "device_targets", lambda path: [B.ARCH])
    if not headers:
        monkeypatch.setattr(B, "args_command", lambda out, csrc: None)
    if present:
        (tmp_path / "_stepq_args.so").write_text("earlier")
    ran = []

    def fake(cmd, **kw):
        ran.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").write("new")
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(B.subprocess, "run", fake)
    out = B.build(out=str(tmp_path / name), build_dir=str(tmp_path / "obj"))
    assert open(out).read() == "new"
    module = tmp_path / "_stepq_args.so"
    assert any(B.ARGS_SOURCE in " ".join(c) for c in ran) == built
    if built:
        assert module.read_text() == "new"
    else:
        # kept where another library is built, dropped with the package's own: it may not fit this torch
        assert module.exists() == (present and name != "libstepq.so")
