"""The C ABI library is built and used without torch's headers; the binding works without its native part."""
import importlib.util
import os
import shutil
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2006_16236_amd")


def load_build(tmp_path):
    """build.py by path, with its outputs under tmp_path"""
    spec = importlib.util.spec_from_file_location("la_build_under_test", os.path.join(PACKAGE, "build.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    m.LIB, m.CALL, m.OBJ = (str(tmp_path / n) for n in ("libla_hip.so", "_call.so", "obj"))
    return m


def test_the_library_is_built_without_torch(tmp_path, monkeypatch):
    build = load_build(tmp_path)
    commands = []

    def run(command, **kw):
        commands.append(command)
        open(command[command.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(command, 0)

    monkeypatch.setattr(build.subprocess, "run", run)
    monkeypatch.setitem(sys.modules, "torch", None)             # import torch: ImportError
    open(build.CALL, "w").close()                               # one of older sources
    assert build.build_library(force=True) == build.LIB
    assert os.path.exists(build.LIB) and not os.path.exists(build.CALL)
    assert len(commands) == len(build.sources()) + 1 and not any(c[0] == "g++" for c in commands)
    assert build.is_current()


def test_a_compiler_error_in_the_native_part_is_reported(tmp_path, monkeypatch):
    build = load_build(tmp_path)

    def run(command, **kw):
        if command[0] == "g++":
            raise subprocess.CalledProcessError(1, command, output=b"error")
        open(command[command.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(command, 0)

    monkeypatch.setattr(build.subprocess, "run", run)
    if build._call_command() is None:
        return
    try:
        build.build_library(force=True)
    except Exception:
        return
    raise AssertionError("the error was swallowed")


def test_the_binding_works_without_its_native_part(tmp_path):
    package = tmp_path / "paper_2006_16236_amd"
    package.mkdir()
    for name in os.listdir(PACKAGE):
        if name.endswith(".py"):
            shutil.copy(os.path.join(PACKAGE, name), package)
    os.symlink(os.path.join(PACKAGE, "libla_hip.so"), package / "libla_hip.so")
    code = """
import torch, paper_2006_16236_amd as la
assert la.la_causal_fwd_workspace(2, 8, 65536, 64, 64) > 0
t = torch.zeros(1, 1, 16, 32)
for call in (lambda: la.la_causal_fwd(t, t, t, t), lambda: la.la_recurrent_step(t[0], t[0], t[0], t, t[0], t[0])):
    try:
        call()
    except (ValueError, la.LaError):
        continue
    raise SystemExit("a host tensor was taken")
"""
    subprocess.run([sys.executable, "-c", code], cwd=tmp_path, check=True, timeout=120)
