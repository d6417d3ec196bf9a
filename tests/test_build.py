"""What the build and the loading of the library need, on the CPU: the C library neither torch nor a host compiler, the
headers' place whatever HIPCC is called."""
import os
import subprocess
import sys

import pytest

from paper_2505_14969_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="no hipcc")
@pytest.mark.parametrize("hipcc", [None, "hipcc", "/opt/rocm/bin/hipcc", "/nowhere/bin/hipcc"])
def test_hip_headers_are_found(hipcc, monkeypatch):
    monkeypatch.delenv("ROCM_PATH", raising=False)
    monkeypatch.delenv("HIPCC", raising=False)
    if hipcc:
        monkeypatch.setenv("HIPCC", hipcc)
        monkeypatch.setenv("PATH", "/opt/rocm/bin" + os.pathsep + os.environ["PATH"])
    line = build.host_command()
    places = [line[i + 1] for i, a in enumerate(line) if a == "-isystem"]
    assert any(os.path.isabs(d) and os.path.exists(os.path.join(d, "hip", "hip_runtime.h")) for d in places), places


def test_host_compiler_with_arguments(monkeypatch):
    monkeypatch.setenv("CXX", "ccache g++")
    assert build.host_command()[:2] == ["ccache", "g++"]


@pytest.mark.parametrize("how", ["compile", "torch"])
def test_library_is_built_where_the_native_half_is_not(how, tmp_path, monkeypatch):
    """A failure of the host compile, or no torch to compile against, is raised behind the library's build."""
    def run(cmd, verbose):
        if cmd[0] == "host":
            raise RuntimeError("host failed")
        open(cmd[cmd.index("-o") + 1], "w").close()

    def command():
        if how == "torch":
            raise ImportError("no torch")
        return ["host"]
    monkeypatch.setattr(build, "_run", run)
    monkeypatch.setattr(build, "host_command", command)
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libstree.so"))
    monkeypatch.setattr(build, "HOST", str(tmp_path / "_host.so"))
    with pytest.raises((RuntimeError, ImportError), match="host failed|no torch"):
        build.build()
    assert (tmp_path / "libstree.so").exists() and not (tmp_path / "_host.so").exists()


def test_library_loads_without_the_native_half():
    code = ("import sys; sys.modules['paper_2505_14969_amd._host'] = None\n"
            "from paper_2505_14969_amd import binding as st\n"
            "assert st.load().stree_version() >= 1\n"
            "assert st.stree_workspace_bytes(st.make_dims(1, 64, 8, 64, 128, 1)) == 0\n"
            "try: st.stree_gate_norm(None, None, None, 1)\n"
            "except ImportError as e: assert 'build.py' in str(e)\n"
            "else: raise SystemExit('no error')\n")
    run = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
