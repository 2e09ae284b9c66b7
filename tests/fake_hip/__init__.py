"""The library's host code on a stand-in HIP runtime: what it launches, and what it does when the runtime reports an error.

``run(script)`` runs a Python script in a process of its own with the stand-in preloaded; the script finds ``B`` (the binding),
``F`` (the stand-in), ``ctx``, ``np`` and the helpers of ``script_prelude.py``."""
import os
import shutil
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))


def build(out_dir) -> str:
    path = os.path.join(str(out_dir), "libfake_hip.so")
    cxx = shutil.which("g++") or shutil.which("clang++")
    subprocess.run([cxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", path], check=True)
    return path


def run(lib_path: str, script: str, timeout: float = 60.0) -> str:
    """Output of the script; an AssertionError with everything it printed if it fails or does not end."""
    prelude = open(os.path.join(HERE, "script_prelude.py")).read()
    preload = ":".join(v for v in (lib_path, os.environ.get("LD_PRELOAD")) if v)
    env = dict(os.environ, LD_PRELOAD=preload, FAKE_HIP=lib_path, PYTHONPATH=ROOT)
    try:
        p = subprocess.run([sys.executable, "-c", prelude + textwrap.dedent(script)], env=env, cwd=ROOT, text=True,
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=timeout)
    except subprocess.TimeoutExpired as e:
        raise AssertionError(f"did not end within {timeout} s: {e.stdout!r}") from None
    assert p.returncode == 0, p.stdout[-4000:]
    return p.stdout
