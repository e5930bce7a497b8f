"""Compiles probe.cpp against the built librc.so and runs commands through it (CPU only)."""
import functools
import os
import subprocess
import tempfile

from paper_1505_05655_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@functools.lru_cache(maxsize=None)
def _binary():
    out = os.path.join(tempfile.mkdtemp(prefix="rc_probe_"), "probe")
    libdir = os.path.dirname(build.LIB)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
           "-I", build.INCLUDE, "-I", build.CSRC, os.path.join(HERE, "probe.cpp"), build.LIB,
           f"-Wl,-rpath,{libdir}", f"-L{rocm}/lib", f"-Wl,-rpath,{rocm}/lib", "-lamdhip64", "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return out


def ask(commands, timeout=60, plan_cache=None):
    """The output line of each command; plan_cache: the plan cache file (none if not given)."""
    env = dict(os.environ, RC_TUNE_CACHE=str(plan_cache or "/nonexistent"))
    res = subprocess.run([_binary()], input="\n".join(commands) + "\n", capture_output=True,
                         text=True, timeout=timeout, env=env)
    assert res.returncode == 0, f"probe ended with {res.returncode}: {res.stderr}"
    lines = res.stdout.splitlines()
    assert len(lines) == len(commands)
    return lines
