"""What calls of the built library launch, told by launch_probe.cpp (no GPU)."""
import functools
import pathlib
import shutil
import subprocess
import tempfile

import pytest

HERE = pathlib.Path(__file__).resolve().parent
ROOT = HERE.parent
LIB = ROOT / "paper_1411_3656_amd" / "libppf.so"
ROCM = "/opt/rocm"


@functools.lru_cache(maxsize=None)
def probe() -> pathlib.Path:
    if not LIB.exists() or not shutil.which("g++"):
        pytest.skip("needs the built library and g++")
    exe = pathlib.Path(tempfile.mkdtemp(prefix="ppf_probe_")) / "launch_probe"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT / 'include'}",
                    str(HERE / "launch_probe.cpp"), str(LIB), "-rdynamic", "-pthread", "-o", str(exe),
                    f"-Wl,-rpath,{LIB.parent}", f"-Wl,-rpath,{ROCM}/lib", f"-Wl,-rpath-link,{ROCM}/lib"],
                   check=True)
    return exe


def run(*commands: str) -> list[list[str]]:
    """One list of words per command (launch_probe.cpp says which there are)."""
    res = subprocess.run([str(probe())], input="\n".join(commands) + "\n", capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stderr
    return [line.split() for line in res.stdout.splitlines()]


def kernel(word: str) -> str:
    return word.split("<")[0]
