"""The library's threaded host loops (sem_threads.h), built with a host compiler:
under sanitizers, and without them where the address space is closed to new
threads."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2207_07098_amd", "csrc")
MAIN = os.path.join(ROOT, "tests", "native", "threads_main.cpp")

if shutil.which("g++") is None:
    pytest.skip("no host compiler", allow_module_level=True)


@pytest.mark.parametrize("flags, args", [
    (["-fsanitize=address,undefined", "-fno-sanitize-recover=all"], []),
    (["-fsanitize=thread"], []), ([], ["closed"])])
def test_host_ranges(tmp_path, flags, args):
    exe = str(tmp_path / "threads")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", *flags, "-I" + CSRC, MAIN, "-o", exe,
                           "-pthread"])
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr)


def test_threads_start_in_one_place():
    """A thread started elsewhere would end the process with what it throws."""
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".cpp", ".h")) and name != "sem_threads.h":
            with open(os.path.join(CSRC, name)) as f:
                code = re.sub(r"//[^\n]*", "", f.read())
            assert "std::thread" not in code, name
