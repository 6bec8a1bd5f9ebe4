"""The autotune cache's key, on the CPU (a C++ driver under sanitizers): choices
recorded before a candidate's meaning changed are not taken, and what decides
which kernels a configuration runs is part of the key."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tune_key(tmp_path):
    exe = str(tmp_path / "tunekey_test")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
                           "-fno-sanitize-recover=all", "-g", "-I", os.path.join(ROOT, "paper_2511_16298_amd", "csrc"),
                           os.path.join(ROOT, "tests", "native", "tunekey_test.cpp"), "-o", exe])
    r = subprocess.run([exe, str(tmp_path)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-4000:]
    assert r.stdout.strip() == "OK"
