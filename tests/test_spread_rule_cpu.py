"""The rules that choose the spread passes, on the CPU (a C++ driver under
sanitizers): spare capacity does not count as work, and each boundary lies
where its comment puts it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_spread_rule(tmp_path):
    exe = str(tmp_path / "spread_rule_test")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
                           "-fno-sanitize-recover=all", "-g", "-I", os.path.join(ROOT, "paper_2511_16298_amd", "csrc"),
                           os.path.join(ROOT, "tests", "native", "spread_rule_test.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-4000:]
    assert r.stdout.strip() == "OK"
