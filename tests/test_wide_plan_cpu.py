"""CPU check of the wide batched plans (csrc/ts_plan.cpp, HIP-free), built
with g++ and the sanitizers on."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_wide_plan_invariants(tmp_path):
    csrc = os.path.join(ROOT, "paper_2406_05955_amd", "csrc")
    exe = str(tmp_path / "wide_plan_check")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, "-o", exe,
                    os.path.join(HERE, "native", "wide_plan_check.cpp"), os.path.join(csrc, "ts_plan.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.stdout, r.stderr)
