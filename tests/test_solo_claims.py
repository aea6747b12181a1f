"""The claim tables of the one-block rounds on the host: whatever the order in which the waves of the
block come by, a round's claims stand until every wave has read them."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_claims_stand_until_every_wave_has_read_them(tmp_path):
    exe = tmp_path / "solo_claims"
    build = subprocess.run(
        ["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Wextra", "-Wno-unknown-pragmas", "-fsanitize=address,undefined",
         "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2509_19086_amd", "csrc"), "-o", str(exe),
         os.path.join(ROOT, "tests", "solo_claims_driver.cpp")], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout + run.stderr[-4000:]
    assert "claims ok" in run.stdout
