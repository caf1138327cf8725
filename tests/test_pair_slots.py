"""The slots of the sparse matrix product in the dense backward, enumerated on the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_selected_pair_is_summed_once_and_slots_ascend(tmp_path):
    exe = str(tmp_path / "pair_slots")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_2502_07590_amd", "csrc"), os.path.join(ROOT, "tests", "sanitize", "pair_slots_main.cpp"),
                    "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and "pair slots ok" in out.stdout, out.stderr
