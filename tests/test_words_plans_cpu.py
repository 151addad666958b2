"""Work lists of the digit-word product, swept on the CPU under sanitizers (tests/words_plan_sweep.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_word_product_lists_cover_every_step_once(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path / "words_plan_sweep"
    subprocess.run([gxx, "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_1809_11165_amd", "csrc"), os.path.join(ROOT, "tests", "words_plan_sweep.cpp"),
                    "-o", str(exe)], check=True)
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)
    proc = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=300, env=env)
    assert proc.returncode == 0 and proc.stdout.startswith("OK "), proc.stderr[-2000:]
