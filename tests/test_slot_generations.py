"""Exchange slots' 16-bit generations over more than 65536 exchanges: no used unit
may carry an exchange's generation before the exchange has written it (a model of
the slots with the engine's own rule of when a slot is written whole)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_no_unit_passes_for_a_later_exchange(tmp_path):
    exe = str(tmp_path / "slot_generations")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_1709_06816_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "native", "slot_generations.cpp")], check=True)
    res = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout
