"""The rules that choose a GEMM's tile (csrc/gemm_plan.h), built for the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("plan") / "dump")
    subprocess.run([cxx, "-std=c++17", "-O2", os.path.join(ROOT, "tests", "host", "gemm_plan_dump.cpp"), "-o", exe], check=True)

    def run(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", stdout=subprocess.PIPE, text=True, check=True, timeout=60).stdout
        return out.split()
    return run


def test_expert_matrices_beyond_32_bit_offsets_stay_on_the_large_tile(rules):
    """The small tiles reach an expert's up rows through byte offsets of up to (ffn + 64) x hidden x 2, where 2^31 means
    "outside": from there on only the 256-row tile, with a base for gate and one for up, may be chosen."""
    sizes = [(768, 2048), (14336, 4096), (16384, 32768), (32512, 32768), (32576, 32768), (65536, 16384), (1 << 18, 8192)]
    asked = [(rows, f, d) for f, d in sizes for rows in (1, 18, 40, 90, 500)]
    for (rows, f, d), tile in zip(asked, rules([f"moe {r} {f} {d}" for r, f, d in asked])):
        fits = (f + 64) * d * 2 < 1 << 31
        assert int(tile) in (32, 64, 128, 256) and (fits or int(tile) == 256), (rows, f, d, tile)
    assert rules(["moe 18 768 2048", "moe 40 14336 4096", "moe 500 768 2048"]) == ["32", "64", "256"]
