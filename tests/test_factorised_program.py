"""The factorised contraction program (tensors contracted two at a time and
shared between graphs, in four and in eight clusters) computes the V, B_alpha
and dV/dM of the expanded program (sums of monomials): both compiled for the
host and compared on random moments.  Sums of at most a few thousand products
of order-one numbers in double precision: 1e-12 of the largest entry."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2304_13144_amd", "csrc")


@pytest.fixture(scope="module")
def gen(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = tmp_path_factory.mktemp("gen") / "gen_contract"
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", str(exe), os.path.join(CSRC, "gen_contract.cpp"),
                    os.path.join(CSRC, "basis.cpp")], check=True)
    return str(exe)


@pytest.mark.parametrize("level", [2, 4, 6, 8, 12, 16, 20])
def test_factorised_program_equals_expanded_program(gen, level, tmp_path):
    for form in ("single", "factorised"):
        (tmp_path / form).mkdir()
        subprocess.run([gen, str(tmp_path / form), f"--{form}", str(level)], check=True, capture_output=True)
    exe = tmp_path / "check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", f"-DLV={level}",
                    f'-DLEVEL_A="{tmp_path}/single/mtp_level{level}.inc"',
                    f'-DLEVEL_B="{tmp_path}/factorised/mtp_level{level}.inc"',
                    os.path.join(HERE, "factorised_check.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    print(r.stdout.strip())
    assert r.returncode == 0, r.stdout
