"""The rule that gives a 16-row tile of a 2D layer solve one or more wavefronts
counts the problems of its own launch (CPU, host-only plans): m for the M
problems, 2 m - 2 for the R and L problems, two for those of a sequential
sweep; problems of 64 rows take one in FP32.  tests/solve_rules.cpp asks the built library."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1504_04058_amd")
FP64, FP32, SPLIT = 0, 1, 2


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(PKG, "libasp.so")):
        from paper_1504_04058_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("rules") / "solve_rules")
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", os.path.join(HERE, "solve_rules.cpp"), "-o", exe,
           "-I" + os.path.join(PKG, "csrc"), "-I" + os.path.join(os.path.dirname(PKG), "include"),
           "-L" + PKG, "-lasp", "-Wl,-rpath," + PKG]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]

    def ask(n, b, gamma, prec, seq=0):
        out = subprocess.run([exe, *map(str, (n, b, gamma, prec, seq))], capture_output=True, text=True)
        assert out.returncode == 0, out.stderr
        return tuple(map(int, out.stdout.split()))
    return ask


# M and R/L problems: 512 tiles (problems x 2 halves x rows / 16) is the line in FP32
@pytest.mark.parametrize("n,b,gamma,prec,seq,m,rl", [
    (1023, 4, 12, FP32, 0, 1, 1),      # 251 layers: 1004 and 1000 tiles
    (511, 4, 12, FP32, 0, 4, 4),       # 123 layers: 492 and 488
    (640, 4, 12, FP32, 0, 1, 1),       # 155 layers: 620 and 616
    (134, 1, 4, FP32, 0, 4, 4),        # 128 layers: 256 and 508 (16 rows both)
    (136, 1, 4, FP32, 0, 4, 1),        # 130 layers: 260 and 516
    (262, 1, 4, FP32, 0, 4, 1),        # 256 layers: 512
    (263, 1, 4, FP32, 0, 1, 1),        # 257 layers: 514
    (300, 1, 12, FP32, 1, 1, 4),       # sequential, 278 layers: two R/L problems at a time
    (150, 4, 12, FP32, 1, 4, 4),
    (1023, 4, 12, FP64, 0, 4, 4),
    (180, 4, 20, FP32, 0, 1, 4),       # M problems of 64 rows: one in FP32,
    (180, 4, 20, FP64, 0, 2, 4),       # two in FP64
    (120, 10, 24, FP32, 0, 1, 1),      # R and L problems of 64 rows too
    (1023, 4, 12, SPLIT, 0, 1, 1),
])
def test_wavefronts_of_layer_solves(rules, n, b, gamma, prec, seq, m, rl):
    assert rules(n, b, gamma, prec, seq)[:2] == (m, rl)


# map chains (4 x (2 m - 4) problems x chunks of 16 columns of a half x (rows / 16)^2): two
# wavefronts up to 8192 products of 16 x 16 tiles in FP32, 4096 in FP64; one for 64 rows
@pytest.mark.parametrize("n,b,gamma,prec,maps", [
    (255, 4, 12, FP64, 2),      # 59 layers: 3648
    (300, 4, 12, FP64, 1),      # 70 layers: 5440
    (300, 4, 12, FP32, 2),
    (511, 8, 9, FP32, 2),       # 62 layers: 7680
    (383, 4, 12, FP32, 1),      # 91 layers: 8544
    (1023, 4, 12, FP64, 1),
    (200, 8, 20, FP32, 2),      # 32 rows
    (300, 3, 17, FP32, 1),
    (120, 10, 24, FP32, 1),     # 64 rows
    (150, 24, 13, FP64, 1),
    (383, 4, 12, SPLIT, 1),
])
def test_wavefronts_of_map_chains(rules, n, b, gamma, prec, maps):
    assert rules(n, b, gamma, prec)[2] == maps
