"""Host check of the tile that the projection on a prepared layer takes (csrc/kv_gemm_forms.h), compiled for the CPU: the
sizes on which tests/test_gpu_gemm_tiles.py compares every tile with the 256 x 256 kernel do take every one."""
import os
import subprocess

import test_gpu_gemm_tiles as tiles

HERE = os.path.dirname(os.path.abspath(__file__))


def test_the_compared_sizes_take_every_tile(tmp_path):
    exe = str(tmp_path / "gemm_forms_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", os.path.join(HERE, "host", "gemm_forms_check.cpp"), "-o", exe])

    def picks(cases):
        args = [str(v) for M, d in cases for v in (M, d)]
        lines = subprocess.check_output([exe, "256"] + args, text=True).split("\n")
        return int(lines[0]), [tuple(int(v) for v in line.split()) for line in lines[1:len(cases) + 1]]

    count, taken = picks([(B * L, H * dh) for H, dh, B, L in tiles.SIZES])
    assert len(set(taken)) == count == 11, sorted(set(taken))
    # one row and the largest problems: the ends of the range
    assert picks([(1, 128), (64 * 4096, 9216), (64 * 4096, 4096)])[1] == [(32, 32), (256, 256), (256, 256)]
