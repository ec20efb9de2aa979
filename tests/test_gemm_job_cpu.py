"""The host rules of the binary64 products (csrc/iso_gemm_job.h, plain C++) in a program of their own: the entries
that a one-triangle job computes, counted tile by tile here."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_19331_amd", "csrc")


def _program(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include "iso_gemm_job.h"\n#include <cstdio>\n#include <cstdlib>\nusing namespace iso;\n' + body)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    return lambda *args: subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True).stdout.split()


def test_entries_of_one_triangle(tmp_path):
    run = _program(tmp_path, "int main(int, char** v) { printf(\"%lld\\n\", (long long)gemm_upper_entries(atoll(v[1]), "
                             "atoi(v[2]))); }")
    for side in (32, 64, 128):
        for n in (1, 31, 32, 33, 127, 128, 129, 1000, 2048):
            want = sum((min(n, i + side) - i) * (min(n, j + side) - j) for i in range(0, n, side) for j in range(i, n, side))
            assert int(run(n, side)[0]) == want, (n, side)
            assert want == n * n or n > side
