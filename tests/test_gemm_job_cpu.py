"""The host rules of the binary64 products (csrc/iso_gemm_job.h, plain C++) in a program of their own: the entries
that a one-triangle job computes, counted tile by tile here, and the forms that the kernels take."""
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


def test_forms_the_kernels_do_not_take(tmp_path):
    run = _program(tmp_path, """int main(int, char** v) {
      GemmJob J{};
      int64_t* f[4] = {&J.as0, &J.as1, &J.bs0, &J.bs1};
      for (int i = 0; i < 4; ++i) *f[i] = atoll(v[1 + i]);
      J.M = atoll(v[5]); J.N = 7; J.K = 9; J.upper = atoi(v[6]);
      GemmJob two[2] = {GemmJob{}, J};                       // a job without outputs is in order
      printf("%d %d\\n", gemm_job_ok(J, atoi(v[7])), gemm_table_ok(two, 2, atoi(v[7])));
    }""")
    for strides, M, upper, one_triangle, ok in [
            ((1, 5, 1, 9), 5, 0, 0, 1), ((9, 1, 7, 1), 5, 0, 0, 1), ((1, 1, 1, 1), 1, 0, 0, 1),
            ((2, 5, 1, 9), 5, 0, 0, 0), ((1, 5, 3, 9), 5, 0, 0, 0), ((2, 5, 1, 9), 0, 0, 0, 1),
            ((1, 5, 1, 9), 5, 0, 1, 0), ((1, 5, 1, 9), 5, 1, 1, 1), ((1, 5, 1, 9), 5, 2, 1, 1), ((1, 5, 1, 9), 5, 2, 0, 1)]:
        assert run(*strides, M, upper, one_triangle) == [str(ok)] * 2, (strides, M, upper, one_triangle)
