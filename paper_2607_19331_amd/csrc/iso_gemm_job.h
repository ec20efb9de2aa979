// Binary64 product jobs: what one is, which forms the kernels take, how its output is cut into tiles.
// Plain C++ (no HIP), so that the CPU tests can compile it.
#pragma once

#include <stdint.h>

namespace iso {

// A batch of independent GEMMs in one launch: grid.z indexes the job; blocks outside a
// job's M x N exit.  C(i,j) = alpha * sum_k A(i,k) B(k,j) + beta * C(i,j) with X(i,k) at
// X[i*xs0 + k*xs1].  `upper`: only the tiles on or above the diagonal are computed, for a
// symmetric product; 1: the caller fills in the lower triangle where it needs one, 2: a tile above
// the diagonal is also stored transposed below it.  `skip`: if set and *skip is nonzero when the
// kernel runs, the job is left out (an iteration whose job has converged).
struct GemmJob {
  const double* A;
  const double* B;
  double* C;
  int64_t as0, as1, bs0, bs1, cs0, cs1;
  int64_t M, N, K;
  double alpha, beta;
  int upper;
  const int* skip;
};

// The forms that the kernels take: each operand has a stride of 1 (they read 16 bytes along it), and in a launch
// whose grid numbers one triangle of tiles (`upper`) every job is `upper`.  They do not check it: a job of
// another form would give wrong numbers.  A job without outputs is left out by them.
inline bool gemm_job_ok(const GemmJob& J, bool upper = false) {
  if (J.M <= 0 || J.N <= 0) return true;
  return (J.as0 == 1 || J.as1 == 1) && (J.bs0 == 1 || J.bs1 == 1) && (!upper || J.upper != 0);
}

// n jobs of a host table.
inline bool gemm_table_ok(const GemmJob* jobs, int64_t n, bool upper = false) {
  for (int64_t j = 0; j < n; ++j)
    if (!gemm_job_ok(jobs[j], upper)) return false;
  return true;
}

// Tiles gemm_tile_of numbers (for `upper` a few of them lie below the diagonal).
constexpr int gemm_tiles(int gx, int gy, bool upper) {
  if (!upper) return gx * gy;
  int n = 0;
  for (int j0 = 0; j0 < gy; j0 += 4) {
    const int wd = (gy - j0 < 4) ? gy - j0 : 4;
    n += ((gx < j0 + wd) ? gx : j0 + wd) * wd;
  }
  return n;
}

// Tile side for n products of M x N outputs: the largest of 128, 64 and 32 that still gives every
// CU a workgroup and computes at most a quarter more padding than the next smaller one.  With fewer
// workgroups than CUs the chip idles and one tile's serial k loop sets the time.
inline int gemm_side(int64_t M, int64_t N, int64_t n) {
  const int64_t cus = 256;
  auto tiles = [&](int64_t side) { return ((M + side - 1) / side) * ((N + side - 1) / side); };
  for (int side = 128; side > 32; side /= 2)
    if (tiles(side) * n >= cus && 16 * tiles(side) <= 5 * tiles(side / 2)) return side;
  return 32;
}

// Entries of an n x n output that an `upper` job computes: those of its tiles on or above the diagonal.
inline int64_t gemm_upper_entries(int64_t n, int side) {
  int64_t e = 0;
  for (int64_t j0 = 0; j0 < n; j0 += side) {
    const int64_t end = (n < j0 + side) ? n : j0 + side;
    e += end * (end - j0);
  }
  return e;
}

}  // namespace iso
