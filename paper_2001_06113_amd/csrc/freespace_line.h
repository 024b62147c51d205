// Small parts of the free-space line transforms, shared by the line kernels
// (freespace_kernels.hip) and the one-workgroup 1D run (freespace_run1d.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "fft_lds.h"
#include "tdse_internal.h"

namespace tdse {

__device__ __forceinline__ double2 fs_mul_mi(double c, double2 z) { return double2{c * z.y, -c * z.x}; }

// Grid points a thread can hold, of its EPT FFT slots: one when M <= nu/EPT
// (the short ends of fft_lds.h: the first pass going in and most of the last
// pass coming out drop out), two when M <= 2 nu/EPT, half when M <= nu/2 (the
// other slots are compile-time zeros going in and unused coming out), else all.
// Two of eight: a 3D row pass of 38 points at nu = 256 took 563 us with half the
// slots, whose dense sums mostly worked on empty ones, and takes 512 us.
__host__ __device__ constexpr int fs_points(int nu, int M, int ept) {
  return M <= nu / ept ? 1 : M <= 2 * nu / ept ? 2 : M <= nu / 2 ? ept / 2 : ept;
}

// sum_{j0 <= j < j1} r^(j - j0) f[j] (f in LDS): four interleaved Horner sums
// in r^4, since one is a chain of dependent products (100 points of a row on
// one thread: 4.6 us of a 20 us pass).
__device__ __forceinline__ double2 geometric_sum(const double2* f, int j0, int j1, double2 r) {
  const double2 r2 = cmul(r, r), r4 = cmul(r2, r2);
  double2 s[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) s[k] = double2{0.0, 0.0};
  for (int j = j0 + ((j1 - j0 + 3) / 4 - 1) * 4; j >= j0; j -= 4) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double2 x = f[min(j + k, j1 - 1)];
      s[k] = cadd(cmul(s[k], r4), j + k < j1 ? x : double2{0.0, 0.0});
    }
  }
  return cadd(cadd(s[0], cmul(r, s[1])), cmul(r2, cadd(s[2], cmul(r, s[3]))));
}

__device__ __forceinline__ double2 conj_if(bool c, double2 z) { return c ? double2{z.x, -z.y} : z; }

}  // namespace tdse
