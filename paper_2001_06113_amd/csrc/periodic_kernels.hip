// HIP kernels of the periodic marching scheme, gfx950: the per-instance
// column and row passes (bodies in periodic_body.h), the middle-axis FFT
// passes of 3D grids, their dispatch over line lengths, and the
// complex128 -> complex64 narrowing.
#include <hip/hip_ext.h>

#include "periodic_body.h"

namespace tdse {

// ------------------------------------------------------------- column pass

template <typename C, int N, int LPW, int TL>
__global__ __launch_bounds__(LPW * TL, (sizeof(C) == sizeof(double2) && N >= 256 && N <= 1024 && (N & (N - 1)) == 0) ? 4 : 1) void k_col(LineArgs a) {
  __shared__ C lds[col_lds<C, N, LPW>::elems];
  // tiles sharing a 128-byte line of the potential share an XCD
  const int tile = xcd_tile<(16 / LPW > 1 ? 16 / LPW : 1)>(blockIdx.x, gridDim.x);
  col_body<C, N, LPW, TL>(a, tile * LPW, blockIdx.x, gridDim.x, lds);
}

// FFT-only pass over the middle axis of a 3D grid, in the transform precision
template <typename C, int N, int LPW, int TL, bool INV>
__global__ __launch_bounds__(LPW * TL) void k_mid(LineArgs a) {
  __shared__ C lds[col_lds<C, N, LPW>::elems];
  const int tile = xcd_tile<(16 / LPW > 1 ? 16 / LPW : 1)>(blockIdx.x, gridDim.x);
  mid_body<C, N, LPW, TL, INV>(a, tile * LPW, lds);
}

// ---------------------------------------------------------------- row pass

template <typename C, int N, int LPW, int TL, bool PW = false>
__global__ __launch_bounds__(LPW * TL) void k_row(LineArgs a) {
  __shared__ C lds[row_lds<C, N, LPW>::elems];
  row_body<C, N, LPW, TL, PW>(a, blockIdx.x * LPW, lds);
}

// ------------------------------------------------------ FP64, lengths 3 * 2^a

template <int N, int LPW>
__global__ __launch_bounds__(LPW * tri_tl(N)) void k_tri_col(LineArgs a) {
  __shared__ double2 lds[tri_lds<N, LPW>::elems];
  const int tile = xcd_tile<(16 / LPW > 1 ? 16 / LPW : 1)>(blockIdx.x, gridDim.x);
  tri_col_body<N, LPW>(a, tile * LPW, blockIdx.x, gridDim.x, lds);
}
template <int N, int LPW, bool INV>
__global__ __launch_bounds__(LPW * tri_tl(N)) void k_tri_mid(LineArgs a) {
  __shared__ double2 lds[tri_lds<N, LPW>::elems];
  const int tile = xcd_tile<(16 / LPW > 1 ? 16 / LPW : 1)>(blockIdx.x, gridDim.x);
  tri_mid_body<N, LPW, INV>(a, tile * LPW, lds);
}
template <int N, int LPW, bool PW>
__global__ __launch_bounds__(LPW * tri_tl(N)) void k_tri_row(LineArgs a) {
  __shared__ double2 lds[tri_lds<N, LPW>::elems];
  tri_row_body<N, LPW, PW>(a, blockIdx.x * LPW, lds);
}

// One pass of several Richardson levels of a start-up step, level blockIdx.y's
// arguments in la.a[blockIdx.y] (FP64; the same bodies and schedules).
template <int N, int LPW, int TL>
__global__ __launch_bounds__(LPW * TL, (N >= 256 && N <= 1024 && (N & (N - 1)) == 0) ? 4 : 1) void k_col_lv(LevelArgs la) {
  __shared__ double2 lds[col_lds<double2, N, LPW>::elems];
  const int tile = xcd_tile<(16 / LPW > 1 ? 16 / LPW : 1)>(blockIdx.x, gridDim.x);
  col_body<double2, N, LPW, TL>(la.a[blockIdx.y], tile * LPW, blockIdx.x, gridDim.x, lds);
}

template <int N, int LPW, int TL>
__global__ __launch_bounds__(LPW * TL) void k_row_lv(LevelArgs la) {
  __shared__ double2 lds[row_lds<double2, N, LPW>::elems];
  row_body<double2, N, LPW, TL, false>(la.a[blockIdx.y], blockIdx.x * LPW, lds);
}

template <int N, int LPW>
__global__ __launch_bounds__(LPW * tri_tl(N)) void k_tri_col_lv(LevelArgs la) {
  __shared__ double2 lds[tri_lds<N, LPW>::elems];
  const int tile = xcd_tile<(16 / LPW > 1 ? 16 / LPW : 1)>(blockIdx.x, gridDim.x);
  tri_col_body<N, LPW>(la.a[blockIdx.y], tile * LPW, blockIdx.x, gridDim.x, lds);
}

template <int N, int LPW>
__global__ __launch_bounds__(LPW * tri_tl(N)) void k_tri_row_lv(LevelArgs la) {
  __shared__ double2 lds[tri_lds<N, LPW>::elems];
  tri_row_body<N, LPW, false>(la.a[blockIdx.y], blockIdx.x * LPW, lds);
}

// ---------------------------------------------------------------- dispatch

bool line_length_supported(int N) {
  switch (N) {
#define X(n) case n:
    TDSE_LINE_SIZES(X)
#undef X
    return true;
    default:
      return false;
  }
}

// With events e0/e1 the launch records them at the kernel's own start and
// end (hipExtLaunchKernelGGL), which times the kernel without launch gaps.
#define TDSE_LAUNCH(K, G, B, S, E0, E1, A) \
  do { \
    if (E0) hipExtLaunchKernelGGL(K, G, B, 0, S, E0, E1, 0, A); \
    else hipLaunchKernelGGL(K, G, B, 0, S, A); \
  } while (0)

// The pointwise pass of a 1D problem (length 1) fills one workgroup with its
// M2 points; it gets extra, inactive workgroups so that the next row pass's
// phase table has one entry per thread.
inline int64_t col_blocks(int N, const LineArgs& a, int L, int T) {
  int64_t nb = (a.nlines + L - 1) / L;
  if (N == 1) {
    const int64_t entries = (int64_t)a.req.nj * (a.M1 + a.M2);
    nb = std::max<int64_t>(nb, std::min<int64_t>((entries + L * T - 1) / (L * T), 1024));
  }
  return nb;
}

// Lengths 3 * 2^a of FP64 plans take the passes in two layouts.  A split plan
// (ph32) keeps the one-layout passes in its FP64 start-up: another order of the
// same sums would change the last bits of what is then narrowed, and with them
// the rounding of the whole complex64 run.
template <typename C>
hipError_t col_pass(int N, const LineArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  switch (N) {
#define X(n) \
  case n: { \
    if (sizeof(C) == sizeof(double2) && three_smooth(n) && !a.ph32) { \
      constexpr int NN = three_smooth(n) ? n : 24, L = tri_col_lpw(NN); \
      TDSE_LAUNCH((k_tri_col<NN, L>), dim3((unsigned)((a.nlines + L - 1) / L)), dim3(L * tri_tl(NN)), s, e0, e1, a); \
    } else { \
      constexpr int L = (sizeof(C) == sizeof(float2) && n == 128) ? 16 : col_lpw(n), T = col_tl(n); \
      TDSE_LAUNCH((k_col<C, n, L, T>), dim3((unsigned)col_blocks(n, a, L, T)), dim3(L * T), s, e0, e1, a); \
    } \
    break; \
  }
    X(1)
    TDSE_LINE_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// middle-axis pass: the column pass's schedules (the lines are strided the same way)
template <typename C>
hipError_t mid_pass(int N, bool inverse, const LineArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (a.slab_lines < 1) return hipErrorInvalidValue;
  switch (N) {
#define X(n) \
  case n: { \
    if (sizeof(C) == sizeof(double2) && three_smooth(n) && !a.ph32) { \
      constexpr int NN = three_smooth(n) ? n : 24, L = tri_col_lpw(NN); \
      const dim3 g((unsigned)((a.nlines + L - 1) / L)); \
      if (inverse) TDSE_LAUNCH((k_tri_mid<NN, L, true>), g, dim3(L * tri_tl(NN)), s, e0, e1, a); \
      else TDSE_LAUNCH((k_tri_mid<NN, L, false>), g, dim3(L * tri_tl(NN)), s, e0, e1, a); \
    } else { \
      constexpr int L = (sizeof(C) == sizeof(float2) && n == 128) ? 16 : col_lpw(n), T = col_tl(n); \
      const dim3 g((unsigned)((a.nlines + L - 1) / L)); \
      if (inverse) TDSE_LAUNCH((k_mid<C, n, L, T, true>), g, dim3(L * T), s, e0, e1, a); \
      else TDSE_LAUNCH((k_mid<C, n, L, T, false>), g, dim3(L * T), s, e0, e1, a); \
    } \
    break; \
  }
    TDSE_LINE_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ... and rows with phase factors of their own along the line (no powers) where
// there are so many that the registers of seven terms and their factors, one
// wave per SIMD, cost more than the two layouts gain.  us per row pass, two
// layouts less one, in sub-steps (at most one term): 2048 x 384 +2.5, 4096 x 384
// +6.2, 1024 x 768 +1.2, 4096 x 768 +9.8, 16384 x 96 +5.4, 8192 x 192 +4.4; 1024 x 384
// -0.2, 512 x 768 -1.2, 8192 x 96 -0.5, 4096 x 192 -0.7.  Adams steps with a field along
// the rows, two layouts / one: 1536 x 768 42.1 / 34.8, 2048 x 384 29.6 / 26.3, 4096 x
// 384 50.1 / 49.4 (one wave per line fills two per SIMD with 2048 lines); 3072 x 384
// 40.0 / 43.3, 512 x 768 18.3 / 22.4, 4096 x 768 109 / 119, 16384 x 96 46.9 / 47.4.
inline bool tri_row(int N, const LineArgs& a) {
  if (a.pf_pow || N < 48) return true;
  const int64_t P = (int64_t)a.nlines * N;
  if (P < (N >= 384 ? 3 << 18 : 3 << 19)) return true;
  if (a.nh <= 1) return false;
  return N < 384 || P > 1 << 21 || (N == 384 && a.nlines % 2048 != 0);
}

template <typename C>
hipError_t row_pass(int N, const LineArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  switch (N) {
#define X(n) \
  case n: { \
    if (sizeof(C) == sizeof(double2) && three_smooth(n) && !a.ph32 && tri_row(n, a)) { \
      constexpr int NN = three_smooth(n) ? n : 24, L = tri_row_lpw(NN); \
      const dim3 g((a.nlines + L - 1) / L), b(L * tri_tl(NN)); \
      if (a.pf_pow) TDSE_LAUNCH((k_tri_row<NN, L, true>), g, b, s, e0, e1, a); \
      else TDSE_LAUNCH((k_tri_row<NN, L, false>), g, b, s, e0, e1, a); \
    } else { \
      constexpr int L = row_lpw(n), T = row_tl(n); \
      const dim3 g((a.nlines + L - 1) / L); \
      if (a.pf_pow) TDSE_LAUNCH((k_row<C, n, L, T, true>), g, dim3(L * T), s, e0, e1, a); \
      else TDSE_LAUNCH((k_row<C, n, L, T>), g, dim3(L * T), s, e0, e1, a); \
    } \
    break; \
  }
    TDSE_LINE_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_narrow(const double2* __restrict__ src, float2* __restrict__ dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = float2{(float)src[i].x, (float)src[i].y};
}

hipError_t launch_narrow(const double2* src, float2* dst, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_narrow, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}


hipError_t launch_col_pass(int prec, int N, const LineArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  return prec == P_SPLIT ? col_pass<float2>(N, a, s, e0, e1) : col_pass<double2>(N, a, s, e0, e1);
}
// `count` levels of one pass (2D FP64 plans; every level has the geometry of the first)
hipError_t launch_col_levels(int N, const LevelArgs& la, int count, hipStream_t s) {
  const LineArgs& a = la.a[0];
  switch (N) {
#define X(n) \
  case n: { \
    if constexpr (three_smooth(n)) { \
      constexpr int NN = three_smooth(n) ? n : 24, L = tri_col_lpw(NN); \
      hipLaunchKernelGGL((k_tri_col_lv<NN, L>), dim3((unsigned)((a.nlines + L - 1) / L), count), dim3(L * tri_tl(NN)), 0, s, la); \
    } else { \
      constexpr int NN = three_smooth(n) ? 8 : n, L = col_lpw(NN), T = col_tl(NN); \
      hipLaunchKernelGGL((k_col_lv<NN, L, T>), dim3((unsigned)((a.nlines + L - 1) / L), count), dim3(L * T), 0, s, la); \
    } \
    break; \
  }
    TDSE_LINE_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
hipError_t launch_row_levels(int N, const LevelArgs& la, int count, hipStream_t s) {
  const LineArgs& a = la.a[0];
  switch (N) {
#define X(n) \
  case n: { \
    if constexpr (three_smooth(n)) { \
      constexpr int NN = three_smooth(n) ? n : 24, L = tri_row_lpw(NN); \
      hipLaunchKernelGGL((k_tri_row_lv<NN, L>), dim3((unsigned)((a.nlines + L - 1) / L), count), dim3(L * tri_tl(NN)), 0, s, la); \
    } else { \
      constexpr int NN = three_smooth(n) ? 8 : n, L = row_lpw(NN), T = row_tl(NN); \
      hipLaunchKernelGGL((k_row_lv<NN, L, T>), dim3((unsigned)((a.nlines + L - 1) / L), count), dim3(L * T), 0, s, la); \
    } \
    break; \
  }
    TDSE_LINE_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
hipError_t launch_mid_pass(int prec, int N, bool inverse, const LineArgs& a, hipStream_t s, hipEvent_t e0,
                           hipEvent_t e1) {
  return prec == P_SPLIT ? mid_pass<float2>(N, inverse, a, s, e0, e1) : mid_pass<double2>(N, inverse, a, s, e0, e1);
}
hipError_t launch_row_pass(int prec, int N, const LineArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  return prec == P_SPLIT ? row_pass<float2>(N, a, s, e0, e1) : row_pass<double2>(N, a, s, e0, e1);
}

}  // namespace tdse
