// HIP kernels of the reverse-mode derivative (adjoint) of the periodic
// scheme, FP64, gfx950.
//
// For a fixed vector potential the scheme (eq. (uadamsk) with the
// Richardson start-up of eq. (utrapk)) is linear in the state, and A enters
// only through the phase factors of Lemma 1,
//   E = exp(-i |k|^2 tau + i k . dphi),  dphi = phi(t_b) - phi(t_a).
// The reverse sweep applies the conjugate transpose of each operation; the
// transforms and the conjugated implicit solve reuse the forward passes, and
// these kernels do the mode-wise parts:
//   k_adj_am     the Adams phase's part of a reverse step n <= n_start: the
//                adjoint omega_{n-1} of What_{n-1} and per-workgroup partial
//                sums of dJ/d(dphi) of the phase factors of step n+1;
//   k_adj_sub    the conjugated phase factor of the Adams start;
//   k_adj_axpy, k_adj_phase, k_adj_phases, k_adj_reduce, k_adj_to_A  (helpers);
// and fused with the line FFTs on either side of them, as in the forward
// passes (periodic_body.h), for the many steps of the sweeps:
//   k_adj_row_am   forward FFT, an implicit Adams step, inverse FFT along axis 1;
//   k_adj_row_sub  forward FFT, a sub-step's phase factor, inverse FFT along axis 1;
//   k_adj_col      inverse FFT, a diagonal factor on the grid, forward FFT along axis 0.
// A reverse step is one column and one row pass (it was five launches, with
// Z, omega and the per-step phase table going through memory, and a gradient's
// time was the host's launch rate: 8 instances of 200 steps 90 ms).
#include <hip/hip_runtime.h>

#include "periodic_body.h"

namespace tdse {

__device__ __forceinline__ double2 conjd(double2 z) { return double2{z.x, -z.y}; }

// E at (k1 index, k2 index) from entry e of the per-axis table
__device__ __forceinline__ double2 adj_phase(const double2* ph, int per, int M1, int e, int i1, int i2) {
  return cmul(ph[e * per + i1], ph[e * per + M1 + i2]);
}

// Per-axis factors exp(i(-k^2 tau + k dphi_a)) of up to ADJ_PH entries.
__global__ __launch_bounds__(256) void k_adj_phase(AdjPhase q) {
  const int per = q.M1 + q.M2;
  const int total = q.nj * per;
  for (int idx = blockIdx.x * 256 + threadIdx.x; idx < total; idx += gridDim.x * 256) {
    const int e = idx / per;
    const int kk = idx - e * per;
    double k, dphi;
    if (kk < q.M1) {
      k = (double)signed_mode(kk, q.M1);
      dphi = q.dphi1[e];
    } else {
      k = (double)signed_mode(kk - q.M1, q.M2);
      dphi = q.dphi2[e];
    }
    double s, c;
    sincos(-(k * k) * q.tau[e] + k * dphi, &s, &c);
    q.ph[idx] = double2{c, s};
  }
}

__global__ __launch_bounds__(256) void k_adj_phases(AdjPhases q) {
  const int per = q.M1 + q.M2;
  const int64_t total = (int64_t)q.ne * per;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const int e = (int)(idx / per);
    const int kk = (int)(idx - (int64_t)e * per);
    const double* l = q.list + 3 * (int64_t)e;
    const bool row = kk < q.M1;
    const double k = (double)(row ? signed_mode(kk, q.M1) : signed_mode(kk - q.M1, q.M2));
    double s, c;
    sincos(-(k * k) * l[0] + k * l[row ? 1 : 2], &s, &c);
    q.ph[idx] = double2{c, s};
  }
}

// Block sum of NV values per thread into part[v * nblk + blockIdx.x].
template <int NV>
__device__ __forceinline__ void block_partials(double (&val)[NV], double* part, int nblk) {
  __shared__ double buf[NV][256];
  const int t = threadIdx.x;
#pragma unroll
  for (int v = 0; v < NV; ++v) buf[v][t] = val[v];
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) {
#pragma unroll
      for (int v = 0; v < NV; ++v) buf[v][t] += buf[v][t + s];
    }
    __syncthreads();
  }
  if (t < NV) part[(int64_t)t * nblk + blockIdx.x] = buf[t][0];
}

__global__ __launch_bounds__(256) void k_adj_am(AdjAm a) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool live = g < a.P;
  const int per = a.M1 + a.M2;
  const int H = a.H;
  double val[2 * MAXH];
#pragma unroll
  for (int v = 0; v < 2 * MAXH; ++v) val[v] = 0.0;
  if (live) {
    const int i1 = (int)(g / a.M2), i2 = (int)(g - (int64_t)i1 * a.M2);
    const double k1 = (double)signed_mode(i1, a.M1), k2 = (double)signed_mode(i2, a.M2);
    const double2 b1 = a.slot_b1 >= 0 ? a.beta[a.slot_b1 * a.P + g] : double2{0.0, 0.0};
    if (a.has_grad) {
      // step n+1: B_{n+1} = sum_j E^(j)_{n+1} x_j,
      //   x_1 = B_n - i c_1 What_n,  x_j = -i c_j What_{n+1-j};
      // dJ/dtheta = Re(conj(beta_{n+1}) i E x), weighted by k_a
      for (int j = 1; j <= H; ++j) {
        const double2 W = a.Wx[j][g];
        double2 x = double2{a.cx[j] * W.y, -a.cx[j] * W.x};   // -i c_j W
        if (j == 1) x = cadd(x, a.Bn[g]);
        const double2 Ex = cmul(adj_phase(a.ph, per, a.M1, j - 1, i1, i2), x);
        const double2 cb = conjd(b1);
        const double term = -(cb.x * Ex.y + cb.y * Ex.x);   // Re(conj(b) i E x)
        val[2 * (j - 1)] = k1 * term;
        val[2 * (j - 1) + 1] = k2 * term;
      }
    }
    if (a.omega) {
      // omega_{n-1} = sum_j i w_j conj(E^(j)_{n-1+j}) beta_{n-1+j}, beta_n = 0
      double2 om = double2{0.0, 0.0};
      for (int j = 2; j <= H; ++j) {
        if (a.wj[j] == 0.0 || a.slot_bj[j] < 0) continue;
        const double2 b = a.beta[a.slot_bj[j] * a.P + g];
        const double2 t = cmul(conjd(adj_phase(a.ph, per, a.M1, H + j - 1, i1, i2)), b);
        om = cadd(om, double2{-a.wj[j] * t.y, a.wj[j] * t.x});
      }
      a.omega[g] = om;
    }
  }
  if (a.has_grad) block_partials<2 * MAXH>(val, a.part, a.nblk);
}

// y = conj(E) y with the phase factor of entry 0 of the table
__global__ __launch_bounds__(256) void k_adj_sub(AdjSub a) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= a.P) return;
  const int i1 = (int)(g / a.M2), i2 = (int)(g - (int64_t)i1 * a.M2);
  a.y[g] = cmul(conjd(adj_phase(a.ph, a.M1 + a.M2, a.M1, 0, i1, i2)), a.y[g]);
}

// out = x + c y (complex c)
__global__ __launch_bounds__(256) void k_adj_axpy(int64_t P, const double2* x, const double2* y, double cr, double ci,
                                                  double2* out) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= P) return;
  out[g] = cadd(x[g], cmul(double2{cr, ci}, y[g]));
}

// red[r] = sum_b part[r * nblk + b], one workgroup per row
__global__ __launch_bounds__(256) void k_adj_reduce(const double* part, double* red, int nblk) {
  __shared__ double buf[256];
  const int r = blockIdx.x, t = threadIdx.x;
  double s = 0.0;
  for (int b = t; b < nblk; b += 256) s += part[(int64_t)r * nblk + b];
  buf[t] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) buf[t] += buf[t + w];
    __syncthreads();
  }
  if (t == 0) red[r] = buf[0];
}

// out[o] = sum_{e in [rowptr[o], rowptr[o+1])} wt[e] red[src[e]]
__global__ __launch_bounds__(256) void k_adj_to_A(const double* red, const int* rowptr, const int* src, const double* wt,
                                                  double* out, int nout) {
  const int o = blockIdx.x * 256 + threadIdx.x;
  if (o >= nout) return;
  double s = 0.0;
  for (int e = rowptr[o]; e < rowptr[o + 1]; ++e) s += wt[e] * red[src[e]];
  out[o] = s;
}

// ------------------------------------------------------------ fused passes

// Block sums of NV values per thread (NT threads, a power of two) into
// part[v * nblk + blockIdx.x], through LDS that holds NV * NT doubles.
template <int NV, int NT>
__device__ __forceinline__ void row_partials(const double (&val)[NV], double* buf, double* part, int nblk) {
  const int t = threadIdx.x;
  __syncthreads();   // the buffer held a transform's line
#pragma unroll
  for (int v = 0; v < NV; ++v) buf[v * NT + t] = val[v];
  __syncthreads();
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (t < s) {
#pragma unroll
      for (int v = 0; v < NV; ++v) buf[v * NT + t] += buf[v * NT + t + s];
    }
    __syncthreads();
  }
  for (int v = t; v < NV; v += NT) part[(int64_t)v * nblk + blockIdx.x] = buf[v * NT];
  __syncthreads();
}

// LDS of a fused row pass: the lines and twiddles of row_lds, or NV sums
template <int N, int L, int NT, int NV>
constexpr int adj_row_lds() {
  const int a = row_lds<double2, N, L>::elems, b = (NV * NT + 1) / 2;
  return a > b ? a : b;
}

// A row pass moves 18 entries of 16 bytes per mode (tile in and out, seven
// adjoint states and a new one, seven history entries, B_n) and is bound by
// that traffic on large grids, by latency on small ones.  PF: everything is
// loaded before the forward FFT, 16 entries per element in registers, which
// leaves one wave per SIMD; else term by term after it (four waves).
template <int N, int L, int TL, bool PF>
__global__ __launch_bounds__(L * TL) void k_adj_row_am(AdjRowAm a) {
  constexpr int NT = L * TL, EPT = N / TL, NH = MAXH - 1, PITCH = row_lds<double2, N, L>::PITCH;
  constexpr bool TWL = row_lds<double2, N, L>::TWL;
  __shared__ double2 lds[adj_row_lds<N, L, NT, 2 * NH>()];
  double2* twl = lds + L * PITCH;
  const int tid = threadIdx.x, i = tid / TL, t = tid % TL;
  const int i1 = blockIdx.x * L + i;
  const bool active = i1 < a.M1;
  const int per = a.M1 + a.M2, H = a.H;
  const int64_t g0 = (int64_t)(active ? i1 : 0) * N + t;
  const double2* __restrict__ prow = a.ph + (active ? i1 : 0);
  const double2* __restrict__ pcol = a.ph + a.M1 + t;
  if constexpr (TWL) {
    for (int q = tid; q < N; q += NT) twl[q] = a.tw[q];
  }
  double2 v[EPT], b1[EPT], om[EPT];
  double2 Bn[PF ? EPT : 1], Wr[PF ? NH : 1][EPT], br[PF ? NH - 1 : 1][EPT];
#pragma unroll
  for (int m = 0; m < EPT; ++m) {
    v[m] = active ? a.src[g0 + TL * m] : double2{0.0, 0.0};
    b1[m] = active && a.slot_b1 >= 0 ? a.beta[a.slot_b1 * a.P + g0 + TL * m] : double2{0.0, 0.0};
  }
  if constexpr (PF) {
    if (active && a.has_grad) {
#pragma unroll
      for (int m = 0; m < EPT; ++m) Bn[m] = a.Bn[g0 + TL * m];
#pragma unroll
      for (int j = 1; j <= NH; ++j) {
        if (j <= H) {
#pragma unroll
          for (int m = 0; m < EPT; ++m) Wr[j - 1][m] = a.Wx[j][g0 + TL * m];
        }
      }
    }
#pragma unroll
    for (int j = 2; j <= NH; ++j) {
      if (active && j <= H && a.slot_bj[j] >= 0) {
#pragma unroll
        for (int m = 0; m < EPT; ++m) br[j - 2][m] = a.beta[a.slot_bj[j] * a.P + g0 + TL * m];
      }
    }
  }
  if constexpr (TWL) __syncthreads();
  const double2* tw = TWL ? twl : a.tw;
  double2* myline = &lds[i * PITCH];
  fft_regs<N, TL, false>(v, t, myline, tw);
  double val[2 * NH];
#pragma unroll
  for (int j = 0; j < 2 * NH; ++j) val[j] = 0.0;
#pragma unroll
  for (int m = 0; m < EPT; ++m) om[m] = double2{0.0, 0.0};
  if (active) {
    const double k1 = (double)signed_mode(i1, a.M1);
    // beta_n = conj(E^(1)_{n+1}) beta_{n+1} + Z
    {
      const double2 R = prow[0];
#pragma unroll
      for (int m = 0; m < EPT; ++m) {
        v[m] = cadd(cmul(conjd(cmul(R, pcol[TL * m])), b1[m]), v[m]);
        a.beta[a.slot_bn * a.P + g0 + TL * m] = v[m];
      }
    }
    if (a.has_grad) {
      // B_{n+1} = sum_j E^(j)_{n+1} x_j, x_1 = B_n - i c_1 What_n, x_j = -i c_j What_{n+1-j};
      // dJ/dtheta = Re(conj(beta_{n+1}) i E x), weighted by k_a
#pragma unroll
      for (int j = 1; j <= NH; ++j) {
        if (j <= H) {
          const double2 R = prow[(j - 1) * per];
          const double2* __restrict__ W = a.Wx[j];
          double s1 = 0.0, s2 = 0.0;
#pragma unroll
          for (int m = 0; m < EPT; ++m) {
            const double2 w = PF ? Wr[PF ? j - 1 : 0][m] : W[g0 + TL * m];
            double2 x = double2{a.cx[j] * w.y, -a.cx[j] * w.x};
            if (j == 1) x = cadd(x, PF ? Bn[PF ? m : 0] : a.Bn[g0 + TL * m]);
            const double2 Ex = cmul(cmul(R, pcol[(j - 1) * per + TL * m]), x);
            const double term = b1[m].y * Ex.x - b1[m].x * Ex.y;
            s1 += term;
            s2 += (double)signed_mode(t + TL * m, N) * term;
          }
          val[2 * (j - 1)] = k1 * s1;
          val[2 * (j - 1) + 1] = s2;
        }
      }
    }
    // omega_{n-1} = sum_j i w_j conj(E^(j)_{n-1+j}) beta_{n-1+j}
#pragma unroll
    for (int j = 1; j <= NH; ++j) {
      if (j <= H && a.wj[j] != 0.0 && (j == 1 || a.slot_bj[j] >= 0)) {
        const double2 R = prow[(H + j - 1) * per];
        const double2* __restrict__ b = a.beta + (int64_t)(j == 1 ? 0 : a.slot_bj[j]) * a.P;
#pragma unroll
        for (int m = 0; m < EPT; ++m) {
          const double2 bb = j == 1 ? v[m] : PF ? br[PF ? j - 2 : 0][m] : b[g0 + TL * m];
          const double2 z = cmul(conjd(cmul(R, pcol[(H + j - 1) * per + TL * m])), bb);
          om[m] = cadd(om[m], double2{-a.wj[j] * z.y, a.wj[j] * z.x});
        }
      }
    }
    if (a.omega) {
#pragma unroll
      for (int m = 0; m < EPT; ++m) a.omega[g0 + TL * m] = om[m];
    }
  }
  if (a.has_grad) {
    row_partials<2 * NH, NT>(val, (double*)lds, a.part, a.nblk);
    if constexpr (TWL) {   // the sums took the twiddles' place
      for (int q = tid; q < N; q += NT) twl[q] = a.tw[q];
      __syncthreads();
    }
  }
  fft_regs<N, TL, true>(om, t, myline, tw);
  if (active) {
#pragma unroll
    for (int m = 0; m < EPT; ++m) a.dst[g0 + TL * m] = om[m];
  }
}

template <int N, int L, int TL>
__global__ __launch_bounds__(L * TL) void k_adj_row_sub(AdjRowSub a) {
  constexpr int NT = L * TL, EPT = N / TL, PITCH = row_lds<double2, N, L>::PITCH;
  constexpr bool TWL = row_lds<double2, N, L>::TWL;
  __shared__ double2 lds[row_lds<double2, N, L>::elems];
  __shared__ double sums[2 * NT];
  double2* twl = lds + L * PITCH;
  const int tid = threadIdx.x, i = tid / TL, t = tid % TL;
  const int i1 = blockIdx.x * L + i;
  const bool active = i1 < a.M1;
  const int64_t g0 = (int64_t)(active ? i1 : 0) * N + t;
  const double2 R = a.ph[active ? i1 : 0];
  const double2* __restrict__ pcol = a.ph + a.M1 + t;
  if constexpr (TWL) {
    for (int q = tid; q < N; q += NT) twl[q] = a.tw[q];
  }
  double2 v[EPT], G[EPT];
#pragma unroll
  for (int m = 0; m < EPT; ++m) {
    v[m] = active ? a.src[g0 + TL * m] : double2{0.0, 0.0};
    G[m] = active && a.rev ? a.G[g0 + TL * m] : double2{0.0, 0.0};
  }
  if constexpr (TWL) __syncthreads();
  const double2* tw = TWL ? twl : a.tw;
  double2* myline = &lds[i * PITCH];
  fft_regs<N, TL, false>(v, t, myline, tw);
  if (a.rev) {
    double val[2] = {0.0, 0.0};
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
      const double2 E = cmul(R, pcol[TL * m]);
      const double2 Ex = cmul(E, G[m]);
      const double term = v[m].y * Ex.x - v[m].x * Ex.y;   // Re(conj(y) i E g)
      val[0] += term;
      val[1] += (double)signed_mode(t + TL * m, N) * term;
      v[m] = cmul(conjd(E), v[m]);
    }
    val[0] *= (double)signed_mode(active ? i1 : 0, a.M1);
    row_partials<2, NT>(val, sums, a.part, a.nblk);
  } else {
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
      if (active) a.G[g0 + TL * m] = v[m];
      v[m] = cmul(cmul(R, pcol[TL * m]), v[m]);
    }
    if (!a.inv) return;
  }
  fft_regs<N, TL, true>(v, t, myline, tw);
  if (active) {
#pragma unroll
    for (int m = 0; m < EPT; ++m) a.dst[g0 + TL * m] = v[m];
  }
}

template <int N, int LPW, int TL>
__global__ __launch_bounds__(LPW * TL) void k_adj_col(AdjCol a) {
  constexpr int NT = LPW * TL, EPT = N / TL, PITCH = col_lds<double2, N, LPW>::PITCH;
  constexpr bool TWL = col_lds<double2, N, LPW>::TWL;
  __shared__ double2 lds[col_lds<double2, N, LPW>::elems];
  double2* twl = lds + LPW * PITCH;
  const int tid = threadIdx.x, i = tid % LPW, t = tid / LPW;
  const int tile = xcd_tile<(16 / LPW > 1 ? 16 / LPW : 1)>(blockIdx.x, gridDim.x);
  const int line = tile * LPW + i;
  const bool active = line < a.M2;
  const int64_t g0 = active ? (int64_t)t * a.M2 + line : 0, gs = active ? (int64_t)TL * a.M2 : 0;
  if constexpr (TWL) {
    for (int q = tid; q < N; q += NT) twl[q] = a.tw[q];
  }
  double2 v[EPT];
  const double2* __restrict__ x = a.src ? a.src : a.xin;
#pragma unroll
  for (int m = 0; m < EPT; ++m) v[m] = x[g0 + m * gs];
  double Vs[EPT];
#pragma unroll
  for (int m = 0; m < EPT; ++m) Vs[m] = 0.0;
  for (int r = 0; r < a.nV; ++r) {
#pragma unroll
    for (int m = 0; m < EPT; ++m) Vs[m] += a.fV[r] * a.V[r * a.vstride + g0 + m * gs];
  }
  if constexpr (TWL) __syncthreads();
  const double2* tw = TWL ? twl : a.tw;
  double2* myline = &lds[i * PITCH];
  if (a.src) fft_regs<N, TL, true>(v, t, myline, tw);
#pragma unroll
  for (int m = 0; m < EPT; ++m) {
    const double q = a.di * Vs[m], iv = a.s / (1.0 + q * q);
    // s (a + b V) / (1 + i q) = s (a + b V) (1 - i q) / (1 + q^2)
    const double2 f = cmul(double2{a.ar + a.br * Vs[m], a.bi * Vs[m]}, double2{iv, -q * iv});
    v[m] = cmul(f, v[m]);
    if (a.yout && active) {
      double2 y = v[m];
      if (a.accumulate) y = cadd(y, a.yout[g0 + m * gs]);
      a.yout[g0 + m * gs] = y;
    }
  }
  if (!a.dst) return;
  fft_regs<N, TL, false>(v, t, myline, tw);
  if (active) {
#pragma unroll
    for (int m = 0; m < EPT; ++m) a.dst[g0 + m * gs] = v[m];
  }
}

// Row schedules of the fused passes: those of the forward passes, but six
// elements per thread at 1536 and 3072.  A thread holds three arrays of its
// elements here; with twelve, lines of these lengths were slower than the
// unfused passes where there are few (adjoints of 100 steps, ms, unfused / twelve /
// six: 1536 points 15.3 / 16.6 / 13.3, 3072 17.5 / 18.5 / 17.1, 8 x 1536 17.4 / 17.9 /
// 14.6, 512 x 1536 35.3 / 31.3 / 27.0, 1536^2 112 / 98.6 / 85.0).
constexpr int adj_ept(int N) { return N == 1536 || N == 3072 ? 6 : row_ept(N); }
constexpr int adj_tl(int N) { return N / adj_ept(N); }
constexpr int adj_lpw(int N) { return N == 1536 || N == 3072 ? 1 : row_lpw(N); }

static int nb(int64_t n) { return (int)((n + 255) / 256); }

hipError_t launch_adj_phase(const AdjPhase& q, hipStream_t s) {
  hipLaunchKernelGGL(k_adj_phase, dim3(std::max(1, nb((int64_t)q.nj * (q.M1 + q.M2)))), dim3(256), 0, s, q);
  return hipGetLastError();
}
hipError_t launch_adj_am(const AdjAm& a, hipStream_t s) {
  hipLaunchKernelGGL(k_adj_am, dim3(a.nblk), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_adj_phases(const AdjPhases& q, hipStream_t s) {
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>(((int64_t)q.ne * (q.M1 + q.M2) + 255) / 256, 4096));
  hipLaunchKernelGGL(k_adj_phases, dim3((unsigned)blocks), dim3(256), 0, s, q);
  return hipGetLastError();
}
int adj_row_blocks(int M1, int M2) {
  switch (M2) {
#define X(n) case n: return (M1 + adj_lpw(n) - 1) / adj_lpw(n);
    TDSE_LINE_SIZES(X)
#undef X
    default:
      return 0;
  }
}
hipError_t launch_adj_row_am(const AdjRowAm& a, hipStream_t s) {
  // one wave per SIMD is all there is up to 2^18 modes (1024 waves of four
  // elements a lane): whole adjoints of 193 steps 13.95 -> 13.1 ms at 256^2,
  // 13.2 -> 12.3 at 1 x 1024, no difference at 512^2; beyond, the lost
  // occupancy costs (30.6 -> 34.4 ms at 512 x 1024, 49.7 -> 60.8 at 1024^2)
  const bool few = a.P < (1 << 18);
  const dim3 grid((unsigned)adj_row_blocks(a.M1, a.M2));
  switch (a.M2) {
#define X(n)                                                                                              \
  case n: {                                                                                               \
    constexpr bool PF = adj_ept(n) <= 4;                                                                  \
    const dim3 block(adj_lpw(n) * adj_tl(n));                                                             \
    if (PF && few) hipLaunchKernelGGL((k_adj_row_am<n, adj_lpw(n), adj_tl(n), PF>), grid, block, 0, s, a); \
    else hipLaunchKernelGGL((k_adj_row_am<n, adj_lpw(n), adj_tl(n), false>), grid, block, 0, s, a);        \
    break;                                                                                                \
  }
    TDSE_LINE_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
hipError_t launch_adj_row_sub(const AdjRowSub& a, hipStream_t s) {
  const dim3 grid((unsigned)adj_row_blocks(a.M1, a.M2));
  switch (a.M2) {
#define X(n)                                                                                             \
  case n: {                                                                                              \
    constexpr int L = adj_lpw(n), T = adj_tl(n);                                                         \
    hipLaunchKernelGGL((k_adj_row_sub<n, L, T>), grid, dim3(L * T), 0, s, a);                            \
    break;                                                                                               \
  }
    TDSE_LINE_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
hipError_t launch_adj_col(const AdjCol& a, hipStream_t s) {
  switch (a.M1) {
#define X(n)                                                                                             \
  case n: {                                                                                              \
    constexpr int L = col_lpw(n), T = col_tl(n);                                                         \
    hipLaunchKernelGGL((k_adj_col<n, L, T>), dim3((unsigned)((a.M2 + L - 1) / L)), dim3(L * T), 0, s, a); \
    break;                                                                                               \
  }
    X(1)
    TDSE_LINE_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
hipError_t launch_adj_sub(const AdjSub& a, hipStream_t s) {
  hipLaunchKernelGGL(k_adj_sub, dim3(nb(a.P)), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_adj_axpy(int64_t P, const double2* x, const double2* y, double cr, double ci, double2* out,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_adj_axpy, dim3(nb(P)), dim3(256), 0, s, P, x, y, cr, ci, out);
  return hipGetLastError();
}
hipError_t launch_adj_reduce(const double* part, double* red, int nrows, int nblk, hipStream_t s) {
  if (nrows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_adj_reduce, dim3(nrows), dim3(256), 0, s, part, red, nblk);
  return hipGetLastError();
}
hipError_t launch_adj_to_A(const double* red, const int* rowptr, const int* src, const double* wt, double* out, int nout,
                           hipStream_t s) {
  if (nout <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_adj_to_A, dim3(nb(nout)), dim3(256), 0, s, red, rowptr, src, wt, out, nout);
  return hipGetLastError();
}

}  // namespace tdse
