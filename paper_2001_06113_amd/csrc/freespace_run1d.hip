// One-workgroup run of a 1D free-space problem, gfx950: the implicit Adams
// steps of eq. (uadamsk) on the contour modes of one line inside one kernel.
//
// A 1D problem has one mode row, so the passes of the general path are one
// workgroup each, and a step of them is two launches whose time is the latency
// of tables, history and phase factors read from memory (M = 100, nu = 1024:
// row 16.0 us, pointwise pass and phase table 4.6 us, 21-24 us per step with
// the gaps).  Here the workgroup keeps everything for the whole launch: B and
// the history of its modes in registers, the transform tables in registers
// and LDS, the line in LDS.  Threads as in the ray-split line kernels (TL =
// nu/8 threads and four modes per thread on each ray); thread q < N_D also
// holds the dense mode q.  Per step m:
//   u = F^-1 B_m / (1 + i mu_0 dt V(t_m)),  W_m = F(V(t_m) u),
//   B_{m+1} = E (B_m - i dt (mu_0 + mu_1) W_m - i dt sum_{j>=2} mu_j G_j),
// with E the phase factor of Lemma 3.1 over [t_m, t_{m+1}] and G_j =
// What_{m+1-j} propagated to t_m: E^(j) is the product of the j intervals'
// factors, so a step multiplies each held entry by E once (G_{j+1} <- E G_j)
// and reads one factor per mode.  Those come from a table of the launch's
// steps that k_fs_run1d_phase fills on the whole device first.
//
// The propagated history stays in memory between two launches (a launch of one
// step that propagates the ring anew: M = 100, nu = 1024 30.2 -> 16.0 us, 64, 256
// 30.4 -> 19.2, 256, 2048 58.5 -> 38.4).
//
// The dense rows' sums are spread over all threads as (row, chunk) pairs going
// forward and (point, chunk) pairs coming back.
#include <hip/hip_runtime.h>

#include "fft_lds.h"
#include "freespace_line.h"
#include "tdse_internal.h"

namespace tdse {

// etab[(i - i0) N + k] = exp(i(-zeta_k^2 dt + zeta_k (phi(t_i) - phi(t_{i-1})))), i0 <= i < i0 + rows
__global__ __launch_bounds__(256) void k_fs_run1d_phase(FSRun1DArgs a, int rows) {
  const int N = a.ax.N;
  const int64_t total = (int64_t)rows * N;
  for (int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x; g < total; g += (int64_t)gridDim.x * 256) {
    const int i = (int)(g / N), k = (int)(g - (int64_t)i * N);
    const double2 z = a.ax.zeta[k], z2 = cmul(z, z);
    const double dphi = a.tab[FSRUN1D_COLS * (int64_t)(a.i0 + i) + FSRUN1D_COLS - 1];
    const double tr = -z2.x * a.dt + z.x * dphi, ti = -z2.y * a.dt + z.y * dphi;
    const double mag = exp(-ti);
    double s, c;
    sincos(tr, &s, &c);
    a.etab[g] = double2{mag * c, mag * s};
  }
}

// chunks of the dense sums: forward pairs (row, chunk), inverse pairs (point, chunk)
__host__ __device__ inline int fsr_chunks(int nth, int n) { return nth / n > 1 ? nth / n : 1; }

// LDS: line f[M] | dense modes[ND] | rows' values[NR] | partials | two FFT
// lines | nu twiddles | the inverse dense rows [NR][M] if they fit
size_t fs_run1d_lds_bytes(int nu, const CFAxis& ax, bool dinv) {
  const int nth = nu / 4;
  const size_t part = (size_t)std::max(ax.NR * fsr_chunks(nth, ax.NR), ax.M * fsr_chunks(nth, ax.M));
  return sizeof(double2) * ((size_t)ax.M + ax.ND + ax.NR + part + 2 * lds_line_len(nu) + nu +
                            (dinv ? (size_t)ax.NR * ax.M : 0));
}

template <int NU, bool CH, int MP>
__global__ __launch_bounds__(NU / 4) void k_fs_run1d(FSRun1DArgs a) {
  constexpr int EPT = 8, TL = NU / EPT, NTH = 2 * TL, RAY = EPT / 2, H = MAXH - 1;
  HIP_DYNAMIC_SHARED(double2, fsr_lds)
  const CFAxis& ax = a.ax;
  const int M = ax.M, N = ax.N, NE = ax.NE, ND = ax.ND, NR = CH ? ax.NR : ND, nh = a.order - 1;
  const int CF = fsr_chunks(NTH, NR), LF = (M + CF - 1) / CF;   // forward: chunks of a row, points of a chunk
  const int CI = fsr_chunks(NTH, M), LI = (NR + CI - 1) / CI;   // inverse: chunks of a point, rows of a chunk
  double2* fin = fsr_lds;
  double2* dm = fin + M;
  double2* dr = dm + ND;
  double2* part = dr + NR;
  double2* fline = part + max(NR * CF, M * CI);
  double2* fline2 = fline + lds_line_len(NU);
  double2* tw = fline2 + lds_line_len(NU);
  double2* dinv = tw + NU;
  const int tid = threadIdx.x;
  const bool ray = tid >= TL;   // false: E3 (forward FFT going in), true: E1 (inverse FFT)
  const int t = ray ? tid - TL : tid;
  double2* line = ray ? fline2 : fline;
  for (int q = tid; q < NU; q += NTH) tw[q] = ax.tw[q];
  if (a.dinv_lds)
    for (int q = tid; q < NR * M; q += NTH) dinv[q] = ax.Dinv[q];
  const double2* __restrict__ D = a.dinv_lds ? dinv : ax.Dinv;

  // the thread's modes (lanes past the end of the ray take its last mode and
  // count for nothing) and its entries of the transform tables
  int kk[RAY];
  bool live[RAY];
  double2 post[RAY], ipre[RAY], pre[MP], ipost[MP];
#pragma unroll
  for (int m = 0; m < RAY; ++m) {
    const int e = t + TL * m, ec = min(e, NE - 1);
    live[m] = e < NE;
    kk[m] = ray ? NE - 1 - ec : N - NE + ec;
    post[m] = (ray ? ax.post1 : ax.post3)[ec];
    ipre[m] = (ray ? ax.ipre1 : ax.ipre3)[ec];
  }
#pragma unroll
  for (int m = 0; m < MP; ++m) {
    const int ec = min(t + TL * m, M - 1);
    pre[m] = (ray ? ax.pre1 : ax.pre3)[ec];
    ipost[m] = (ray ? ax.ipost1 : ax.ipost3)[ec];
  }
  // the thread's pair of a dense row going forward
  const int fq = tid / CF, fj0 = (tid - fq * CF) * LF, fj1 = min(fj0 + LF, M);
  const bool fpair = fq < NR && fj0 < M;
  double2 fd = {0.0, 0.0}, fr = {0.0, 0.0};
  if (fpair) {
    fd = ax.Dfwd[(int64_t)fq * M + fj0];
    fr = ax.rfwd[fq];
  }
  const bool dense = tid < ND;
  const int kd = NE + min(tid, ND - 1);

  // B_{m0+1} and the history propagated to t_{m0+1}
  double2 B[RAY], G[H - 1][RAY], Bd = {0.0, 0.0}, Gd[H - 1];
  {
    const int m = a.m0 + 1;
#pragma unroll
    for (int q = 0; q < RAY; ++q) B[q] = live[q] ? a.Bm[kk[q]] : double2{0.0, 0.0};
    if (dense) Bd = a.Bm[kd];
#pragma unroll
    for (int j = 2; j <= H; ++j) {
#pragma unroll
      for (int q = 0; q < RAY; ++q) G[j - 2][q] = double2{0.0, 0.0};
      Gd[j - 2] = double2{0.0, 0.0};
      if (j <= nh && a.held) {
        const double2* __restrict__ g = a.G + (int64_t)(j - 2) * N;
#pragma unroll
        for (int q = 0; q < RAY; ++q) G[j - 2][q] = live[q] ? g[kk[q]] : double2{0.0, 0.0};
        if (dense) Gd[j - 2] = g[kd];
      } else if (j <= nh) {
        const double2* __restrict__ rj = a.ring + (int64_t)(((m + 1 - j) % nh + nh) % nh) * N;
#pragma unroll
        for (int q = 0; q < RAY; ++q) G[j - 2][q] = live[q] ? rj[kk[q]] : double2{0.0, 0.0};
        if (dense) Gd[j - 2] = rj[kd];
        for (int i = m + 2 - j; i <= m; ++i) {
          const double2* __restrict__ E = a.etab + (int64_t)(i - a.i0) * N;
#pragma unroll
          for (int q = 0; q < RAY; ++q) G[j - 2][q] = cmul(E[kk[q]], G[j - 2][q]);
          Gd[j - 2] = cmul(E[kd], Gd[j - 2]);
        }
      }
    }
  }
  if (dense) dm[tid] = Bd;
  __syncthreads();

  for (int m = a.m0 + 1; m <= a.m1; ++m) {
    const double* __restrict__ st = a.tab + FSRUN1D_COLS * (int64_t)m;   // f[8], first field, fields, -, dphi
    const bool last = m == a.nsteps;
    // the factors of [t_m, t_{m+1}], needed after the transforms
    double2 E[RAY], Ed = {0.0, 0.0};
    if (!last) {
      const double2* __restrict__ e = a.etab + (int64_t)(m + 1 - a.i0) * N;
#pragma unroll
      for (int q = 0; q < RAY; ++q) E[q] = e[kk[q]];
      Ed = e[kd];
    }
    // ------------------------------------------------ inverse transform of B_m
    {
      double2 w[EPT];
#pragma unroll
      for (int q = 0; q < EPT; ++q)
        w[q] = q < RAY ? conj_if(!ray, cmul(ipre[q < RAY ? q : 0], B[q < RAY ? q : 0])) : double2{0.0, 0.0};
      if constexpr (MP == 1) w[0] = fft_short_out<NU, TL, false>(w, t, line, tw);
      else fft_regs<NU, TL, false>(w, t, line, tw);
      // both rays' points into their lines (free: the transform ends with a barrier)
#pragma unroll
      for (int q = 0; q < MP; ++q)
        if (t + TL * q < M) line[t + TL * q] = cmul(ipost[q], conj_if(!ray, w[q]));
    }
    const double2* drow = dm;
    if constexpr (CH) {
      // contract the C-modes onto the interpolation nodes
      const int P = ax.NP, NT = ax.NT, NC = ND - 2 * P;
      const int LC = (NC + CF - 1) / CF;
      for (int i = tid; i < NR * CF; i += NTH) {
        const int r = i / CF, c = i - r * CF;
        double2 acc = {0.0, 0.0};
        if (r < P || r >= P + NT) {
          if (c == 0) acc = dm[r < P ? r : r - NT + NC];
        } else {
          const double2* __restrict__ pr = ax.Pi + (int64_t)(r - P) * NC;
          const int k1 = min(c * LC + LC, NC);
          for (int k = c * LC; k < k1; ++k) acc = cadd(acc, cmul(pr[k], dm[P + k]));
        }
        part[i] = acc;
      }
      __syncthreads();
      for (int r = tid; r < NR; r += NTH) {
        double2 acc = {0.0, 0.0};
        for (int c = 0; c < CF; ++c) acc = cadd(acc, part[r * CF + c]);
        dr[r] = acc;
      }
      __syncthreads();
      drow = dr;
    }
    for (int i = tid; i < M * CI; i += NTH) {   // pair (point e, chunk c): consecutive threads, consecutive points
      const int c = i / M, e = i - c * M;
      const int q1 = min(c * LI + LI, NR);
      double2 acc = {0.0, 0.0};
      for (int q = c * LI; q < q1; q += 4) {
        double2 d[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = D[(int64_t)min(q + k, q1 - 1) * M + e];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (q + k < q1) acc = cadd(acc, cmul(d[k], drow[q + k]));
      }
      part[i] = acc;
    }
    __syncthreads();
    // ------------------------------------------------ the diagonal solve
    const double* __restrict__ V = a.V + (int64_t)st[8] * a.vstride;
    const int nV = (int)st[9];
    for (int e = tid; e < M; e += NTH) {
      double2 wv = cadd(fline[e], fline2[e]);
      for (int c = 0; c < CI; ++c) wv = cadd(wv, part[c * M + e]);
      double Vs = 0.0;
      for (int r = 0; r < nV; ++r) Vs += st[r] * V[r * a.vstride + e];
      const double q = a.c0 * Vs, iv = 1.0 / (1.0 + q * q);
      const double2 u = double2{(wv.x + q * wv.y) * iv, (wv.y - q * wv.x) * iv};
      if (m == a.m1) a.uout[e] = u;
      fin[e] = double2{Vs * u.x, Vs * u.y};
    }
    if (last) break;
    __syncthreads();
    // ------------------------------------------------ forward transform of V u
    if (fpair) part[tid] = cmul(fd, geometric_sum(fin, fj0, fj1, fr));
    else if (fq < NR) part[tid] = double2{0.0, 0.0};
    double2 W[RAY], Wd = {0.0, 0.0};
    {
      double2 w[EPT];
#pragma unroll
      for (int q = 0; q < EPT; ++q) {
        const int e = t + TL * q;
        const double2 x = q < MP ? conj_if(ray, cmul(pre[q < MP ? q : 0], fin[min(e, M - 1)])) : double2{0.0, 0.0};
        w[q] = q < MP && e < M ? x : double2{0.0, 0.0};
      }
      if constexpr (MP == 1) fft_short_in<NU, TL, false>(w[0], w, t, line, tw);
      else fft_regs<NU, TL, false>(w, t, line, tw);
#pragma unroll
      for (int q = 0; q < RAY; ++q) W[q] = live[q] ? cmul(post[q], conj_if(ray, w[q])) : double2{0.0, 0.0};
    }
    // the transform's barriers published the rows' partial sums
    if constexpr (!CH) {
      if (dense)
        for (int c = 0; c < CF; ++c) Wd = cadd(Wd, part[tid * CF + c]);
    } else {
      for (int r = tid; r < NR; r += NTH) {
        double2 acc = {0.0, 0.0};
        for (int c = 0; c < CF; ++c) acc = cadd(acc, part[r * CF + c]);
        dr[r] = acc;
      }
      __syncthreads();
      if (dense) {
        const int P = ax.NP, NT = ax.NT, NC = ND - 2 * P;
        if (tid < P) Wd = dr[tid];
        else if (tid >= P + NC) Wd = dr[tid - NC + NT];
        else {
          const double* __restrict__ pr = ax.Pf + (int64_t)(tid - P) * NT;
          for (int k = 0; k < NT; ++k) {
            const double wt = pr[k];
            const double2 y = dr[P + k];
            Wd.x += wt * y.x;
            Wd.y += wt * y.y;
          }
        }
      }
    }
    // the newest nh history entries stay in memory for what follows the launch
    if (m + nh > a.m1) {
      double2* __restrict__ rw = a.ring + (int64_t)(m % nh) * N;
#pragma unroll
      for (int q = 0; q < RAY; ++q)
        if (live[q]) rw[kk[q]] = W[q];
      if (dense) rw[kd] = Wd;
    }
    // ------------------------------------------------ the Adams step
    const double c01 = a.c0 + a.ch[1];
#pragma unroll
    for (int q = 0; q < RAY; ++q) {
      double2 s = cadd(B[q], fs_mul_mi(c01, W[q]));
#pragma unroll
      for (int j = 2; j <= H; ++j) s = cadd(s, fs_mul_mi(a.ch[j], G[j - 2][q]));   // ch[j] = 0 past n - 1
      B[q] = live[q] ? cmul(E[q], s) : double2{0.0, 0.0};
#pragma unroll
      for (int j = H; j > 2; --j) G[j - 2][q] = cmul(E[q], G[j - 3][q]);
      G[0][q] = cmul(E[q], W[q]);
    }
    {
      double2 s = cadd(Bd, fs_mul_mi(c01, Wd));
#pragma unroll
      for (int j = 2; j <= H; ++j) s = cadd(s, fs_mul_mi(a.ch[j], Gd[j - 2]));
      Bd = cmul(Ed, s);
#pragma unroll
      for (int j = H; j > 2; --j) Gd[j - 2] = cmul(Ed, Gd[j - 3]);
      Gd[0] = cmul(Ed, Wd);
    }
    if (dense) dm[tid] = Bd;   // read after the next inverse transform's barriers
  }
  // B_{m1+1}, or B_N at T
#pragma unroll
  for (int q = 0; q < RAY; ++q)
    if (live[q]) a.Bm[kk[q]] = B[q];
  if (dense) a.Bm[kd] = Bd;
  if (a.m1 == a.nsteps) return;
#pragma unroll
  for (int j = 2; j <= H; ++j) {
    if (j <= nh) {
      double2* __restrict__ g = a.G + (int64_t)(j - 2) * N;
#pragma unroll
      for (int q = 0; q < RAY; ++q)
        if (live[q]) g[kk[q]] = G[j - 2][q];
      if (dense) g[kd] = Gd[j - 2];
    }
  }
}

constexpr size_t FSR_LDS = 160 * 1024;

// Eligible lines: every dense mode on a thread of its own, every grid point in
// the rays' lines, and the LDS of one compute unit.  us per Adams step over 600
// steps, the passes / this kernel: M = 64, nu = 256 16.7 / 8.7; 100, 1024 20.2 /
// 7.8; 128, 1024 through the interpolant 22.1 / 10.2; 256, 2048 22.9 / 17.7 (512
// threads: 160 of their registers spill).
bool fs_run1d_supported(int nu, const CFAxis& ax) {
  return ax.ND <= nu / 4 && ax.NR <= nu / 4 && ax.M <= nu && fs_run1d_lds_bytes(nu, ax, false) <= FSR_LDS;
}

hipError_t launch_fs_run1d(int nu, const FSRun1DArgs& a0, hipStream_t s) {
  FSRun1DArgs a = a0;
  a.dinv_lds = fs_run1d_lds_bytes(nu, a.ax, true) <= FSR_LDS;
  const size_t lds = fs_run1d_lds_bytes(nu, a.ax, a.dinv_lds != 0);
  const int rows = std::min(a.m1 + 1, a.nsteps) - a.i0 + 1;
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>(((int64_t)rows * a.ax.N + 255) / 256, 4096));
  if (rows > 0) {
    hipLaunchKernelGGL(k_fs_run1d_phase, dim3((unsigned)blocks), dim3(256), 0, s, a, rows);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
#define Y(n, mp)                                                                                       \
  case mp:                                                                                             \
    if (a.ax.NT) hipLaunchKernelGGL((k_fs_run1d<n, true, mp>), dim3(1), dim3(n / 4), lds, s, a);      \
    else hipLaunchKernelGGL((k_fs_run1d<n, false, mp>), dim3(1), dim3(n / 4), lds, s, a);             \
    break;
#define X(n)                                 \
  case n:                                    \
    switch (fs_points(n, a.ax.M, 8)) {       \
      Y(n, 1) Y(n, 2) Y(n, 4) Y(n, 8)        \
    }                                        \
    break;
  switch (nu) {
    X(256) X(512) X(1024) X(2048)
    default:
      return hipErrorInvalidValue;
  }
#undef X
#undef Y
  return hipGetLastError();
}

}  // namespace tdse
