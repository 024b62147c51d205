// One-workgroup run of a 1D periodic problem, gfx950: every time step of a
// tdse_step call (the Richardson start-up of Section 2.2 and the implicit
// Adams steps of eq. (uadamsk)) inside one kernel.
//
// A 1D line of N <= 2048 points fits one workgroup, so the two passes per
// step of the multi-launch path (a pointwise pass and a row pass, each a
// kernel launch) become one loop in which nothing leaves the workgroup: the
// physical values, the carried state B and the history sit in registers, the
// FFTs exchange through LDS (fft_held of fft_lds.h: the physical values in
// layout A, the modes in layout B), and a single potential field stays in
// registers too.  Per step the same arithmetic as the multi-launch path:
//   w = F^-1 B,  u = w / (1 + i mu_0 dt V(t_m)),  What_m = F(V(t_m) u),
//   uhat_m = B - i mu_0 dt What_m,
//   B_{m+1} = E^(1)(uhat_m - i dt mu_1 What_m) - i dt sum_{j>=2} mu_j E^(j) What_{m+1-j}.
// E^(j), the phase factor of Lemma 1 over [t_{m+1-j}, t_{m+1}], is the product
// of the j intervals' factors, so the history is held propagated: G_j =
// What_{m+1-j} carried to t_m, and a step multiplies each entry by the one
// factor E of [t_m, t_{m+1}]:
//   B_{m+1} = E (uhat_m - i dt mu_1 What_m - i dt sum_{j>=2} mu_j G_j),  G_{j+1} <- E G_j.
// E = exp(-i k^2 dt) exp(i k (phi(t_{m+1}) - phi(t_m))): a static factor (a
// table built once per plan in extended precision) times an increment computed
// from its own small argument (1 with A = 0), so no angle error grows with k or
// with the step count.  The newest n-1 entries What_m go to the history ring in
// memory, from which the next launch propagates them anew, by the same
// products in the same order; the longest lines leave the propagated entries
// themselves for it (run1d_holds), unless the field is changed in between.
//
// A step is latency: two transforms of three to five exchanges on one
// workgroup.  With the history read from the ring, a factor per history term
// and the twiddles, the factors and V read from LDS, a step of a 400-step run
// with a pulse took 6.2 us at N = 256 and 7.6 at 512; now 3.1 and 3.8.
//
// The start-up step from t_{m-1} runs, for each level l, 2^l order-2
// sub-steps of eq. (utrapk) with delta = dt / 2^l, chained through B in
// mode space as in the multi-launch path, and adds the level's result with
// its folded Richardson weight.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "fft_lds.h"
#include "tdse_internal.h"

namespace tdse {

namespace {

__device__ __forceinline__ int mode_of(int idx, int N) { return idx < (N >> 1) ? idx : idx - N; }

// (-i c) z
__device__ __forceinline__ double2 mi(double c, double2 z) { return double2{c * z.y, -c * z.x}; }

// a b with its roundings fixed: a history entry is propagated by the same
// operations inside a launch and at the start of the next one
__device__ __forceinline__ double2 cmul_fixed(double2 a, double2 b) {
  return double2{fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}

}  // namespace

// modes per thread (layout B), threads, and whether each thread holds its
// twiddles in registers (else the full table is in LDS)
constexpr int run1d_ept(int N) { return N % 3 == 0 ? 3 : 4; }
constexpr int run1d_threads(int N) { return N / run1d_ept(N); }
constexpr bool run1d_held(int N) { return N <= 512; }

// Lines whose propagated history stays in memory between launches.  At 2048
// points a launch of one step took 35.3 us when it propagated the ring anew,
// mostly the sines of that, and takes 21.0; below, the host's 38 us per launch
// hide it (15 us at 512), and the stores would cost the loop 2.5 to 3 % (512
// points 3.00 -> 3.10 us per step).
constexpr bool run1d_holds(int N) { return N >= 2048; }

// PH: the field A is nonzero, so the phase factors carry increments
template <int N, bool PH>
__global__ __launch_bounds__(run1d_threads(N)) void k_run1d(Run1DArgs a) {
  constexpr int EA = 4, TA = N / EA, EB = run1d_ept(N), TB = N / EB, H = MAXH - 1;
  constexpr bool HELD = run1d_held(N), HOLD = run1d_holds(N);
  constexpr double PI = 3.14159265358979323846264338327950288;
  HIP_DYNAMIC_SHARED(double2, run1d_lds)
  double2* la = run1d_lds;                          // the two exchange lines
  double2* lb = la + lds_line_len(N);
  double2* twl = lb + lds_line_len(N);              // twiddles (not held)
  const int t = threadIdx.x;
  const bool inA = N % 3 != 0 || t < TA;            // this thread has physical points
  const int n = a.order, nh = n - 1;
  const double* __restrict__ tab = a.tab;
  double2 hab[HELD ? held_count<N, false>() : 1], hba[HELD && N % 3 == 0 ? held_count<N, true>() : 1];
  if constexpr (HELD) {
    hold_twiddles<N, false>(hab, t, a.tw);
    if constexpr (N % 3 == 0) hold_twiddles<N, true>(hba, t, a.tw);
  } else {
    for (int q = t; q < N; q += TB) twl[q] = a.tw[q];
    __syncthreads();
  }
  const double2* twab = HELD ? hab : twl;
  const double2* twba = HELD ? (N % 3 == 0 ? hba : hab) : twl;
  // physical values (layout A) to modes (layout B), and back
  auto fwd = [&](double2* v) { fft_held<N, false, false, HELD>(v, t, la, lb, twab); };
  auto inv = [&](double2* v) { fft_held<N, true, true, HELD>(v, t, la, lb, twba); };

  // the first potential field at the thread's points
  double V0[EA];
#pragma unroll
  for (int q = 0; q < EA; ++q) V0[q] = a.vkind == 0 && a.nV > 0 && inA ? a.V[t + TA * q] : 0.0;
  // the potential at point t + TA q for the time factors fV (stored fields, or
  // the moving well with fV = {-V0, 1/(2 beta^2), -, centre, images})
  auto Vat = [&](const double* fV, int q) -> double {
    if (a.vkind == 1) {
      double d = -PI + 2.0 * PI * (t + TA * q) / N - fV[3];
      d -= 2.0 * PI * floor((d + PI) / (2.0 * PI));
      const double s = fV[1];
      double acc = exp(-(d * d) * s);
      const int K = (int)fV[4];
      for (int k = 1; k <= K; ++k) {
        const double y1 = d + 2.0 * PI * k, y2 = d - 2.0 * PI * k;
        acc += exp(-(y1 * y1) * s) + exp(-(y2 * y2) * s);
      }
      return fV[0] * acc;
    }
    double v = fV[0] * V0[q];
    for (int r = 1; r < a.nV; ++r) v += fV[r] * (inA ? a.V[r * a.vstride + t + TA * q] : 0.0);
    return v;
  };
  const double scale = 1.0 / N;
  // What = F(V(fV) u), into ring slot s
  auto history = [&](const double2* u, const double* fV, int s) {
    double2 w[EA];
#pragma unroll
    for (int q = 0; q < EA; ++q) {
      const double vs = Vat(fV, q) * scale;
      w[q] = double2{vs * u[q].x, vs * u[q].y};
    }
    fwd(w);
#pragma unroll
    for (int q = 0; q < EB; ++q) a.ring[(int64_t)s * N + t + TB * q] = w[q];
  };
  // exp(i k dphi) at mode t + TB q
  auto incr = [&](double dphi, int q) -> double2 {
    double s, c;
    sincos((double)mode_of(t + TB * q, N) * dphi, &s, &c);
    return double2{c, s};
  };

  double2 u[EA], B[EB];
  const int ns = a.ns;
  int m = a.m0 + 1;
  // ------------------------------------------------ Richardson start-up
#pragma unroll
  for (int q = 0; q < EA; ++q) u[q] = double2{0.0, 0.0};
  if (inA && (m <= ns || (m == ns + 1 && m <= a.m1))) {
#pragma unroll
    for (int q = 0; q < EA; ++q) u[q] = a.u_in[t + TA * q];
  }
  for (; m <= a.m1 && m <= ns; ++m) {
    if (m == 1) history(u, tab + a.oH, 0);
    const double* fpre = tab + a.oH + 8 * (m - 1);
    const double* lev = tab + a.oR + (int64_t)(m - 1) * 9 * ((1 << a.L) - 1);
    double2 acc[EA];
#pragma unroll
    for (int q = 0; q < EA; ++q) acc[q] = double2{0.0, 0.0};
    for (int l = 0; l < a.L; ++l) {
      const int nsub = 1 << l;
      const double hd = 0.5 * a.dt / nsub;   // delta / 2
      const double* sub = lev + 9 * (nsub - 1);
      double2 Sl[EB], v[EA];
#pragma unroll
      for (int q = 0; q < EB; ++q) Sl[q] = a.stab[(int64_t)(1 + l) * N + t + TB * q];
      // v = F((1 - i delta/2 V(t)) u)
#pragma unroll
      for (int q = 0; q < EA; ++q) {
        const double ci = -hd * Vat(fpre, q);
        v[q] = double2{(u[q].x - ci * u[q].y) * scale, (u[q].y + ci * u[q].x) * scale};
      }
      fwd(v);
      double2 Bs[EB];
#pragma unroll
      for (int q = 0; q < EB; ++q) {
        double2 E = Sl[q];
        if (PH) E = cmul(E, incr(sub[8], q));
        Bs[q] = cmul(E, v[q]);
      }
      for (int k = 0; k < nsub; ++k) {
        const double* fpost = sub + 9 * k;
#pragma unroll
        for (int q = 0; q < EB; ++q) v[q] = Bs[q];
        inv(v);
        double2 W[EA];
#pragma unroll
        for (int q = 0; q < EA; ++q) {
          const double Vs = Vat(fpost, q);
          const double qq = hd * Vs;
          const double iv = 1.0 / (1.0 + qq * qq);
          const double2 uu = double2{(v[q].x + qq * v[q].y) * iv, (v[q].y - qq * v[q].x) * iv};
          if (k == nsub - 1) {
            acc[q].x += a.rich[l] * uu.x;
            acc[q].y += a.rich[l] * uu.y;
          }
          const double s = Vs * scale;
          W[q] = double2{s * uu.x, s * uu.y};
        }
        if (k == nsub - 1) break;
        fwd(W);
        const double dphi = fpost[9 + 8];   // the next sub-step's phase increment
#pragma unroll
        for (int q = 0; q < EB; ++q) {
          double2 E = Sl[q];
          if (PH) E = cmul(E, incr(dphi, q));
          Bs[q] = cmul(E, double2{Bs[q].x + 2.0 * hd * W[q].y, Bs[q].y - 2.0 * hd * W[q].x});
        }
      }
    }
#pragma unroll
    for (int q = 0; q < EA; ++q) u[q] = acc[q];
    history(u, tab + a.oH + 8 * m, m % nh);
  }
  if (a.m1 <= ns) {
    if (inA) {
#pragma unroll
      for (int q = 0; q < EA; ++q) a.u_out[t + TA * q] = u[q];
    }
    return;
  }
  // ------------------------------------------------ implicit Adams steps
  double2 S1[EB];   // exp(-i k^2 dt)
#pragma unroll
  for (int q = 0; q < EB; ++q) S1[q] = a.stab[t + TB * q];
  // the factor of [t_{i-1}, t_i]
  auto factor = [&](int i, int q) -> double2 {
    if constexpr (PH) return cmul_fixed(S1[q], incr(tab[a.oD + i - 1], q));
    else return S1[q];
  };
  // the history propagated to t_{mm}: G_j = What_{mm+1-j}, j = 2..n-1
  double2 G[H - 1][EB];
  auto load_hist = [&](int mm) {
#pragma unroll
    for (int j = 2; j <= H; ++j)
#pragma unroll
      for (int q = 0; q < EB; ++q)
        G[j - 2][q] = j <= nh ? a.ring[(int64_t)(((mm + 1 - j) % nh + nh) % nh) * N + t + TB * q] : double2{0.0, 0.0};
    for (int i = mm + 2 - H; i <= mm; ++i) {
      if (i < 1) continue;
#pragma unroll
      for (int q = 0; q < EB; ++q) {
        const double2 E = factor(i, q);
#pragma unroll
        for (int j = 2; j <= H; ++j)
          if (i >= mm + 2 - j) G[j - 2][q] = cmul_fixed(E, G[j - 2][q]);   // past What_{mm+1-j}'s time
      }
    }
  };
  // B_{mm+1} from B (or uhat) and What_mm = W; the history moves on by one step
  auto form_B = [&](const double2* b, const double2* W, double c1, int mm) {
#pragma unroll
    for (int q = 0; q < EB; ++q) {
      double2 s = cadd(b[q], mi(c1, W[q]));
#pragma unroll
      for (int j = 2; j <= H; ++j) s = cadd(s, mi(a.ch[j], G[j - 2][q]));   // ch[j] = 0 past n - 1
      const double2 E = factor(mm + 1, q);
      B[q] = cmul(E, s);
#pragma unroll
      for (int j = H; j > 2; --j) G[j - 2][q] = cmul_fixed(E, G[j - 3][q]);
      G[0][q] = cmul_fixed(E, W[q]);
    }
  };
  if (m == ns + 1) {
    // the Adams start: uhat_ns = F u_ns, What_ns in the ring
    if (ns == 0) history(u, tab + a.oH, 0);
    double2 uh[EA], W[EB];
#pragma unroll
    for (int q = 0; q < EA; ++q) uh[q] = double2{u[q].x * scale, u[q].y * scale};
#pragma unroll
    for (int q = 0; q < EB; ++q) W[q] = a.ring[(int64_t)(ns % nh) * N + t + TB * q];
    load_hist(ns);
    fwd(uh);
    form_B(uh, W, a.ch[1], ns);
  } else {
#pragma unroll
    for (int q = 0; q < EB; ++q) B[q] = a.B[t + TB * q];
    if (HOLD && a.held) {
#pragma unroll
      for (int j = 2; j <= H; ++j)
#pragma unroll
        for (int q = 0; q < EB; ++q)
          G[j - 2][q] = j <= nh ? a.G[(int64_t)(j - 2) * N + t + TB * q] : double2{0.0, 0.0};
    } else {
      load_hist(m);
    }
  }
  for (; m <= a.m1; ++m) {
    const double* fV = tab + a.oA + 8 * (m - ns - 1);
    double2 v[EA];
#pragma unroll
    for (int q = 0; q < EB; ++q) v[q] = B[q];
    inv(v);
    double2 W[EA];
#pragma unroll
    for (int q = 0; q < EA; ++q) {
      const double Vs = Vat(fV, q);
      const double qq = a.c0 * Vs;
      const double iv = 1.0 / (1.0 + qq * qq);
      u[q] = double2{(v[q].x + qq * v[q].y) * iv, (v[q].y - qq * v[q].x) * iv};
      const double s = Vs * scale;
      W[q] = double2{s * u[q].x, s * u[q].y};
    }
    if (m == a.nsteps) break;
    fwd(W);
    // the newest entries stay in memory for what follows the launch
    if (m + nh > a.m1) {
#pragma unroll
      for (int q = 0; q < EB; ++q) a.ring[(int64_t)(m % nh) * N + t + TB * q] = W[q];
    }
    form_B(B, W, a.c0 + a.ch[1], m);
  }
  if (a.write_u && inA) {
#pragma unroll
    for (int q = 0; q < EA; ++q) a.u_out[t + TA * q] = u[q];
  }
  if (a.m1 < a.nsteps) {
#pragma unroll
    for (int q = 0; q < EB; ++q) a.B[t + TB * q] = B[q];
    if constexpr (HOLD) {
#pragma unroll
      for (int j = 2; j <= H; ++j)
#pragma unroll
        for (int q = 0; q < EB; ++q)
          if (j <= nh) a.G[(int64_t)(j - 2) * N + t + TB * q] = G[j - 2][q];
    }
  }
}

// Lengths 2^a up to 2048 and 3 * 2^a up to 1536: at most 512 threads, so that a
// thread has at least 256 registers for its modes and history.  us per step in
// pieces of 64 Adams steps with a pulse, two launches per step / this kernel:
// N = 192 31.9 / 3.0, 384 20.2 / 3.6, 768 23.9 / 4.3, 1024 14.1 / 5.2, 1536 36.7 /
// 8.3, 2048 28.2 / 10.6.
#define TDSE_RUN1D_SIZES(X) \
  X(8) X(16) X(32) X(64) X(128) X(256) X(512) X(1024) X(2048) X(24) X(48) X(96) X(192) X(384) X(768) X(1536)

bool run1d_supported(int N) {
  switch (N) {
#define X(n) case n:
    TDSE_RUN1D_SIZES(X)
#undef X
    return true;
    default:
      return false;
  }
}

size_t run1d_lds_bytes(int N) {
  return sizeof(double2) * (2 * (size_t)lds_line_len(N) + (run1d_held(N) ? 0 : N));
}

template <bool PH>
hipError_t run1d_dispatch(const Run1DArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const size_t lds = run1d_lds_bytes(a.M);
  switch (a.M) {
#define X(n)                                                                                                  \
  case n:                                                                                                     \
    if (e0) hipExtLaunchKernelGGL((k_run1d<n, PH>), dim3(1), dim3(run1d_threads(n)), lds, s, e0, e1, 0, a);   \
    else hipLaunchKernelGGL((k_run1d<n, PH>), dim3(1), dim3(run1d_threads(n)), lds, s, a);                    \
    break;
    TDSE_RUN1D_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_run1d(const Run1DArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  return a.has_phase ? run1d_dispatch<true>(a, s, e0, e1) : run1d_dispatch<false>(a, s, e0, e1);
}

}  // namespace tdse
