// Persistent implicit Adams steps of a square 2D periodic FP64 problem,
// gfx950: one co-resident grid marches many steps of eq. (uadamsk) with the
// multistep state held on chip.
//
// The grid has one workgroup per LPW = 2 lines (N/2 workgroups, one per
// compute unit for N = 512).  Workgroup b owns rows 2b, 2b+1 of the mode
// array in the row phase and columns 2b, 2b+1 of the grid in the column
// phase.  Per step m (the same arithmetic as the two-pass path):
//   column phase: inverse FFT along axis 0 of the tile (w = F^-1 B_m on the
//     grid), u = w / (1 + i mu_0 dt V(t_m)), g = V u / (N^2), forward FFT;
//   row phase:    forward FFT along axis 1 (What_m), uhat_m = B_m - i mu_0 dt What_m,
//     B_{m+1} = E^(1)(uhat_m - i dt mu_1 What_m) - i dt sum_{j>=2} mu_j E^(j) What_{m+1-j},
//     What_m into the history ring, inverse FFT along axis 1 (the next tile).
// The carried state B of a workgroup's rows stays in registers and its
// history ring in LDS for the whole launch, so per step only the N^2 tile
// crosses between workgroups (the two transposes of Section 2.2's 2D
// transform); a single potential field stays in registers too.  B and the
// ring touch memory only at the launch's start and end.
//
// Phase factor of Lemma 1: E^(j)(k1,k2) = T1_j(k1) T2_j(k2) with
// T_a,j(k) = exp(-i k^2 j dt + i k dphi_a,j); the row factor T1 is computed
// per step by 2 (n-1) threads of the workgroup with sincos, the column factor
// is a static table exp(-i k2^2 j dt) in registers times, when the field has
// a component along axis 1, a product of per-step increments
// exp(i k2 (phi_2(t_i) - phi_2(t_{i-1}))) kept as a shift register.
//
// The tile crosses workgroups (and XCDs, whose L2 caches are not coherent
// with each other) through device-scope accesses: every load and store of
// exchanged data is a 16-byte buffer access with device scope (sc1), served
// at the device's point of coherence, so no cache is ever written back or
// invalidated.  Each direction has a buffer of its own (xrow: column phase to
// row phase; xcol: row phase to column phase) in a blocked layout: the 2 x 2
// block of rows 2r, 2r+1 and columns 2c, 2c+1 is 64 contiguous bytes, blocks
// of a row pair in column order, so a row-phase workgroup reads and writes
// 32 N contiguous bytes and a column-phase workgroup moves whole 64-byte
// blocks.  The launch's first column phase reads the row-major tile of the
// two-pass path, and a launch that stops before T writes its last row phase
// in row-major order.
//
// What bounds a step is the latency of the two exchanges, so the data is its
// own flag: a buffer entry that has not arrived holds a signalling NaN that
// no arithmetic produces (results of the FFTs' additions are quiet), a reader
// polls its own entries until both halves of each are there, and puts the
// mark back.  No barrier, no arrival counter and no separate flag is needed:
// a workgroup can only write an entry again after it has received data that
// the entry's reader sent after its marks were complete (the reader waits
// for its own stores, then passes a workgroup barrier, before it sends).
// Measured at 512^2 (1000 steps, us per Adams step inside the launch): grid
// barriers with arrival counters 17.6, marked data 14.5, with the twiddles in
// registers and one barrier per exchange of a transform (fft_held) 13.1, with
// the marks put back behind the first transform 12.85; a copy without any
// exchange between workgroups takes 7.3.  The history stays at 16 bytes an
// entry and the column factors in a table: as powers of the first one
// they measured 0.5 slower.
//
// Every wait is bounded: a reader that polled spin_limit times reports a
// timeout to the host, takes what is there and waits no more, so every
// workgroup always runs to the end of the kernel.  What it takes early are
// marks, so the line it transforms becomes NaN, and with it all that the line
// reaches: a run that timed out never ends with finite wrong values.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fft_lds.h"
#include "tdse_internal.h"

namespace tdse {

namespace {

__device__ __forceinline__ int smode(int idx, int N) { return idx < (N >> 1) ? idx : idx - N; }

__device__ __forceinline__ double2 mi2(double c, double2 z) { return double2{c * z.y, -c * z.x}; }

// device-scope 16-byte accesses of a buffer (cache policy sc1)
constexpr int SC1 = 16;
__device__ __forceinline__ double2 cload(__amdgpu_buffer_rsrc_t rs, int64_t i) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(i * 16), 0, SC1));
}
__device__ __forceinline__ void cstore(__amdgpu_buffer_rsrc_t rs, int64_t i, double2 v) {
  using V4 = decltype(__builtin_amdgcn_raw_buffer_load_b128(rs, 0, 0, 0));
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(V4, v), rs, (int)(i * 16), 0, SC1);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const double2* p, int N) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, N * N * 16, 0x00020000);
}
// blocked exchange layout: element (k1, k2) of an N x N tile
__device__ __forceinline__ int64_t blk(int k1, int k2, int N) {
  return ((int64_t)(k1 >> 1) * (N >> 1) + (k2 >> 1)) * 4 + (k1 & 1) * 2 + (k2 & 1);
}

// the mark of an entry that has not arrived: a signalling NaN (an 8-byte half
// is written and read as one)
constexpr unsigned long long XMARK = 0x7FF0A5A5DEADBEEFull;
__device__ __forceinline__ double2 xmark() {
  const double d = __builtin_bit_cast(double, XMARK);
  return double2{d, d};
}
__device__ __forceinline__ bool arrived(double2 v) {
  return __builtin_bit_cast(unsigned long long, v.x) != XMARK && __builtin_bit_cast(unsigned long long, v.y) != XMARK;
}

// this thread's EPT entries (idx(q)) of an exchange buffer, once they are
// there.  `late`: this thread timed out before.
template <int EPT, typename F>
__device__ __forceinline__ void receive(__amdgpu_buffer_rsrc_t rs, F idx, double2 (&v)[EPT], int limit, unsigned* flag,
                                        unsigned run, bool& late) {
  int it = 0;
  for (;;) {
    bool ok = true;
#pragma unroll
    for (int q = 0; q < EPT; ++q) v[q] = cload(rs, idx(q));
#pragma unroll
    for (int q = 0; q < EPT; ++q) ok = ok && arrived(v[q]);
    if (ok || late) break;
    if (++it > limit) {
      late = true;
      __hip_atomic_store(flag, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");   // the loads are issued anew
  }
}
// this thread's stores are complete; the barriers of the transform that
// follows extend that to the workgroup before any of its sends
__device__ __forceinline__ void marks_complete() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
}

}  // namespace

// two lines, four elements per thread (three for 3 * 2^a)
constexpr int persist2d_threads(int N) { return 2 * (N / (N % 3 == 0 ? 3 : 4)); }

// PH2: the field has a component along axis 1 (the column factor carries increments)
template <int N, bool PH2>
__global__ __launch_bounds__(persist2d_threads(N)) void k_persist2d(Persist2DArgs a) {
  constexpr int LPW = 2, H = MAXH - 1;
  // elements per thread and threads per line of the transforms' two layouts:
  // A where data is received and sent, B where the pointwise work is done
  constexpr int EA = 4, TA = N / EA, EPT = N % 3 == 0 ? 3 : 4, TL = N / EPT;
  static_assert(EA < N, "the transforms must pass workgroup barriers (marks_complete)");
  constexpr int PC = lds_line_len(N) + 1;
  HIP_DYNAMIC_SHARED(double2, p2_lds)
  double2* xch = p2_lds;                          // FFT exchange lines (two of LPW * PC)
  double2* t1s = xch + 2 * LPW * PC;              // row factors T1 [LPW][H]
  double2* ringL = t1s + LPW * H;                 // history of the workgroup's rows [nh][LPW][N]
  const int tid = threadIdx.x, b = blockIdx.x;
  const int nh = a.order - 1;
  const double* __restrict__ tab = a.tab;
  // both phases: line i of the workgroup (lanes alternate between the two
  // lines); row phase: row LPW b + i, column phase: column LPW b + i
  const int i = tid % LPW, t = tid / LPW;
  const int line = LPW * b + i;
  double2* la = xch + i * PC;
  double2* lb = xch + (LPW + i) * PC;
  const bool inA = N % 3 != 0 || t < TA;
  const __amdgpu_buffer_rsrc_t rtile = rsrc(a.tile, N), xrow = rsrc(a.xrow, N), xcol = rsrc(a.xcol, N);

  double2 hab[held_count<N, false>()], hba[N % 3 == 0 ? held_count<N, true>() : 1];
  hold_twiddles<N, false>(hab, t, a.tw);
  if constexpr (N % 3 == 0) hold_twiddles<N, true>(hba, t, a.tw);
  auto fft_ab = [&](double2* v, auto inv) { fft_held<N, false, decltype(inv)::value>(v, t, la, lb, hab); };
  auto fft_ba = [&](double2* v, auto inv) {
    fft_held<N, true, decltype(inv)::value>(v, t, la, lb, N % 3 == 0 ? hba : hab);
  };
  using Fwd = std::false_type;
  using Inv = std::true_type;
  // state of the workgroup's rows: B in registers, the ring in LDS
  double2 B[EPT];
#pragma unroll
  for (int q = 0; q < EPT; ++q) B[q] = a.B[(int64_t)line * N + t + TL * q];
  for (int s = 0; s < nh; ++s) {
    if (s == (a.m0 + 1) % nh) continue;   // the entry the first step replaces
#pragma unroll
    for (int q = 0; q < EPT; ++q)
      ringL[(s * LPW + i) * N + t + TL * q] = a.ring[(int64_t)s * N * N + (int64_t)line * N + t + TL * q];
  }
  // static column factors exp(-i k2^2 j dt)
  double2 S2[H][EPT];
#pragma unroll
  for (int j = 1; j <= H; ++j)
#pragma unroll
    for (int q = 0; q < EPT; ++q) S2[j - 1][q] = j <= nh ? a.S2[(j - 1) * N + t + TL * q] : double2{1.0, 0.0};
  double2 dh[PH2 ? H : 1][EPT];
  auto incr2 = [&](double dphi, int q) -> double2 {
    double s, c;
    sincos((double)smode(t + TL * q, N) * dphi, &s, &c);
    return double2{c, s};
  };
  auto dphi2_at = [&](int ii) -> double { return ii >= 1 ? tab[a.oD2 + ii - 1] : 0.0; };
  if constexpr (PH2) {
#pragma unroll
    for (int ii = 1; ii < H; ++ii)
#pragma unroll
      for (int q = 0; q < EPT; ++q) dh[ii][q] = (ii < nh) ? incr2(dphi2_at(a.m0 + 2 - ii), q) : double2{1.0, 0.0};
  }
  // the first potential field at the workgroup's column
  double V0[EPT];
#pragma unroll
  for (int q = 0; q < EPT; ++q) V0[q] = a.V[(int64_t)(t + TL * q) * N + line];
  __syncthreads();

  bool late = false;
  const double scale = a.scale;
  for (int m = a.m0 + 1; m <= a.m1; ++m) {
    const double* st = tab + (int64_t)a.ostep * (m - a.mbase);   // fV[8], dphi1[H]
    // ------------------------------------------------ column phase (column `line`)
    {
      double2 v[EA];
      double vs[EPT];
#pragma unroll
      for (int q = 0; q < EPT; ++q) vs[q] = st[0] * V0[q];
      for (int r = 1; r < a.nV; ++r)
#pragma unroll
        for (int q = 0; q < EPT; ++q) vs[q] += st[r] * a.V[r * a.vstride + (int64_t)(t + TL * q) * N + line];
      if (inA) {
        if (m == a.m0 + 1) {   // the row-major tile of the two-pass path
#pragma unroll
          for (int q = 0; q < EA; ++q) v[q] = cload(rtile, (int64_t)(t + TA * q) * N + line);
        } else {
          receive<EA>(xcol, [&](int q) { return blk(t + TA * q, line, N); }, v, a.spin_limit, a.flag, a.run, late);
        }
      }
      fft_ab(v, Inv());
      if (inA && m > a.m0 + 1) {   // the marks go back, behind the transform's exchanges
#pragma unroll
        for (int q = 0; q < EA; ++q) cstore(xcol, blk(t + TA * q, line, N), xmark());
      }
      const bool out = a.write_u && m == a.m1;
#pragma unroll
      for (int q = 0; q < EPT; ++q) {
        const double qq = a.c0 * vs[q];
        const double iv = 1.0 / (1.0 + qq * qq);
        const double2 u = double2{(v[q].x + qq * v[q].y) * iv, (v[q].y - qq * v[q].x) * iv};
        if (out) a.uout[(int64_t)(t + TL * q) * N + line] = u;
        const double s = vs[q] * scale;
        v[q] = double2{s * u.x, s * u.y};
      }
      if (m == a.nsteps) break;   // the last step ends with u(T)
      marks_complete();
      fft_ba(v, Fwd());
      if (inA) {
#pragma unroll
        for (int q = 0; q < EA; ++q) cstore(xrow, blk(t + TA * q, line, N), v[q]);
      }
    }
    // ------------------------------------------------ row phase (row `line`)
    {
      double2 v[EA];
      // row factors T1_j for the workgroup's two rows, while the data is on
      // its way (the last reads of t1s lie behind the barriers above)
      if (tid < LPW * nh) {
        const int rr = tid / nh, j = tid % nh + 1;
        const double k = (double)smode(LPW * b + rr, N);
        double s, c;
        sincos(-(k * k) * (j * a.dt) + k * st[8 + j - 1], &s, &c);
        t1s[rr * H + j - 1] = double2{c, s};
      }
      if constexpr (PH2) {
#pragma unroll
        for (int q = 0; q < EPT; ++q) dh[0][q] = incr2(dphi2_at(m + 1), q);
      }
      if (inA) receive<EA>(xrow, [&](int q) { return blk(line, t + TA * q, N); }, v, a.spin_limit, a.flag, a.run, late);
      fft_ab(v, Fwd());   // its barriers publish t1s
      if (inA) {
#pragma unroll
        for (int q = 0; q < EA; ++q) cstore(xrow, blk(line, t + TA * q, N), xmark());
      }
      const int sw = m % nh;
      double2 T1[H];
#pragma unroll
      for (int j = 1; j <= H; ++j) T1[j - 1] = j <= nh ? t1s[i * H + j - 1] : double2{1.0, 0.0};
#pragma unroll
      for (int q = 0; q < EPT; ++q) {
        const int k2 = t + TL * q;
        const double2 W = v[q];
        const double2 uh = cadd(B[q], mi2(a.c0, W));
        double2 D = PH2 ? dh[0][q] : double2{1.0, 0.0};
        double2 E1 = cmul(T1[0], S2[0][q]);
        if constexpr (PH2) E1 = cmul(E1, D);
        double2 acc = cmul(E1, cadd(uh, mi2(a.ch[1], W)));
        double2 hist = double2{0.0, 0.0};
#pragma unroll
        for (int j = 2; j <= H; ++j) {
          if (j <= nh) {
            double2 Ej = cmul(T1[j - 1], S2[j - 1][q]);
            if constexpr (PH2) {
              D = cmul(D, dh[j - 1][q]);
              Ej = cmul(Ej, D);
            }
            const int sr = ((m + 1 - j) % nh + nh) % nh;
            hist = cadd(hist, mi2(a.ch[j], cmul(Ej, ringL[(sr * LPW + i) * N + k2])));
          }
        }
        B[q] = cadd(acc, hist);
        ringL[(sw * LPW + i) * N + k2] = W;
        v[q] = B[q];
      }
      if constexpr (PH2) {
#pragma unroll
        for (int ii = H - 1; ii >= 1; --ii)
#pragma unroll
          for (int q = 0; q < EPT; ++q) dh[ii][q] = dh[ii - 1][q];
      }
      marks_complete();
      fft_ba(v, Inv());
      if (!inA) continue;
      if (m == a.m1) {   // the launch ends before T: the row-major tile for the two-pass path
#pragma unroll
        for (int q = 0; q < EA; ++q) a.tile[(int64_t)line * N + t + TA * q] = v[q];
      } else {
#pragma unroll
        for (int q = 0; q < EA; ++q) cstore(xcol, blk(line, t + TA * q, N), v[q]);
      }
    }
  }
  // the state goes back to memory for the next launch (or the two-pass path):
  // of the history, the entries this launch made
  if (a.m1 < a.nsteps) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < EPT; ++q) a.B[(int64_t)line * N + t + TL * q] = B[q];
    for (int m = max(a.m0 + 1, a.m1 + 1 - nh); m <= a.m1; ++m) {
      const int s = m % nh;
#pragma unroll
      for (int q = 0; q < EPT; ++q)
        a.ring[(int64_t)s * N * N + (int64_t)line * N + t + TL * q] = ringL[(s * LPW + i) * N + t + TL * q];
    }
  }
}

// marks in both exchange buffers (n entries each), before the first launch of
// a run: every launch that ends before T leaves each entry marked, as its
// reader put it back and the last row phase sends none
__global__ __launch_bounds__(256) void k_persist2d_reset(double2* xrow, double2* xcol, int n) {
  const int g = blockIdx.x * 256 + threadIdx.x;
  if (g < n) {
    xrow[g] = xmark();
    xcol[g] = xmark();
  }
}

// Lengths 2^a and 3 * 2^a from 32 to 512 (at 512 two rows' history fills the
// LDS).  Faster than two kernel passes per step at each of them: 7.7-9.0 us
// per step of a whole run at 32..128, 10.0 against 29.7 at 192^2, 9.7 against
// 17 at 256^2, 13.1 against 28-31 at 384^2, 14.7 against 22 at 512^2.
#define TDSE_PERSIST2D_SIZES(X) X(32) X(48) X(64) X(96) X(128) X(192) X(256) X(384) X(512)

bool persist2d_supported(int N) {
  switch (N) {
#define X(n) case n:
    TDSE_PERSIST2D_SIZES(X)
#undef X
    return true;
    default:
      return false;
  }
}

size_t persist2d_lds_bytes(int N, int order) {
  return sizeof(double2) *
         (4 * (size_t)(lds_line_len(N) + 1) + 2 * (MAXH - 1) + (size_t)(order - 1) * 2 * N);
}

template <int N, bool PH2>
hipError_t persist2d_launch(const Persist2DArgs& a, hipStream_t s) {
  Persist2DArgs arg = a;
  void* args[] = {&arg};
  const size_t lds = persist2d_lds_bytes(N, a.order);
  if (!a.marked) {
    hipLaunchKernelGGL(k_persist2d_reset, dim3((N * N + 255) / 256), dim3(256), 0, s, a.xrow, a.xcol, N * N);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipLaunchCooperativeKernel(k_persist2d<N, PH2>, dim3(N / 2), dim3(persist2d_threads(N)), args, (unsigned)lds, s);
}

// Workgroups of the co-resident grid that fit the device at once (0 if the
// kernel cannot run), for the launch-time co-residency check.
int persist2d_capacity(int N, int order, bool ph2) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  const size_t lds = persist2d_lds_bytes(N, order);
  hipError_t e = hipErrorInvalidValue;
  switch (N) {
#define X(n)                                                                                                 \
  case n:                                                                                                    \
    e = ph2 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_persist2d<n, true>, persist2d_threads(n), lds)  \
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_persist2d<n, false>, persist2d_threads(n), lds); \
    break;
    TDSE_PERSIST2D_SIZES(X)
#undef X
    default:
      break;
  }
  return e == hipSuccess ? per * cus : 0;
}

hipError_t launch_persist2d(const Persist2DArgs& a, hipStream_t s) {
  const bool ph2 = a.ph2 != 0;
  switch (a.N) {
#define X(n) \
  case n:    \
    return ph2 ? persist2d_launch<n, true>(a, s) : persist2d_launch<n, false>(a, s);
    TDSE_PERSIST2D_SIZES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace tdse
