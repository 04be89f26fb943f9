// Newton's-method localisation of a point source from one row of FFT-beam
// intensities of a linear array (Sec. "Localization"), batched over rows.
//
// With the regridded pointed beam of eq. e:bp_max_arbitrary,
//   b_p(y) = sum_A w^A(y) b_A,   w^A(y) = D(y - A/M) / M,
//   D(u) = sin((2n-1) pi u) / sin(pi u),
// the estimator in y = (d/lambda) sin(theta) replaces the likelihood's
// curvature by its value at the maximum (the baseline moment of inertia,
// eq. e:baseline_MOI) and iterates
//   y <- y + n^2 b_p'(y) / (4 pi^2 MOI b_p(y)),
// starting from the strongest FFT beam and summing over the K beams nearest
// it (the paper keeps ~10).  An update is not taken, and the iteration
// stops, when b_p <= 0 or when it would leave one beam spacing around the
// starting beam.
//
// Each 64-lane wavefront owns 64 rows.  It takes their argmax four rows at
// a time (lane l holds the PER consecutive beams from l PER on) while the next
// four rows' loads are in flight: the largest value by a prefix maximum over
// the lanes (DPP), its lowest index from the masks of the lanes that hold it
// (one compare per beam of a lane, the rest on the scalar unit).  The four rows
// pass through LDS, from where 16 lanes a row pick the K window beams (more than
// 16: one row at a time, a lane a beam); then
// every lane runs the Newton phase for one row.  Bound by the reads: 131072
// rows of 512 beams (268 MB) take 61 us, 4.4 TB/s; with each four rows' loads
// waited for, a (value, index) argmax of about 120 vector instructions a row
// and the closed form of D and D' beam by beam it took 79.
//
// The window beams A_j = A_0 + j sit at u_j = u_0 - j/M, and with M = 2 n,
// N = 2 n - 1 = M - 1,
//   D(u_j) = (-1)^j (P t_j - Q),  D'(u_j) = (-1)^j pi (M (Q t_j + P) - P (1 + t_j^2)),
//   t_j = cot(pi u_j),  P = sin(pi M u_0),  Q = cos(pi M u_0),
// so an evaluation is one sincospi pair of u_0 and one of M u_0, and per beam
// the angle addition with the FP64 constants of j/M (held in LDS), one
// reciprocal and the sums of (-1)^j b_j t_j and (-1)^j b_j t_j^2; a Taylor branch
// within 0.01 / (pi N) of an integer takes over where these cancel.
#include "dev_common.h"
#include "kernels.h"

namespace fftbf {

namespace {

constexpr double kPiD = 3.14159265358979323846;

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// max with the lane that the DPP control CTRL brings in, in the rows of ROWS
template <int CTRL, int ROWS>
__device__ __forceinline__ float max_dpp(float v) {
  const int x = __builtin_bit_cast(int, v);
  return fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, x, CTRL, ROWS, 0xF, false)));
}

// the largest of the wavefront's values, NaN ignored (NaN if there are only NaN)
__device__ __forceinline__ float wave_max(float v) {
  v = max_dpp<0x111, 0xF>(v);      // row_shr 1, 2, 4, 8: lane 15 of a row holds the row's
  v = max_dpp<0x112, 0xF>(v);
  v = max_dpp<0x114, 0xF>(v);
  v = max_dpp<0x118, 0xF>(v);
  v = max_dpp<0x142, 0xA>(v);      // row_bcast 15, 31: lane 63 holds all
  v = max_dpp<0x143, 0xC>(v);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Window of up to KMAX beams per row (16 or 64); PER = max(1, m / 64) beams
// per lane in the argmax; VEC loads them as 16-byte vectors (PER >= 4 and a
// 16-byte aligned input).
template <int PER, bool VEC, int KMAX>
__global__ __launch_bounds__(256) void k_localize(LocArgs a) {
  constexpr int WS = KMAX + 1;                     // padded LDS row of window beams
  // rows that pass through LDS at a time: with the wide window four would leave
  // room for one workgroup per CU instead of two (131072 rows of 512 beams, 64 of
  // them in the window: 153 us against 111)
  constexpr int RB = KMAX > 16 ? 1 : 4;
  static_assert(2 * (4 * 4 * 64 * WS + 2 * 8 * KMAX + 4 * 4 * RB * 64 * PER) <= 160 * 1024, "two workgroups per CU");
  __shared__ float win[4][64 * WS];
  __shared__ double tab[2][KMAX];                  // cos, sin of pi j/M
  __shared__ __attribute__((aligned(16))) float rows[4][RB][64 * PER];  // the rows at hand
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = a.m, K = a.n_window, N = 2 * a.n - 1;
  const double inv_m = 1.0 / (double)m;
  if (threadIdx.x < KMAX) {
    const int jj = threadIdx.x;
    sincospi((double)jj * inv_m, &tab[1][jj], &tab[0][jj]);
  }
  __syncthreads();
  const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * 64;
  if (row0 >= a.n_rows) return;                    // wave-uniform, after the only barrier
  float* w = win[wave];
  const int half = (K - 1) / 2;

  // ---- argmax of the wave's 64 rows, four at a time; window beams to LDS ----
  int my_a0 = 0;
  float nv[4][PER];                                // the next four rows, in flight
  auto load = [&](int rb) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t rr = row0 + rb + r < a.n_rows ? row0 + rb + r : a.n_rows - 1;   // rows past the end: unused
      const float* x = a.in + rr * m + lane * PER;
      if constexpr (VEC) {
#pragma unroll
        for (int q = 0; q < PER / 4; ++q) {
          const float4 f = reinterpret_cast<const float4*>(x)[q];
          nv[r][4 * q] = f.x;
          nv[r][4 * q + 1] = f.y;
          nv[r][4 * q + 2] = f.z;
          nv[r][4 * q + 3] = f.w;
        }
      } else {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          nv[r][i] = -INFINITY;
          if (lane * PER + i < m) nv[r][i] = x[i];   // lanes past a short row load nothing
        }
      }
    }
  };
  load(0);
  for (int rb = 0; rb < 64; rb += 4) {
    float v[4][PER];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < PER; ++i) v[r][i] = nv[r][i];
    if (rb + 4 < 64) load(rb + 4);
    int a0[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float best = v[r][0];
#pragma unroll
      for (int i = 1; i < PER; ++i) best = fmaxf(best, v[r][i]);
      best = wave_max(best);
      // lowest lane that holds it, then that lane's lowest beam (no lane: 0)
      uint64_t at[PER], any = 0;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        at[i] = __ballot(v[r][i] == best);
        any |= at[i];
      }
      const int l = any ? __builtin_ctzll(any) : 0;
      int i0 = 0;
#pragma unroll
      for (int i = PER - 1; i >= 0; --i)
        if (at[i] >> l & 1) i0 = i;
      a0[r] = l * PER + i0;
      if (lane == rb + r) my_a0 = a0[r];
    }
    // window beams A = a0 - half + jj (mod m, a power of two), jj < K
#pragma unroll
    for (int r0 = 0; r0 < 4; r0 += RB) {
#pragma unroll
      for (int r = r0; r < r0 + RB; ++r) {
        float* const x = &rows[wave][r - r0][lane * PER];
        if constexpr (PER >= 4) {
#pragma unroll
          for (int q = 0; q < PER / 4; ++q)
            reinterpret_cast<float4*>(x)[q] = make_float4(v[r][4 * q], v[r][4 * q + 1], v[r][4 * q + 2], v[r][4 * q + 3]);
        } else {
#pragma unroll
          for (int i = 0; i < PER; ++i) x[i] = v[r][i];
        }
      }
      wave_lds_sync();
      if constexpr (RB == 4) {
        const int r = lane >> 4, jj = lane & 15;
        const int ar = r < 2 ? (r ? a0[1] : a0[0]) : (r == 2 ? a0[2] : a0[3]);
        if (jj < K) w[(rb + r) * WS + jj] = rows[wave][r][(ar - half + jj) & (m - 1)];
      } else {
        if (lane < K) w[(rb + r0) * WS + lane] = rows[wave][0][(a0[r0] - half + lane) & (m - 1)];
      }
      wave_lds_sync();
    }
  }
  // ---- Newton phase: lane = row ----
  const int64_t row = row0 + lane;
  const bool row_ok = row < a.n_rows;
  const double y0 = (double)my_a0 * inv_m;
  const double gain = (double)a.n * (double)a.n / (4.0 * kPiD * kPiD * a.moi);
  const double Nd = (double)N;
  const float* wr = w + lane * WS;

  auto eval = [&](double y, double& p, double& dp) {
    // u_j = y - A_j / M with A_j = a0 - half + j; reduced to [-1/2, 1/2] for j = 0
    double u0 = y - (double)(my_a0 - half) * inv_m;
    u0 -= rint(u0);
    double s0, c0, P, Q;
    sincospi(u0, &s0, &c0);
    sincospi((double)m * u0, &P, &Q);
    double sp = 0.0, sdp = 0.0;                      // of the beams at the singular point
    double T0 = 0.0, T1 = 0.0, T2 = 0.0;             // sums of (-1)^j b_j t_j^k over the others
    for (int j = 0; j < K; ++j) {
      const float b = wr[j];
      const double cj = tab[0][j], sj = tab[1][j];
      const double s = s0 * cj - c0 * sj, c = c0 * cj + s0 * sj;      // of pi u_j
      if (fabs(Nd * s) < 0.01) {
        const double x = copysign(s, s * c) * (1.0 + s * s / 6.0), x2 = x * x, N2 = Nd * Nd;
        const double c4 = (3.0 * N2 * N2 - 10.0 * N2 + 7.0);
        sp = fma(Nd * (1.0 - (N2 - 1.0) * x2 / 6.0 + c4 * x2 * x2 / 360.0), (double)b, sp);
        sdp = fma(kPiD * Nd * (-(N2 - 1.0) * x / 3.0 + c4 * x2 * x / 90.0), (double)b, sdp);
      } else {
        double r = __builtin_amdgcn_rcp(s);
        r = fma(fma(-s, r, 1.0), r, r);
        r = fma(fma(-s, r, 1.0), r, r);
        const double t = c * r, bj = (double)(j & 1 ? -b : b), bt = bj * t;
        T0 += bj;
        T1 += bt;
        T2 = fma(bt, t, T2);
      }
    }
    p = (sp + (P * T1 - Q * T0)) * inv_m;
    dp = (sdp + kPiD * ((double)m * (Q * T1 + P * T0) - P * (T0 + T2))) * inv_m;
  };

  double y = y0, p, dp;
  bool done = false;
  for (int it = 0; it < a.n_iter; ++it) {
    eval(y, p, dp);
    if (!done) {
      const double yn = y + gain * dp / p;
      if (!(p > 0.0) || fabs(yn - y0) > inv_m) done = true;
      else y = yn;
    }
  }
  eval(y, p, dp);
  if (row_ok) {
    const double yw = (y + 0.5) - floor(y + 0.5) - 0.5;
    const int chan = (int)((row / a.rows_per_chan_blk) % a.n_chan);
    a.sin_out[row] = yw / a.dl[2 * chan + 1];
    if (a.peak_out) a.peak_out[row] = (float)p;
  }
}

}  // namespace

namespace {

template <int PER, int KMAX>
void launch_loc(const LocArgs& a, bool vec, unsigned nb, hipStream_t s) {
  if constexpr (PER >= 4) {
    if (vec) {
      hipLaunchKernelGGL((k_localize<PER, true, KMAX>), dim3(nb), dim3(256), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((k_localize<PER, false, KMAX>), dim3(nb), dim3(256), 0, s, a);
}

template <int KMAX>
hipError_t launch_loc_k(const LocArgs& a, unsigned nb, hipStream_t s) {
  const bool vec = (reinterpret_cast<uintptr_t>(a.in) % 16) == 0;
  switch (a.m) {
    case 32:
    case 64: launch_loc<1, KMAX>(a, vec, nb, s); break;
    case 128: launch_loc<2, KMAX>(a, vec, nb, s); break;
    case 256: launch_loc<4, KMAX>(a, vec, nb, s); break;
    case 512: launch_loc<8, KMAX>(a, vec, nb, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_localize(const LocArgs& a, hipStream_t s) {
  if (a.n_rows <= 0) return hipSuccess;
  if (a.m != 2 * a.n || a.n_window < 1 || a.n_window > 64 || a.n_window > a.m) return hipErrorInvalidValue;
  const int64_t nb = (a.n_rows + 255) / 256;      // 64 rows per wavefront, 4 wavefronts per workgroup
  if (nb > 0x7FFFFFFF) return hipErrorInvalidConfiguration;
  return a.n_window <= 16 ? launch_loc_k<16>(a, (unsigned)nb, s) : launch_loc_k<64>(a, (unsigned)nb, s);
}

}  // namespace fftbf
