// FFT-beam intensities through redundancy-stacked visibilities (gfx950).
//
// For a transform zero-padded to M >= 2n - 1 the block-summed intensity of
// N-S beam A of one E-W beam is the Fourier transform of the stacked
// visibilities (eq. e:b_V_delta and its inverse e:inv_b2n-1):
//   sum_t |B_A[t]|^2 = (1/n) sum_{|d| < n} R_d e^{-i 2 pi A d / M},
//   R_d = sum_t sum_a x_{a+d}[t] x_a^*[t],
// x the E-W transform of the voltages.  Unwindowed x are small integers, so
// the R_d are formed exactly (int8 products, int32 sums) on the matrix cores,
// and the Fourier transform runs once per block instead of once per sample.
// It runs in FP64: a weak beam beside a strong source is a small difference
// of large R_d, which FP32 would lose.
//
// Split of the matrix products.  With a = 64 w + 16 q + 4 c + g (row 4 g + q
// of an operand) and a' = 16 U + 4 c + n (column n), the 16 x 16 tile of
// U = j + 4 w, summed over w, c and the 16 samples (K), holds the lag
// a' - a = 16 (j - q) + n - g at (4 g + q, n): the four rows q of a lane
// belong to whole 16-lag steps, so the tiles j add up in registers with no
// movement between lanes, and only the four lane groups g meet in LDS.
// (With 16 consecutive antennas as rows every register would need a rotation
// and a select: 224 instead of 104 additions per block and E-W beam.)  10 of
// 16 (j, w) pairs exist: 160 products of 16 x 16 x 64 per 16 samples of one
// E-W beam at n = 256, 136 without the tiles' empty corners.
//
// Per 16 samples of a 4 x 256 lattice and polarisation: 640 matrix products
// (16 cycles each), 159 other vector instructions per sample against 836 of
// an FP32 transform per sample.  MI355X, 4 x 256, 2 polarisations, 256
// channels, 16384 samples, 16-sample blocks, 256 of 512 beams kept:
// 10.0 -> 6.9 ms (FP32 transform per sample -> this); FP16 matrix cores per
// sample 9.1 ms.  4 x 128 (8192 samples) 2.13 -> 1.37, 4 x 64 2.03 -> 1.25,
// 4 x 32 0.93 -> 0.64, 4 x 16 0.53 -> 0.37 ms (256 channels, 2
// polarisations; matrix cores per sample at 4 x 16: FP16 0.38, FP8 0.50 ms).
// Bound at n = 256: 640 cycles of products and 636 of vector issue a frame would
// be 5.0 ms one strictly after the other at the 2.1 GHz that the clock holds on
// random voltages.  The rest is waiting (37 % of the wavefronts' cycles): two
// barriers bracket each step and two workgroups share a CU.  Variants with 25 %
// fewer vector instructions, with two to four wavefronts per SIMD, with half the
// LDS reads or with reads issued ahead all run within 3 % of each other.
#include <type_traits>

#include "dev_bytes.h"
#include "dev_common.h"
#include "kernels.h"

namespace fftbf {

namespace {

struct cd {
  double r, i;
};
__device__ __forceinline__ cd dadd(cd a, cd b) { return {a.r + b.r, a.i + b.i}; }
__device__ __forceinline__ cd dsub(cd a, cd b) { return {a.r - b.r, a.i - b.i}; }
__device__ __forceinline__ cd dmul(cd a, double2 w) {
  return {fma(a.r, w.x, -(a.i * w.y)), fma(a.r, w.y, a.i * w.x)};
}
// a - i b and a + i b
__device__ __forceinline__ cd dsubi(cd a, cd b) { return {a.r + b.i, a.i - b.r}; }
__device__ __forceinline__ cd daddi(cd a, cd b) { return {a.r - b.i, a.i + b.r}; }

__device__ __forceinline__ void dft2(cd* x) {
  const cd a = x[0], b = x[1];
  x[0] = dadd(a, b);
  x[1] = dsub(a, b);
}
__device__ __forceinline__ void dft4(cd* x) {
  const cd s02 = dadd(x[0], x[2]), d02 = dsub(x[0], x[2]), s13 = dadd(x[1], x[3]), d13 = dsub(x[1], x[3]);
  x[0] = dadd(s02, s13);
  x[1] = dsubi(d02, d13);
  x[2] = dsub(s02, s13);
  x[3] = daddi(d02, d13);
}
__device__ __forceinline__ void dft8(cd* x) {
  constexpr double k = 0.70710678118654752440;
  cd e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
  dft4(e);
  dft4(o);
  x[0] = dadd(e[0], o[0]);
  x[4] = dsub(e[0], o[0]);
  x[2] = dsubi(e[2], o[2]);
  x[6] = daddi(e[2], o[2]);
  const cd p{o[1].r + o[1].i, o[1].i - o[1].r};      // sqrt(2) W_8 o_1
  x[1] = cd{fma(k, p.r, e[1].r), fma(k, p.i, e[1].i)};
  x[5] = cd{fma(-k, p.r, e[1].r), fma(-k, p.i, e[1].i)};
  const cd q{o[3].i - o[3].r, -o[3].i - o[3].r};     // sqrt(2) W_8^3 o_3
  x[3] = cd{fma(k, q.r, e[3].r), fma(k, q.i, e[3].i)};
  x[7] = cd{fma(-k, q.r, e[3].r), fma(-k, q.i, e[3].i)};
}
template <int R>
__device__ __forceinline__ void dft_n(cd* x) {
  if constexpr (R == 8) dft8(x);
  else if constexpr (R == 4) dft4(x);
  else if constexpr (R == 2) dft2(x);
}

// E-W 4-point transform of four samples of one N-S position (dwords w0 .. w3:
// byte q holds antenna q, real part in its high nibble), four samples per
// register: y[2 e + part], byte t = sample t, int8.  A byte lane of a word
// holds a digit of sum_t d_t 256^t; sums and differences of such words are
// exact as long as the digits end in [0, 255], so the digits carry a bias,
// 128 at the end, where flipping the top bit leaves the signed byte.
__device__ __forceinline__ void ew_transform4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t* y) {
  uint32_t q[4];
  transpose_bytes(w0, w1, w2, w3, q);
  constexpr uint32_t kM = 0x0F0F0F0Fu, kB = 0x08080808u;
  uint32_t s02p[2], s02m[2], s13[2], d02[2], d13[2];
#pragma unroll
  for (int part = 0; part < 2; ++part) {          // 0 real (high nibbles), 1 imaginary
    uint32_t n[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) n[k] = part ? q[k] : q[k] >> 4;
    const uint32_t x1 = (n[1] & kM) ^ kB, x2 = (n[2] & kM) ^ kB, x3 = (n[3] & kM) ^ kB;   // value + 8
    const uint32_t x0a = (n[0] & kM) ^ 0x68686868u;     // value + 104
    const uint32_t x0b = (n[0] & kM) ^ 0x88888888u;     // value + 136
    s02p[part] = x0a + x2;       // bias 112
    s02m[part] = x0b + x2;       // bias 144
    d02[part] = x0b - x2;        // bias 128
    s13[part] = x1 + x3;         // bias 16
    d13[part] = x1 - x3;         // bias 0
  }
  constexpr uint32_t kT = 0x80808080u;
  y[0] = (s02p[0] + s13[0]) ^ kT;
  y[1] = (s02p[1] + s13[1]) ^ kT;
  y[2] = (d02[0] + d13[1]) ^ kT;      // x_0 - i x_1 - x_2 + i x_3
  y[3] = (d02[1] - d13[0]) ^ kT;
  y[4] = (s02m[0] - s13[0]) ^ kT;
  y[5] = (s02m[1] - s13[1]) ^ kT;
  y[6] = (d02[0] - d13[1]) ^ kT;
  y[7] = (d02[1] + d13[0]) ^ kT;
}

// A task's voltage count n_ns x samples below which every R_d, and the sum of
// two, fits int32 whatever the voltages are: |x|^2 <= 2 * 32^2 per antenna
// and sample, so 2 * 2^11 * count <= 2^31.
constexpr int kLagLimit = 1 << 19;

// One workgroup: four wavefronts, wavefront e owns E-W beam e.  256 / N tasks
// (block, channel, polarisation group) at a time, two rounds per output.
template <int N, bool LONG, bool SPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_lag(LagArgs p) {
  using sum_t = typename std::conditional<LONG, double, int>::type;
  constexpr int M = 2 * N;
  constexpr int G = 256 / N;                 // tasks side by side
  constexpr int NB = N / 16;                 // blocks of 16 antennas
  constexpr int W = N >= 64 ? N / 64 : 1;    // row blocks
  constexpr int RC = NB < 4 ? NB : 4;
  constexpr int GS = N <= 32 ? 4 : 1;        // tasks per guarded step of the matrix-core loop
  constexpr int PL = M / 8;                  // lanes per transform
  constexpr int R3 = M >= 64 ? M / 64 : 1;   // radix of the last pass
  constexpr int NTW = lag_tw_count(M);

  // [e][th][task, antenna]: 16 bytes, samples 8 th .. 8 th + 7 of one antenna
  // (real parts, then imaginary parts); the last entry stays zero
  __shared__ v4i lds_x[4 * 2 * 256 + 1];
  __shared__ double2 lds_tw[NTW];

  const int tid = threadIdx.x, lane = tid & 63;
  const int e = __builtin_amdgcn_readfirstlane(tid >> 6);
  // slot `sub` of the G side by side: steps sub_q, sub_q + parts, ... of task sub_t
  const int parts = SPLIT ? p.parts : 1;
  const int sub = G == 1 ? 0 : tid / N, a = tid % N;
  const int sub_t = SPLIT ? sub / parts : sub, sub_q = SPLIT ? sub - sub_t * parts : 0;
  v4i* const plane = lds_x + e * 512;        // read by wavefront e only

  for (int i = tid; i < NTW; i += 256) lds_tw[i] = p.tw[i];
  if (tid == 0) lds_x[2048] = v4i{0, 0, 0, 0};

  const int n_chunk = (p.block + 15) / 16;
  const int n_all = n_chunk * p.pol_iter, n_step = (n_all + parts - 1) / parts;
  const int64_t frame = (int64_t)p.n_chan * p.n_pol * N;     // dwords per sample
  const uint32_t n_task = (uint32_t)p.n_task, per_unit = p.tpi * p.iters;
  const uint32_t n_unit = (n_task + per_unit - 1) / per_unit;

  // The 16 samples of one step, this thread's antenna.  Every load is
  // unconditional, so the next step's stay in flight during the matrix-core
  // work: threads without a task and samples past the block re-read valid
  // memory, and mask_step clears them.
  struct Raw {
    uint32_t v[16];
  };
  auto load = [&](uint32_t unit, int it, int step) {
    Raw w;
    uint32_t task = unit * per_unit + it * p.tpi + sub_t;
    if (task >= n_task || sub_t >= p.tpi) task = 0;
    step = step * parts + sub_q;
    if (SPLIT && step >= n_all) step = 0;
    const uint32_t pg = p.n_pg == 2 ? task & 1 : 0, rest = p.n_pg == 2 ? task >> 1 : task;
    const uint32_t blk = rest / (uint32_t)p.n_chan, chan = rest - blk * p.n_chan;
    const int pi = step >= n_chunk;          // at most two polarisations
    const int t0 = (step - pi * n_chunk) * 16, nt = p.block - t0;
    const uint32_t* src = p.volts + ((int64_t)blk * p.block + t0) * frame + ((int64_t)chan * p.n_pol + pg + pi) * N;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      w.v[t] = __builtin_nontemporal_load(src + a);
      if (t + 1 < nt) src += frame;
    }
    return w;
  };
  auto mask_step = [&](uint32_t unit, int it, int step, Raw w) {
    const uint32_t task = unit * per_unit + it * p.tpi + sub_t;
    step = step * parts + sub_q;
    const int pi = step >= n_chunk, nt = p.block - (step - pi * n_chunk) * 16;
    if (SPLIT || nt < 16 || p.tpi < G || (unit + 1) * per_unit > n_task) {
      const uint32_t live = (sub_t < p.tpi && task < n_task && step < n_all) ? ~0u : 0u;
#pragma unroll
      for (int t = 0; t < 16; ++t) w.v[t] &= t < nt ? live : 0u;
    }
    return w;
  };

  // operand addresses (16-byte units) of this lane.  Rows: antenna
  // 64 w + 16 q + 4 c + g of row 4 g + q; columns: antenna 16 U + 4 c + n of
  // column n; K group l / 16 = (c & 1, th), c = 2 k2 + (c & 1)
  const int ln = lane & 15, th = (lane >> 4) & 1, kk = lane >> 5;
  const int row0 = e * 512 + th * 256 + 16 * ((ln & 3) & (NB - 1)) + 4 * kk + (ln >> 2);
  const int col0 = e * 512 + th * 256 + 4 * kk + ln;

  uint32_t unit = blockIdx.x;
  Raw w = load(unit < n_unit ? unit : 0, 0, 0);
  for (; unit < n_unit; unit += gridDim.x) {
    sum_t rs[2][4], v[2][4];                 // R_d (real, imaginary parts) of the first round and of this one
    sum_t* const own = reinterpret_cast<sum_t*>(plane);
    for (int it = 0; it < p.iters; ++it) {
      int acc[2][16];
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[0][i] = acc[1][i] = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[0][k] = v[1][k] = 0;

      // R_d summed so far into v: the four lane groups meet in LDS.  Lane
      // (g, n) holds lag 16 m + n - g of task s in acc[s NB + m].
      auto gather = [&]() {
        wave_sync();
        int rl = lane;
        asm volatile("" : "+v"(rl));           // the addresses are formed here, not held through the loops
        int* const area = reinterpret_cast<int*>(plane);
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            area[part * 1024 + (rl >> 4) * 256 + 16 * i + (rl & 15)] = acc[part][i];
            if (LONG) acc[part][i] = 0;
          }
        wave_sync();
        constexpr int NM = N < 64 ? N : 64;
        const int left = NM - rl % NM;          // lags from this one to the end of 64, or of the task
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int* const at = area + rl + (part * 1024 + 64 * k);
            int sum = at[0];
#pragma unroll
            for (int g = 1; g < 4; ++g) {
              int x = at[g * 257];               // lag d of group g: column d + g
              if ((64 * (k + 1)) % N == 0 && g >= left) x = 0;
              sum += x;
            }
            v[part][k] += sum;
          }
        wave_sync();
      };

      for (int step = 0; step < n_step; ++step) {
        w = mask_step(unit, it, step, w);
        __syncthreads();           // the previous step's operands are no longer read
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          uint32_t y0[8], y1[8];
          ew_transform4(w.v[8 * h], w.v[8 * h + 1], w.v[8 * h + 2], w.v[8 * h + 3], y0);
          ew_transform4(w.v[8 * h + 4], w.v[8 * h + 5], w.v[8 * h + 6], w.v[8 * h + 7], y1);
#pragma unroll
          for (int b = 0; b < 4; ++b)
            lds_x[b * 512 + h * 256 + tid] = v4i{(int)y0[2 * b], (int)y1[2 * b], (int)y0[2 * b + 1], (int)y1[2 * b + 1]};
        }
        {
          // the next step's samples, in flight during the matrix-core work
          int ns = step + 1, ni = it;
          uint32_t nu = unit;
          if (ns == n_step) {
            ns = 0;
            if (++ni == p.iters) {
              ni = 0;
              nu += gridDim.x;
            }
          }
          w = load(nu < n_unit ? nu : unit, ni, ns);
        }
        __syncthreads();

        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int s0 = 0; s0 < G; s0 += GS) {
          if (s0 >= p.tpi * parts) break;
#pragma unroll
          for (int s = s0; s < s0 + GS; ++s) {
            // rows for the real parts [x_r, x_i] and the imaginary parts [-x_i, x_r]
            v4i ar[W][2], ai[W][2];
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
              for (int ww = 0; ww < W; ++ww) {
                const v4i v = lds_x[row0 + s * N + 64 * ww + 8 * k2];
                ar[ww][k2] = v;
                ai[ww][k2] = v4i{neg_bytes(v[2]), neg_bytes(v[3]), v[0], v[1]};
              }
#pragma unroll
            for (int r = 0; r < RC; ++r) {
              // columns U = r + 4 u, the last first: each column pair meets
              // the row blocks w <= u, tile j = r + 4 (u - w)
              v4i cr[W], ci[W];
#pragma unroll
              for (int dj = 0; dj < W; ++dj) cr[dj] = ci[dj] = v4i{0, 0, 0, 0};
#pragma unroll
              for (int u = W - 1; u >= 0; --u) {
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2) {
                  int ad = col0 + s * N + 16 * (r + 4 * u) + 8 * k2;
                  if (r + 4 * u == NB - 1 && 4 * kk + 8 * k2 + ln >= 16) ad = 2048;
                  const v4i b = lds_x[ad];
#pragma unroll
                  for (int ww = 0; ww <= u; ++ww) {
                    cr[u - ww] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[ww][k2], b, cr[u - ww], 0, 0, 0);
                    ci[u - ww] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ai[ww][k2], b, ci[u - ww], 0, 0, 0);
                  }
                }
                const int j = r + 4 * u;               // tile j is complete
#pragma unroll
                for (int q = 0; q < RC; ++q)
                  if (j >= q) {
                    acc[0][s * NB + j - q] += cr[u][q];
                    acc[1][s * NB + j - q] += ci[u][q];
                  }
              }
            }
          }
        }
        __builtin_amdgcn_s_setprio(0);
        if (LONG && (step + 1) % (kLagLimit / (16 * N)) == 0) gather();
      }
      gather();
      if (it == 0 && p.iters == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          rs[0][k] = v[0][k];
          rs[1][k] = v[1][k];
        }
      } else {
        // both rounds' R_d: [round][part][task, d]
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            own[part * 256 + lane + 64 * k] = p.iters == 2 ? rs[part][k] : v[part][k];
            own[512 + part * 256 + lane + 64 * k] = p.iters == 2 ? v[part][k] : 0;
          }
      }
    }
    wave_sync();
    if constexpr (SPLIT) {
      // the slots of a task become one
      for (int k = lane; k < 4 * p.tpi * N; k += 64) {
        const int arr = k / (p.tpi * N), r = k - arr * (p.tpi * N), t = r / N;
        sum_t* const at = own + arr * 256 + r % N;
        sum_t sum = at[t * parts * N];
        for (int q = 1; q < parts; ++q) sum += at[(t * parts + q) * N];
        wave_sync();                       // no slot is written before the lanes of this turn have read theirs
        at[t * N] = sum;
      }
      wave_sync();
    }

    // ---- M-point transforms, the two rounds' tasks as one complex series ----
    int fl_lane = lane;
    asm volatile("" : "+v"(fl_lane));      // the addresses below are formed here, not held through the loops
    const int ps = fl_lane / PL, l = fl_lane % PL;
    cd z[8];
    // Rounding leaks about 2^-53 of one task's sums into the other's.  So that
    // it stays that small beside the other's own, tasks whose R_0 differ by
    // more than 2^8 are brought to the same size first (exactly, by 2^sh); a
    // task without signal (R_0 = 0) is zero, its rounding noise is not stored.
    float norm1, norm2;
    {
      sum_t p1 = own[ps * N], p2 = own[512 + ps * N];
      sum_t ur[8], ui[8], vr[8], vi[8];
      const sum_t* const up = own + ps * N + l;
      const sum_t* const down = own + ps * N - l;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const sum_t* const r = i < 4 ? up + PL * i : down + PL * (8 - i);
        ur[i] = r[0];
        ui[i] = r[256];
        vr[i] = r[512];
        vi[i] = r[768];
      }
      int sh;
      if constexpr (LONG) {
        sh = __builtin_amdgcn_frexp_exp(p1) - __builtin_amdgcn_frexp_exp(p2);
      } else {
        if constexpr (PL == 64) {            // one task a wavefront: on the scalar unit
          p1 = __builtin_amdgcn_readfirstlane(p1);
          p2 = __builtin_amdgcn_readfirstlane(p2);
        }
        sh = __builtin_clz(p2 | 1) - __builtin_clz(p1 | 1);
      }
      if (p1 == 0 || p2 == 0 || (sh >= -8 && sh <= 8)) sh = 0;
      norm1 = p1 != 0 ? p.norm : 0.f;
      norm2 = p2 != 0 ? p.norm : 0.f;
      if (!__any(sh != 0)) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          z[i] = i < 4 ? cd{(double)(ur[i] - vi[i]), (double)(ui[i] + vr[i])} : cd{(double)(ur[i] + vi[i]), (double)(vr[i] - ui[i])};
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const double a = (double)ur[i], b = (double)ui[i], c = ldexp((double)vr[i], sh), d = ldexp((double)vi[i], sh);
          z[i] = i < 4 ? cd{a - d, b + c} : cd{a + d, c - b};
        }
        norm2 = ldexpf(norm2, -sh);
      }
      if (l == 0) z[4] = cd{0.0, 0.0};                   // lag N: not formed
    }
    wave_sync();
    double2* const ex = reinterpret_cast<double2*>(plane);
    dft8(z);
#pragma unroll
    for (int r = 1; r < 8; ++r) z[r] = dmul(z[r], lds_tw[(r - 1) * PL + l]);
    float v1[8], v2[8];
    if constexpr (M >= 64) {
      // lane (r, l0) takes l = l0 + R3 l1
      constexpr int SW = 16 / R3 < 8 ? 16 / R3 - 1 : 7;
      const int r = l / R3, l0 = l % R3;
#pragma unroll
      for (int k = 0; k < 8; ++k) ex[ps * M + k * PL + (l ^ (R3 * (k & SW)))] = make_double2(z[k].r, z[k].i);
      wave_sync();
#pragma unroll
      for (int l1 = 0; l1 < 8; ++l1) {
        const double2 v = ex[ps * M + r * PL + l0 + R3 * ((l1 & SW) ^ (r & SW)) + R3 * (l1 & ~SW)];
        z[l1] = cd{v.x, v.y};
      }
      wave_sync();
      dft8(z);
      if constexpr (R3 > 1) {
#pragma unroll
        for (int r2 = 1; r2 < 8; ++r2) z[r2] = dmul(z[r2], lds_tw[7 * PL + (r2 - 1) * R3 + l0]);
        constexpr int F2 = 16 / R3;
#pragma unroll
        for (int r2 = 0; r2 < 8; ++r2)
          ex[ps * M + l0 * 64 + (r ^ ((F2 * l0) & 7)) + 8 * ((r2 & 1) ^ ((F2 * l0) >> 3)) + 16 * (r2 >> 1)] =
              make_double2(z[r2].r, z[r2].i);
        wave_sync();
#pragma unroll
        for (int s = 0; s < 8 / R3; ++s)
#pragma unroll
          for (int k = 0; k < R3; ++k) {
            const double2 v = ex[ps * M + k * 64 + (l ^ (F2 * k)) + PL * s];
            z[s * R3 + k] = cd{v.x, v.y};
          }
        wave_sync();
#pragma unroll
        for (int s = 0; s < 8 / R3; ++s) dft_n<R3>(z + s * R3);
      }
    } else {
#pragma unroll
      for (int r = 0; r < 8; ++r) ex[ps * M + r * 4 + l] = make_double2(z[r].r, z[r].i);
      wave_sync();
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const double2 v = ex[ps * M + (l + 4 * (k / 4)) * 4 + (k % 4)];
        z[k] = cd{v.x, v.y};
      }
      wave_sync();
      dft4(z);
      dft4(z + 4);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      v1[k] = fmaxf((float)z[k].r * norm1, 0.f);
      v2[k] = fmaxf((float)z[k].i * norm2, 0.f);
    }
    // value i of the lane: N-S beam beam(i) of this lane's series
    auto beam = [&](int i) {
      if constexpr (M >= 128) return l + PL * (i / R3) + 64 * (i % R3);
      else if constexpr (M == 64) return l + 8 * i;
      else return (l + 4 * (i / 4)) + 8 * (i % 4);
    };
    float* fl = reinterpret_cast<float*>(own);
    if (p.sel) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        fl[ps * M + beam(i)] = v1[i];
        fl[512 + ps * M + beam(i)] = v2[i];
      }
      wave_sync();
    }
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      if (it >= p.iters) break;
      const uint32_t task = unit * per_unit + it * p.tpi + ps;
      if (ps >= p.tpi || task >= n_task) continue;
      float* const o = p.out + ((int64_t)task * 4 + e) * p.n_keep;
      if (p.sel) {
        const uint32_t chan = (p.n_pg == 2 ? task >> 1 : task) % (uint32_t)p.n_chan;
        const int32_t* const sel = p.sel + (int64_t)chan * p.n_keep;
        for (int j0 = l; j0 < p.n_keep; j0 += 4 * PL) {
          int A[4];                              // four table entries in flight
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int j = j0 + PL * k;
            A[k] = sel[j < p.n_keep ? j : j0];
          }
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (j0 + PL * k < p.n_keep) o[j0 + PL * k] = fl[it * 512 + ps * M + A[k]];
        }
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) o[beam(i)] = it ? v2[i] : v1[i];
      }
    }
    wave_sync();
  }
}

// W_M^{r l} for r = 1..7, l < M/8, then W_{M/8}^{r l0} for r = 1..7, l0 < M/64
__global__ void k_lag_tw(double2* tw, int m) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int n1 = 7 * (m / 8), r3 = m / 64;
  if (i >= lag_tw_count(m)) return;
  int k, mm;
  if (i < n1) {
    mm = m;
    k = (i / (m / 8) + 1) * (i % (m / 8)) % mm;
  } else {
    mm = m / 8;
    k = ((i - n1) / r3 + 1) * ((i - n1) % r3) % mm;
  }
  double s, c;
  sincospi(-2.0 * (double)k / (double)mm, &s, &c);
  tw[i] = make_double2(c, s);
}

template <int N>
void launch_n(LagArgs a, hipStream_t s) {
  constexpr int G = 256 / N;
  constexpr int kWgs = 512;                 // two workgroups per compute unit
  // few tasks: fewer per workgroup, so that they spread over the chip, and a
  // second round only if one does not hold them
  const int64_t per = (a.n_task + kWgs - 1) / kWgs;
  a.iters = per > G ? 2 : 1;
  const int64_t tpi = (per + a.iters - 1) / a.iters;
  a.tpi = tpi < G ? (int)tpi : G;
  // slots left over take every parts-th step of 16 samples each (SPLIT): one
  // block of 1600 samples 141 -> 24 us at 4 x 16, 1.34 -> 0.13 ms at 4 x 128
  // against one wavefront's transforms; 225 channels of 48 samples and two
  // polarisations at 4 x 16 took 14.5 us with a slot each and 11.6 before
  const int n_all = (a.block + 15) / 16 * a.pol_iter;
  a.parts = G / a.tpi < n_all ? G / a.tpi : n_all;
  const int64_t pu = (int64_t)a.tpi * a.iters;
  const int64_t n_unit = (a.n_task + pu - 1) / pu;
  const dim3 grid((unsigned)(n_unit < kWgs ? n_unit : kWgs)), threads(256);
  const bool fits = (int64_t)N * a.block * a.pol_iter < kLagLimit;
  if constexpr (G > 1) {
    if (a.parts > 1) {
      if (fits) hipLaunchKernelGGL((k_lag<N, false, true>), grid, threads, 0, s, a);
      else hipLaunchKernelGGL((k_lag<N, true, true>), grid, threads, 0, s, a);
      return;
    }
  }
  if (fits) hipLaunchKernelGGL((k_lag<N, false, false>), grid, threads, 0, s, a);
  else hipLaunchKernelGGL((k_lag<N, true, false>), grid, threads, 0, s, a);
}

}  // namespace

size_t lag_table_bytes(int n_ns) { return sizeof(double2) * lag_tw_count(2 * n_ns); }

hipError_t launch_lag_table(double2* tw, int n_ns, hipStream_t s) {
  const int n = lag_tw_count(2 * n_ns);
  hipLaunchKernelGGL(k_lag_tw, dim3((n + 255) / 256), dim3(256), 0, s, tw, 2 * n_ns);
  return hipGetLastError();
}

hipError_t launch_lag(const LagArgs& a, int n_ns, hipStream_t s) {
  switch (n_ns) {
    case 16: launch_n<16>(a, s); break;
    case 32: launch_n<32>(a, s); break;
    case 64: launch_n<64>(a, s); break;
    case 128: launch_n<128>(a, s); break;
    case 256: launch_n<256>(a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace fftbf
