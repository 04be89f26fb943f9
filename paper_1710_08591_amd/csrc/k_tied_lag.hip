// Tied-array beam intensities of the 4 x 16 lattice from 2-D stacked
// visibilities (gfx950): beams straight from voltages, and the server's tiles.
//
// The block-summed intensity of the pointed beam of eq. e:c_pointed is a
// linear map of the stacked visibilities (eq. e:b_V_delta on both axes):
//   sum_t |B_p[t]|^2 = (1/n) sum_d R_d e^{-i 2 pi d . y_p},
//   R_d = sum_t sum_a x_{a+d}[t] x_a^*[t],   d = (dx, dy), |dx| < 4, |dy| < 16,
// with y_p = (d/lambda) n_p per axis: the paper's intensity regridding
// carried to the visibilities.  Unwindowed x are int4, so the R_d are exact
// integers (int8 products, int32 sums on the matrix cores), formed once per
// block and shared by every pointing; the half plane dy >= 0 holds them all
// (R_-d = R_d^*).  Per pointing and block that leaves 217 real products
// instead of 128 complex ones per sample.
//
// The contraction R x weights runs on the int8 matrix cores as well, without
// rounding: R_d in three signed base-256 digits, the weights (FP64, rounded
// to a step of 2^-29) in four, products by digit pair summed in int32 and
// joined in FP64.  A weak beam beside a strong source is a small difference
// of large terms, which FP32 sums would lose; the weakest take a second set of
// weight digits, to 2^-60 (see kWeak).  (FP64 matrix products measured
// 112 cycles per 16 x 16 x 4, seven times the digit products' time.)
//
// Work of one 32-block table on a SIMD: eight blocks' R_d, each 16 matrix
// products and about 150 other vector instructions, once per wavefront its 16
// pointings' weights (640 instructions, FP64), and per 16 blocks x 16
// pointings 48 matrix products; three wavefronts per SIMD.  MI355X, 64
// pointings, 256 channels, 16384 samples: 818 -> 162 us against interpolating
// FFT beams per sample on the FP16 matrix cores (bound by those: 48 products
// per 16 samples x 16 pointings).  Bound now by vector issue in the R_d of
// each block; the voltages and outputs alone take 67 us at the copy rate.
// The server's tiles: 24 requests of up to 256 pointings, 65536 samples and
// 256 channels in one burst 7.58 -> 2.10 ms.
#include "dev_bytes.h"
#include "dev_common.h"
#include "kernels.h"

namespace fftbf {

namespace {

constexpr int kLagChunk = 32;              // blocks of one R_d table in LDS
constexpr int kLagPitch = 272;             // bytes of one block's digits: 256, and 16 against bank conflicts
constexpr int kLagPlane = 576;             // bytes of one E-W antenna's operands: 512, a zero entry, pad
constexpr int kLagScratch = 4 * kLagPlane + 7 * 4 * 16 * 8;   // per wavefront: operands, then the R_d of its lane groups
constexpr int kLagLds = 4 * kLagScratch + 3 * kLagChunk * kLagPitch + 64 * 4;
// samples (times polarisations summed) whose R_d, at most 64 * 128 per
// sample, fit three signed digits; longer blocks go in segments
constexpr int kLagSegment = 512;

struct cplx {
  double r, i;
};
__device__ __forceinline__ cplx zmul(cplx a, cplx b) {
  return {fma(a.r, b.r, -(a.i * b.i)), fma(a.r, b.i, a.i * b.r)};
}

// 16 consecutive samples' frames: sample r at base + r frame_dw, those from
// row `wrap` on `back` dwords before that (the end of a ring)
struct Group {
  const uint32_t* base;
  int wrap;
  int64_t back;
};

// The weights' step leaves an absolute error of up to 1e-10 of R_0 (a coherent
// source's peak), 3e-11 in the mean.  Where a tile has outputs below 2^-13 of
// their R_0, these are formed again with a second set of digits that holds what
// the step left out: 1e-16 of R_0.  Noise beside a source that fills the voltages stays above
// 2^-12.1 (25 million outputs of blocks of 16 samples), so data with noise do
// not pay for it beyond the comparison (64 pointings, 256 channels, 16384 samples
// 159 -> 162 us); without noise the same call takes 496 us (818 by FFT beams per
// sample).
// (The pass for these outputs spills: 160 to 200 bytes a lane.  The ordinary pass
// keeps to its registers.)
constexpr float kWeak = 0x1p-13f;
constexpr double kLowUnit = 2147483648.0;  // 2^31

// Weight digits of one pointing (lane column p = l % 16, lane group g = l / 16):
// byte 64 c + 16 g + 4 i + j of the K axis is, of the lag kappa = 16 c + 4 g + i
// (dx = c - 3, dy = 4 g + i) and of kappa + 64 (dx = c + 1), the real part
// (j = 0, 2) or the imaginary part (j = 1, 3).  LOW: what rounding to a step of
// 2^-29 leaves of the weights, to a step of 2^-60.
template <bool LOW>
__device__ __forceinline__ void lag_weights(double y_ew, double y_ns, int g, v4i (&w)[4][4]) {
  cplx zx[4], ay[4];
  zx[0] = {1.0, 0.0};
  sincospi(2.0 * y_ew, &zx[1].i, &zx[1].r);
  zx[2] = zmul(zx[1], zx[1]);
  zx[3] = zmul(zx[2], zx[1]);
  cplx z1;
  sincospi(2.0 * y_ns, &z1.i, &z1.r);
  const cplx z2 = zmul(z1, z1), z4 = zmul(z2, z2), z8 = zmul(z4, z4);
  ay[0] = {1.0, 0.0};
  if (g & 1) ay[0] = z4;
  if (g & 2) ay[0] = zmul(ay[0], z8);
#pragma unroll
  for (int i = 1; i < 4; ++i) ay[i] = zmul(ay[i - 1], z1);

  constexpr double kUnit = 536870912.0, kRound = 6755399441055744.0;   // 2^29; 1.5 * 2^52: the sum's low word is the integer
  auto digits = [&](double v, double f) {
    double u = fma(v, f * kUnit, kRound);
    if constexpr (LOW) u = fma(fma(v, f * kUnit, kRound - u), kLowUnit, kRound);
    return signed_digits((int)(uint32_t)__builtin_bit_cast(uint64_t, u));
  };
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // a lag and its opposite are one term (twice its real part); dy = 0
      // holds both of each pair, so only dx >= 0 counts there
      const bool row0 = g == 0 && i == 0;
      cplx m = ay[i];
      if (c < 3) m = zmul(ay[i], cplx{zx[3 - c].r, -zx[3 - c].i});
      const double f = !row0 ? 2.0 : c < 3 ? 0.0 : 1.0;
      uint32_t y[4];
      y[0] = digits(m.r, f);
      y[1] = digits(m.i, f);
      y[2] = y[3] = signed_digits(0);
      if (c < 3) {
        const cplx q = zmul(ay[i], zx[c + 1]);
        y[2] = digits(q.r, 2.0);
        y[3] = digits(q.i, 2.0);
      }
      uint32_t d[4];
      transpose_bytes(y[0], y[1], y[2], y[3], d);
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j][c][i] = (int)d[j];
    }
}

// Intensities of up to 64 pointings (16 per wavefront) over n_blk blocks of
// 16 gpb samples, n_sum polarisations summed.  group(s, k): where the 16
// samples from sample s on (of the first block's start), polarisation k, lie.
// store(block, value) of this lane's pointing.  Returns whether any output is
// so weak that it needs the weights' low digits; FULL forms and stores those
// outputs, and no others (so none depends on its neighbours).
template <bool FULL, class Locate, class Store>
__device__ __forceinline__ bool tied_lag_pass(char* lds, int lane, int wave, int n_blk, int gpb, int n_sum, double y_ew,
                                              double y_ns, bool wave_live, int64_t frame_dw, Locate group, Store store) {
  char* const xs = lds + wave * kLagScratch;
  int2* const part = reinterpret_cast<int2*>(xs + 4 * kLagPlane);
  char* const rd = lds + 4 * kLagScratch;
  float* const undefined = reinterpret_cast<float*>(rd + 3 * kLagChunk * kLagPitch) + 16 * wave;   // added to the outputs
  const int ln = lane & 15, grp = lane >> 4;

  v4i w[4][4];
  if (!FULL && wave_live) lag_weights<false>(y_ew, y_ns, grp, w);
  bool weak = false;
  // the weights' digits hold no NaN: a direction that is not finite makes the
  // sums of its pointing mean nothing, and they are stored as NaN
  if (grp == 0) undefined[ln] = fabs(y_ew) < INFINITY && fabs(y_ns) < INFINITY ? 0.f : NAN;
  if (lane < 4) *reinterpret_cast<v4i*>(xs + lane * kLagPlane + 512) = v4i{0, 0, 0, 0};

  // Operands of 16 samples: [E-W antenna][th][N-S antenna] 16 bytes, samples
  // 8 th .. 8 th + 7 as (4 real, 4 imaginary) twice.  Rows: antenna
  // (ew = i, ns = 4 c + g) of row 4 g + i; columns: ns = 4 c + n of column n,
  // one E-W antenna at a time; K group l / 16 = (c & 1, th), c = 2 k2 + (c & 1).
  // Tile ew' then holds the lag (ew' - i, n - g) at (4 g + i, n).
  const int kk = lane >> 5, th = grp & 1;
  char* const put = xs + (grp >> 1) * 256 + ln * 16 + (grp & 1) * 8;    // this lane decodes samples 4 grp .. 4 grp + 3
  const char* const row = xs + (ln & 3) * kLagPlane + th * 256 + (4 * kk + (ln >> 2)) * 16;
  const char *col[2];
#pragma unroll
  for (int k2 = 0; k2 < 2; ++k2) {
    const int ns = 8 * k2 + 4 * kk + ln;
    col[k2] = xs + (ns < 16 ? th * 256 + ns * 16 : 512);
  }

  const int seg = kLagSegment / (16 * n_sum);        // groups per segment
  int64_t off[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) off[j] = (4 * grp + j) * frame_dw + ln;
  for (int c0 = 0; c0 < n_blk; c0 += kLagChunk) {
    const int nb = n_blk - c0 < kLagChunk ? n_blk - c0 : kLagChunk;
    float limit = 0.f;                     // 2^-13 R_0 of the table's block lane % 32
    double out[2][4], rest[2][4];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[rt][r] = rest[rt][r] = 0.0;
    for (int g0 = 0; g0 < gpb; g0 += seg) {
      const int ng = gpb - g0 < seg ? gpb - g0 : seg;
      const int n_item = ng * n_sum;
      // ---- R_d of the chunk's blocks, one wavefront per block ----
      auto load = [&](int b, int item, uint32_t (&d)[4]) {
        const int k = n_sum == 1 ? 0 : item / ng, gi = item - k * ng;
        const Group at = group((int64_t)(c0 + b) * gpb * 16 + (g0 + gi) * 16, k);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t* q = at.base + off[j];
          if (4 * grp + j >= at.wrap) q -= at.back;
          d[j] = *q;
        }
      };
      uint32_t d[4] = {0, 0, 0, 0};
      if (wave < nb) load(wave, 0, d);
      for (int b = wave; b < nb; b += 4) {
        v4i cr[4], ci[4];
        auto step = [&](int item, bool first) {
          uint32_t q4[4];
          transpose_bytes(d[0], d[1], d[2], d[3], q4);
          // the next samples, in flight during this group's work
          const int nb1 = item + 1 < n_item ? b : b + 4, ni = item + 1 < n_item ? item + 1 : 0;
          if (nb1 < nb) load(nb1, ni, d);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            // sign-extended nibbles times 8: the negative of -8 must fit too
            const uint32_t v = q4[q];
            const uint32_t re = ((v >> 1) & 0x78787878u) | (v & 0x80808080u);
            const uint32_t im = ((v << 3) & 0x78787878u) | ((v << 4) & 0x80808080u);
            *reinterpret_cast<uint2*>(put + q * kLagPlane) = make_uint2(re, im);
          }
          wave_sync();
#pragma unroll
          for (int k2 = 0; k2 < 2; ++k2) {
            const v4i rr = *reinterpret_cast<const v4i*>(row + k2 * 128);
            const v4i ri = v4i{neg_bytes(rr[1]), rr[0], neg_bytes(rr[3]), rr[2]};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const v4i cc = *reinterpret_cast<const v4i*>(col[k2] + q * kLagPlane);
              const v4i zero = {0, 0, 0, 0};
              cr[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(rr, cc, first && k2 == 0 ? zero : cr[q], 0, 0, 0);
              ci[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ri, cc, first && k2 == 0 ? zero : ci[q], 0, 0, 0);
            }
          }
          wave_sync();
        };
        step(0, true);
        for (int item = 1; item < n_item; ++item) step(item, false);
        // dx = ew' - i: registers of one lane; dy = n - g: the four lane groups meet in LDS
#pragma unroll
        for (int x = 0; x < 7; ++x) {
          int sr = 0, si = 0;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (q - (x - 3) >= 0 && q - (x - 3) < 4) {
              sr += cr[q][q - (x - 3)];
              si += ci[q][q - (x - 3)];
            }
          part[(x * 4 + grp) * 16 + ln] = make_int2(sr, si);
        }
        wave_sync();
        int v[4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int2* const at = part + (lane >> 4) * 64 + ln + 256 * h;
          int2 s = at[0];
#pragma unroll
          for (int g = 1; g < 4; ++g) {
            const int2 a = at[17 * g];
            s.x += ln + g < 16 ? a.x : 0;
            s.y += ln + g < 16 ? a.y : 0;
          }
          const bool ok = h == 0 || lane < 48;
          v[2 * h] = ok ? s.x >> 6 : 0;
          v[2 * h + 1] = ok ? s.y >> 6 : 0;
        }
        wave_sync();
        uint32_t dg[4];
        transpose_bytes(signed_digits(v[0]), signed_digits(v[1]), signed_digits(v[2]), signed_digits(v[3]), dg);
#pragma unroll
        for (int j = 0; j < 3; ++j)
          *reinterpret_cast<uint32_t*>(rd + (j * kLagChunk + b) * kLagPitch + 4 * lane) = dg[j];
      }
      __syncthreads();

      // ---- contraction with the weights: 16 blocks x 16 pointings ----
      auto contract = [&](double (&sum)[2][4]) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
          if (16 * rt >= nb) break;
          v4i s[6];
#pragma unroll
          for (int k = 0; k < 6; ++k) s[k] = v4i{0, 0, 0, 0};
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
              const v4i a = *reinterpret_cast<const v4i*>(rd + (i * kLagChunk + 16 * rt + ln) * kLagPitch + 64 * c + 16 * grp);
#pragma unroll
              for (int j = 0; j < 4; ++j) s[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, w[j][c], s[i + j], 0, 0, 0);
            }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            double t = (double)s[5][r];
#pragma unroll
            for (int k = 4; k >= 0; --k) t = fma(t, 256.0, (double)s[k][r]);
            sum[rt][r] += t;
          }
        }
      };
      if (wave_live) {
        const int8_t* const r0 = reinterpret_cast<const int8_t*>(rd) + (lane % kLagChunk) * kLagPitch + 4 * 48;
        constexpr int kPlane = kLagChunk * kLagPitch;
        limit = fmaf(kWeak, (float)(65536 * r0[2 * kPlane] + 256 * r0[kPlane] + r0[0]), limit);
        if (lane < kLagChunk) reinterpret_cast<float*>(xs)[lane] = limit;
        if constexpr (FULL) {
          asm volatile("" : "+v"(y_ew), "+v"(y_ns));     // made again here: what the two sets share is not held
          lag_weights<false>(y_ew, y_ns, grp, w);
        }
        contract(out);
        if constexpr (FULL) {
          asm volatile("" : "+v"(y_ew), "+v"(y_ns));
          lag_weights<true>(y_ew, y_ns, grp, w);
          contract(rest);
        }
      }
      __syncthreads();               // the R_d table may be overwritten
    }
    if (wave_live) {
      constexpr double kScale = 1.0 / (536870912.0 * 64.0);     // weight step, 1/n
      const float add = undefined[ln];
      float4 low[2];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) low[rt] = reinterpret_cast<const float4*>(xs)[4 * rt + grp];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        const float lim[4] = {low[rt].x, low[rt].y, low[rt].z, low[rt].w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int b = 16 * rt + 4 * grp + r;
          const float v = fmaxf((float)(out[rt][r] * kScale), 0.f);
          const bool low_one = b < nb && v < lim[r];
          if constexpr (FULL) {
            if (low_one) store(c0 + b, fmaxf((float)(fma(rest[rt][r], 1.0 / kLowUnit, out[rt][r]) * kScale), 0.f) + add);
          } else {
            weak |= low_one;
            if (b < nb) store(c0 + b, v + add);
          }
        }
      }
    }
  }
  return weak;
}

// One workgroup per (64 pointings, run of blocks, channel, polarisation group).
template <bool FULL>
__device__ __forceinline__ bool tied_lag_run(const TiedArgs& a, char* lds) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));        // nothing of one pass is held (spilled) for the other
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_ptile = (a.n_point + 63) / 64;
  const int n_pg = a.pol_sum ? 1 : a.n_pol;
  const int ptile = blockIdx.x % n_ptile, run = blockIdx.x / n_ptile;
  const int cs = blockIdx.y, pg = blockIdx.z, chan = a.chan_lo + cs;
  const int p0 = ptile * 64 + wave * 16, p = p0 + (tid & 15);
  const int pp = p < a.n_point ? p : a.n_point - 1;
  const int64_t n_blk = a.n_time / a.block, b0 = (int64_t)run * a.run_units;
  const int nb = (int)(n_blk - b0 < a.run_units ? n_blk - b0 : a.run_units);
  const int64_t frame_dw = (int64_t)a.n_chan * a.n_pol * 16;
  const uint32_t* const src = a.volts + b0 * a.block * frame_dw + ((int64_t)chan * a.n_pol + pg) * 16;
  float* const out = static_cast<float*>(a.out);
  return tied_lag_pass<FULL>(
      lds, tid & 63, wave, nb, a.block / 16, a.pol_sum ? a.n_pol : 1, a.dl[2 * chan] * a.dircos[2 * pp],
      a.dl[2 * chan + 1] * a.dircos[2 * pp + 1], p0 < a.n_point, frame_dw,
      [&](int64_t s, int k) { return Group{src + s * frame_dw + k * 16, 16, 0}; },
      [&](int b, float v) {
        if (p < a.n_point) out[(((b0 + b) * a.n_chan_sub + cs) * n_pg + pg) * (int64_t)a.n_point + p] = v;
      });
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_tied_lag(TiedArgs a) {
  __shared__ __attribute__((aligned(16))) char lds[kLagLds];
  if (__builtin_expect(__syncthreads_or(tied_lag_run<false>(a, lds)), 0)) tied_lag_run<true>(a, lds);
}

// One polarisation of a server's tile (request, channel, 64 pointings, run of
// 16-sample blocks), from the device ring (absolute sample s lives in slot
// s mod ring_samples).
template <bool FULL>
__device__ __forceinline__ bool serve_run(char* lds, const ServeTile* __restrict__ tile, const uint32_t* __restrict__ ring,
                                          int64_t ring_samples, int n_chan, int n_pol, int pol,
                                          const double* __restrict__ dl) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));        // nothing is held (spilled) from tile to tile, or of one pass for the other
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t frame_dw = (int64_t)n_chan * n_pol * 16;
  const ServeTile t = *tile;
  const int p0 = t.ptile * 64 + wave * 16, p = p0 + (tid & 15);
  const int pp = p < t.n_point ? p : t.n_point - 1;
  const int64_t first = (t.t_start + (int64_t)t.blk0 * 16) % ring_samples;   // a window is at most the ring
  const uint32_t* const src = ring + ((int64_t)t.chan * n_pol + pol) * 16;
  return tied_lag_pass<FULL>(
      lds, tid & 63, wave, t.n_blk, 1, 1, dl[2 * t.chan] * t.dircos[2 * pp], dl[2 * t.chan + 1] * t.dircos[2 * pp + 1],
      p0 < t.n_point, frame_dw,
      [&](int64_t s, int) {
        int64_t slot = first + s;
        if (slot >= ring_samples) slot -= ring_samples;
        const int64_t left = ring_samples - slot;
        return Group{src + slot * frame_dw, left < 16 ? (int)left : 16, ring_samples * frame_dw};
      },
      [&](int b, float v) {
        if (p < t.n_point)
          t.out[(((int64_t)(t.blk0 + b) * t.n_chan_req + (t.chan - t.chan_lo)) * n_pol + pol) * t.n_point + p] = v;
      });
}

// Persistent tile worker of the tied-beam server: each workgroup takes tiles
// from the batch.  A tile's arithmetic is exact up to its last rounding and does
// not depend on which other tiles share the launch.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_serve(const ServeTile* __restrict__ tiles, int n_tiles,
                                               const uint32_t* __restrict__ ring, int64_t ring_samples,
                                               int n_chan, int n_pol, const double* __restrict__ dl) {
  __shared__ __attribute__((aligned(16))) char lds[kLagLds];
  for (int ti = blockIdx.x; ti < n_tiles; ti += gridDim.x)
    for (int pol = 0; pol < n_pol; ++pol) {
      const bool weak = serve_run<false>(lds, tiles + ti, ring, ring_samples, n_chan, n_pol, pol, dl);
      if (__builtin_expect(__syncthreads_or(weak), 0))
        serve_run<true>(lds, tiles + ti, ring, ring_samples, n_chan, n_pol, pol, dl);
    }
}

}  // namespace

hipError_t launch_serve(const ServeTile* tiles, int n_tiles, const uint32_t* ring, int64_t ring_samples,
                        int n_chan, int n_pol, const double* dl, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  const int grid = n_tiles < 8192 ? n_tiles : 8192;
  hipLaunchKernelGGL(k_serve, dim3(grid), dim3(256), 0, s, tiles, n_tiles, ring, ring_samples, n_chan, n_pol, dl);
  return hipGetLastError();
}

hipError_t launch_tied_lag(const TiedArgs& args, hipStream_t s) {
  TiedArgs a = args;
  const int n_ptile = (a.n_point + 63) / 64;
  const int n_pg = a.pol_sum ? 1 : a.n_pol;
  const int64_t n_blk = a.n_time / a.block;
  // runs of 32 blocks, or longer ones (the weights are formed once per run)
  // while the grid still holds 2048 workgroups
  const int64_t n32 = (n_blk + kLagChunk - 1) / kLagChunk;
  int64_t times = n32 * n_ptile * a.n_chan_sub * n_pg / 2048;
  times = times < 1 ? 1 : times > 4 ? 4 : times;
  a.run_units = (int)(times * kLagChunk);
  const int64_t n_run = (n_blk + a.run_units - 1) / a.run_units;
  if ((int64_t)n_ptile * n_run > 0x7FFFFFFF || a.n_chan_sub > 65535) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)(n_ptile * n_run), (unsigned)a.n_chan_sub, (unsigned)n_pg);
  hipLaunchKernelGGL(k_tied_lag, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace fftbf
