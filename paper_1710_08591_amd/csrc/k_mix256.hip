// Weighted FFT-beam intensities of the 4 x 256 lattice (gfx950): real
// per-antenna windows (Sec. "Controlling beam shape with windowing") and
// complex gains.
//
// The N-S transform is zero-padded to M = 512 (eq. e:fftbeamform, weights
// of eq. e:w_A^a) and split as 512 = 32 x 16:
//   a = a1 + 16 a2,  A = k2 + 32 k1      (a1, a2, k1 in [0, 16), k2 in [0, 32))
//   stage 1: Y[a1][k2] = sum_{a2} x[a1 + 16 a2] W_32^{a2 k2}   (padded 16 -> 32 DFT)
//   twiddle: Z[a1][k2] = Y[a1][k2] W_512^{a1 k2}
//   stage 2: B[k2 + 32 k1] = sum_{a1} Z[a1][k2] W_16^{a1 k1}
//
// Stage 1 is a dense product on the matrix cores, per sample and E-W beam:
//   C[a1][k2] = A[a1][(a2, re|im)] * B[(a2, re|im)][k2]
// A holds the weighted E-W sums of the E-W beam at N-S position a1 + 16 a2 and
// B the realified coefficients, each as two FP16 terms (hi + lo, about 22
// significant bits); three products accumulate into the same FP32
// accumulators, so stage 1 is accurate to FP32 rounding.  FP32 plans take the
// smallest first; FP16 plans the largest, which needs no low terms yet: a
// lone wavefront per SIMD (4 x 256, 11 channels, 13 blocks of 80 samples)
// takes 151 us that way and 158 the other, which gains 2 % on a full chip.
//
// Stage 2 is the FP32 16-point DFT over a1 in registers, one (E-W beam, k2)
// per lane.  The data go from the stage-1 layout (lane = (a1 group, k2)) to
// the stage-2 layout (lane = (E-W beam, k2), all a1) through an LDS tile of
// one E-W beam pair at a time (9 KB per wavefront), so three wavefronts per
// SIMD fit.  |B|^2 accumulates in registers over the block; at its end the
// sums pass once more through LDS so the kept beams of the channel's clamp
// table can be stored with coalesced writes.
//
// FP32 plans (TAN): the twiddle in tangent form, one fused multiply-add per
// component, the factor Re W carried into stage 2 as the 25 multipliers of
// column k2 (LDS, two wavefronts share them and the weights).  |B|^2 is formed
// first and joins the block sum with one rounding: most of the error is the
// sum's, so with half its roundings the output is nearer to 64 bits than FP32
// operands throughout with two (window, blocks of 16: 2-norm 0.75e-7 against
// 1.01e-7, blocks of 80 1.38e-7 against 1.93e-7; gains 0.89e-7 against
// 1.09e-7), which pays for the terms' 22 bits (0.94e-7 with two).
// FP16 plans: whole twiddles, the weights in registers, two roundings; faster,
// less accurate.
//
// Where any weight other than zero lies more than 2^10 below the largest, the
// low terms of its sums would be lost.  That matters when the antennas of the
// large weights hold no data (calibrations of 1e6 on two dead E-W columns,
// say), so such weights are not scaled to the largest and each frame's sums are
// scaled by their own largest instead (wide_range): an error of 2^-39 of it at most, below
// FP32's rounding, over FP32's whole range.
// 4 x 256, 64 channels, 2 polarisations, 128 blocks of 16 samples, whole
// transform on the vector units -> this: window 488 -> 442 us (464 with a
// frame scale), gains 519 -> 488 us (506 with a frame scale).
// Bound by vector issue: about 750 instructions per
// frame and wavefront, 48 matrix products behind them (a fourth product each
// costs nothing).  Both stages on the matrix cores, without the LDS tile, took
// 893 us: splitting Z costs what the DFT's instructions do.
#include "dev_common.h"
#include "dev_f16.h"
#include "kernels.h"

#include <type_traits>

namespace fftbf {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// plan table layout (bytes)
constexpr size_t kH256B1Off = 0;      // [term 2][kt 2][part 2][lane 64][8] halves
constexpr size_t kH256TwOff = 8192;   // FP16 plans: [lane 64][kt 2][q 4] float2
constexpr size_t kH256Bytes = 8192 + 4096;

// realified coefficient of stage 1: output part `part` (0 Re, 1 Im) of k2
// from input component comp (0 Re, 1 Im) of position a2, W = W_32^{a2 k2} = c + i s,
//   Re(W x) = c xr - s xi,  Im(W x) = s xr + c xi
__device__ double h256_coef(int a2, int comp, int k2, int part) {
  double s, c;
  sincospi(-2.0 * (double)((a2 * k2) & 31) / 32.0, &s, &c);
  return part == 0 ? (comp == 0 ? c : -s) : (comp == 0 ? s : c);
}

// FP64 on the device, rounded once into the operand layouts.
__global__ void k_mix256_tables(void* tab) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  char* base = static_cast<char*>(tab);
  // stage-1 operand B[k = 8 g + j][n] of part `part` of k2 = 16 kt + n,
  // input (a2, comp) = (4 g + j / 2, j % 2), as hi + lo FP16 terms
  if (i < 2 * 2 * 64 * 8) {
    const int j = i & 7, lane = (i >> 3) & 63, part = (i >> 9) & 1, kt = (i >> 10) & 1;
    const double v = h256_coef(4 * (lane >> 4) + (j >> 1), j & 1, 16 * kt + (lane & 15), part);
    _Float16* t = reinterpret_cast<_Float16*>(base + kH256B1Off);
    const _Float16 hi = (_Float16)(float)v;
    t[i] = hi;
    t[2048 + i] = (_Float16)(float)(v - (double)(float)hi);
  }
  // twiddles W_512^{a1 k2} of lane (g, n), slot (kt, q): a1 = 4 g + q, k2 = 16 kt + n
  if (i < 64 * 8) {
    const int kt = (i >> 2) & 1, q = i & 3, lane = i >> 3;
    const int a1 = 4 * (lane >> 4) + q, k2 = 16 * kt + (lane & 15);
    double s, c;
    sincospi(-2.0 * (double)((a1 * k2) & 511) / 512.0, &s, &c);
    reinterpret_cast<float2*>(base + kH256TwOff)[i] = make_float2((float)c, (float)s);
  }
}

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Weighted E-W sums of one N-S position (dword d: byte q holds antenna q, real
// part in its high nibble) for all four E-W beams, sum_q h_q z_q (-i)^{e q}
// with h real (4 floats) or complex (GAIN: 8).
template <bool GAIN>
__device__ __forceinline__ void ew_weighted(uint32_t d, const float* h, cf (&b)[4]) {
  cf z[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    z[q] = cf{(float)(int)__builtin_amdgcn_sbfe((int)d, 8 * q + 4, 4), (float)(int)__builtin_amdgcn_sbfe((int)d, 8 * q, 4)};
  cf s[2], m[2];                             // x_0 + x_2, x_1 + x_3 and the differences
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const cf u = z[k], v = z[k + 2];
    if constexpr (GAIN) {
      const cf hu{h[2 * k], h[2 * k + 1]}, hv{h[2 * k + 4], h[2 * k + 5]};
      const cf w = cmul(u, hu);
      s[k] = cf{fmaf(-hv.i, v.i, fmaf(hv.r, v.r, w.r)), fmaf(hv.i, v.r, fmaf(hv.r, v.i, w.i))};
      m[k] = cf{fmaf(hv.i, v.i, fmaf(-hv.r, v.r, w.r)), fmaf(-hv.i, v.r, fmaf(-hv.r, v.i, w.i))};
    } else {
      const cf w{h[k] * u.r, h[k] * u.i};
      s[k] = cf{fmaf(h[k + 2], v.r, w.r), fmaf(h[k + 2], v.i, w.i)};
      m[k] = cf{fmaf(-h[k + 2], v.r, w.r), fmaf(-h[k + 2], v.i, w.i)};
    }
  }
  b[0] = cadd(s[0], s[1]);
  b[1] = cf{m[0].r + m[1].i, m[0].i - m[1].r};
  b[2] = csub(s[0], s[1]);
  b[3] = cf{m[0].r - m[1].i, m[0].i + m[1].r};
}

// Exponent that takes the largest of the wavefront's m >= 0 to [2^14, 2^15);
// 0 for zero and infinity.  Positive floats are ordered as their bits are.
__device__ __forceinline__ int frame_exponent(float m) {
  int v = __float_as_int(m);
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true));   // row_ror 8, 4, 2, 1
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x124, 0xF, 0xF, true));
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x122, 0xF, 0xF, true));
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x121, 0xF, 0xF, true));
  v = max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
          max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
  return v == 0 || v >= 0x7F800000 ? 0 : (v >> 23) - 127 - 14;
}

// One wavefront per (block, channel, polarisation group).  Lane l = 16 g + n:
// stage 1 holds a1 = 4 g + q (q < 4) and k2 = 16 kt + n (kt < 2); stage 2
// takes E-W beam 2 p + (l >> 5) of pair p and k2 = l & 31.  The weights are
// scaled by a power of two so that the largest lies in [2^8, 2^9): an E-W sum
// is below 64 of the largest, 2^15, within FP16.  The terms of a sum then hold
// it to 2^-25 (half of FP16's smallest step): 2^-23 of the product of the
// smallest weight that the rule lets pass, 2^-2, with a voltage of 1.  The
// block sums are scaled back exactly.  Scaled to [1/2, 1) the low terms of
// weights of e^{+-2} were already subnormal.
template <bool TAN, bool GAIN>
__global__ __launch_bounds__(64 * (TAN ? 2 : 1)) __attribute__((amdgpu_waves_per_eu(3))) void k_mix256(MixArgs a) {
  constexpr int N = 256, M = 512, HW = GAIN ? 8 : 4;
  constexpr int kWpg = TAN ? 2 : 1;           // wavefronts per workgroup
  constexpr int ROW = 18;                     // complex values per (E-W beam, k2) row: 16 a1 + 2 pad
  constexpr int NMU = 28;                     // floats per column of multipliers: 25, in 16-byte loads
  static_assert(dit_slots(16) <= NMU, "multipliers");
  __shared__ float4 lds_tiles[kWpg][2 * 32 * ROW / 2];
  __shared__ __attribute__((aligned(16))) float lds_mu[TAN ? 32 : 1][NMU];
  __shared__ __attribute__((aligned(16))) float lds_h[TAN ? N * HW : 4];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float4* const lds_raw = lds_tiles[wave];
  cf* const tile = reinterpret_cast<cf*>(lds_raw);
  const int n = lane & 15, g = lane >> 4;

  // the weights, scaled by 2^-ex: the largest component in [2^8, 2^9) (every
  // wavefront looks at them all)
  int ex;
  bool wide = false;
  float hw[4][TAN ? 1 : HW];                  // at the lane's N-S positions n + 64 g + 16 i
  {
    constexpr int PER = HW / 4;               // floats per weight
    float m = 0.f, mag[16];                   // the larger component of the lane's 16 weights
    constexpr int kVec = N * HW / 256;        // the lane's 16-byte vectors of weights
    float4 hv[kVec];
#pragma unroll
    for (int i = 0; i < kVec; ++i) {
      hv[i] = reinterpret_cast<const float4*>(a.taper)[lane + 64 * i];
      const float4 v = hv[i];
      const float f[4] = {fabsf(v.x), fabsf(v.y), fabsf(v.z), fabsf(v.w)};
#pragma unroll
      for (int k = 0; k < 4; k += PER) {
        float& w = mag[(4 * i + k) / PER];
        w = fmaxf(f[k], f[k + PER - 1]);
        m = fmaxf(m, w);
      }
    }
#pragma unroll
    for (int d = 1; d < 64; d *= 2) m = fmaxf(m, __shfl_xor(m, d));
    ex = m > 0.f && m < INFINITY ? ilogbf(m) - 8 : 0;
    if constexpr (TAN) {
      // the rule: a weight other than zero below 2^-10 of the largest
      const float low = ldexpf(m, -10);
      bool below = false;
#pragma unroll
      for (int i = 0; i < 16; ++i) below |= mag[i] > 0.f && mag[i] < low;
      wide = __any(below);
      // (strong weights: 2^-12 keeps a block sum of up to 1024 times the largest output finite)
      if (wide) ex = m > 0x1p30f ? 6 : 0;
      // each wavefront stores its half of what both hold (256 blocks of 4 samples,
      // 64 channels, 2 polarisations, gains: 294 us, 317 with the weights read
      // again, 307 with the whole transform on the vector units)
#pragma unroll
      for (int i = 0; i < kVec; i += kWpg) {
        const float4 v = wave ? hv[i + 1] : hv[i];
        reinterpret_cast<float4*>(lds_h)[lane + 64 * (i + wave)] =
            make_float4(ldexpf(v.x, -ex), ldexpf(v.y, -ex), ldexpf(v.z, -ex), ldexpf(v.w, -ex));
      }
      for (int i = tid; i < 32 * dit_slots(16); i += 64 * kWpg)
        lds_mu[i / dit_slots(16)][i % dit_slots(16)] = a.mult[i];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < HW; ++q) hw[i][q] = ldexpf(a.taper[HW * (n + 64 * g + 16 * i) + q], -ex);
    }
  }
  if constexpr (TAN) __syncthreads();
  const int64_t task = (int64_t)blockIdx.x * kWpg + wave;
  if (task >= a.n_wg) return;
  int wg = (int)task;
  const int pg = wg % a.n_pg;
  wg /= a.n_pg;
  const int chan = wg % a.n_chan;
  const int blk = wg / a.n_chan;

  const char* tab = static_cast<const char*>(a.mat);
  half8 B1[2][2][2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int part = 0; part < 2; ++part)
        B1[p][kt][part] = *reinterpret_cast<const half8*>(
            tab + kH256B1Off + 2 * (p * 2048 + ((kt * 2 + part) * 64 + lane) * 8));
  // twiddles of a1 = 4 g + q, k2 = 16 kt + n.  TAN: 1 + i t, in column 16
  // pr + i t; else whole
  float tt[2][4], pr[4];
  cf tw[2][4];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int kt = k >> 2, q = k & 3;
    if constexpr (TAN) {
      const float2 w = a.tw[(4 * g + q) * 32 + 16 * kt + n];
      tt[kt][q] = kt && n == 0 ? w.y : w.x;
      if (kt) pr[q] = n == 0 ? w.x : 1.f;
    } else {
      const float2 w = reinterpret_cast<const float2*>(tab + kH256TwOff)[lane * 8 + k];
      tw[kt][q] = cf{w.x, w.y};
    }
  }
  const int k2s = lane & 31, es = lane >> 5;  // stage-2 column and E-W beam within the pair
  float acc[2][16];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[p][k] = 0.f;

  const int pol_lo = (a.pol_iter == 1) ? pg : 0;
  const int pol_hi = (a.pol_iter == 1) ? pg + 1 : a.n_pol;
  const int64_t frame_stride = (int64_t)a.n_chan * a.n_pol * N;   // dwords per sample
  const int64_t t0 = (int64_t)blk * a.block;

  auto frame = [&](auto wide_range, const uint32_t (&dw)[4]) {
    cf xw[4][4];                              // [E-W beam][position]
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      cf b[4];
      if constexpr (TAN) {
        float h[HW];
#pragma unroll
        for (int v = 0; v < HW / 4; ++v) {
          const float4 f = *reinterpret_cast<const float4*>(&lds_h[HW * (n + 64 * g + 16 * i) + 4 * v]);
          h[4 * v] = f.x;
          h[4 * v + 1] = f.y;
          h[4 * v + 2] = f.z;
          h[4 * v + 3] = f.w;
        }
        ew_weighted<GAIN>(dw[i], h, b);
      } else {
        ew_weighted<GAIN>(dw[i], hw[i], b);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) xw[e][i] = b[e];
    }
    // wide_range: the frame's sums scaled by 2^-fex, the largest in [2^14, 2^15)
    int fex = 0;
    if constexpr (decltype(wide_range)::value) {
      float m = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) m = fmaxf(fmaxf(m, fabsf(xw[i >> 2][i & 3].r)), fabsf(xw[i >> 2][i & 3].i));
      fex = frame_exponent(m);
#pragma unroll
      for (int i = 0; i < 16; ++i)
        xw[i >> 2][i & 3] = cf{ldexpf(xw[i >> 2][i & 3].r, -fex), ldexpf(xw[i >> 2][i & 3].i, -fex)};
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      // ---- stage 1 and twiddle for E-W beams 2p, 2p + 1, into the tile ----
#pragma unroll
      for (int ep = 0; ep < 2; ++ep) {
        const int e = 2 * p + ep;
        f32x4 y[2][2];
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) split2(xw[e][i].r, xw[e][i].i, hi[i], lo[i]);
        const half8 Ah = __builtin_bit_cast(half8, hi), Al = __builtin_bit_cast(half8, lo);
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int part = 0; part < 2; ++part) {
            const half8 A0 = TAN ? Al : Ah, A2 = TAN ? Ah : Al;
            y[kt][part] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A0, B1[0][kt][part], f32x4{0.f, 0.f, 0.f, 0.f},
                                                                 0, 0, 0);
            y[kt][part] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Ah, B1[1][kt][part], y[kt][part], 0, 0, 0);
            y[kt][part] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A2, B1[0][kt][part], y[kt][part], 0, 0, 0);
          }
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          cf z[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float yr = y[kt][0][q], yi = y[kt][1][q];
            if constexpr (decltype(wide_range)::value) {
              yr = ldexpf(yr, fex);
              yi = ldexpf(yi, fex);
            }
            if constexpr (!TAN) z[q] = cmul(cf{yr, yi}, tw[kt][q]);
            else if (kt == 0) z[q] = cf{fmaf(-tt[0][q], yi, yr), fmaf(tt[0][q], yr, yi)};
            else z[q] = cf{fmaf(-tt[1][q], yi, pr[q] * yr), fmaf(tt[1][q], yr, pr[q] * yi)};
          }
          float4* dst = reinterpret_cast<float4*>(&tile[(ep * 32 + 16 * kt + n) * ROW + 4 * g]);
          dst[0] = make_float4(z[0].r, z[0].i, z[1].r, z[1].i);
          dst[1] = make_float4(z[2].r, z[2].i, z[3].r, z[3].i);
        }
      }
      wave_lds_sync();
      // ---- stage 2: 16-point DFT over a1 for (E-W beam 2p + es, k2s) ----
      cf x[16];
      {
        const float4* src = reinterpret_cast<const float4*>(&tile[(es * 32 + k2s) * ROW]);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          const float4 v = src[m];
          x[2 * m] = cf{v.x, v.y};
          x[2 * m + 1] = cf{v.z, v.w};
        }
      }
      if constexpr (TAN) {
        float mu[NMU];
#pragma unroll
        for (int k = 0; k < NMU / 4; ++k) {
          const float4 v = *reinterpret_cast<const float4*>(&lds_mu[k2s][4 * k]);
          mu[4 * k] = v.x;
          mu[4 * k + 1] = v.y;
          mu[4 * k + 2] = v.z;
          mu[4 * k + 3] = v.w;
        }
        wave_lds_sync();
        dit_rs<16>(x, mu);
      } else {
        wave_lds_sync();
        dit<16>(x);
      }
#pragma unroll
      for (int k1 = 0; k1 < 16; ++k1) {
        if constexpr (TAN) acc[p][k1] += fmaf(x[k1].r, x[k1].r, x[k1].i * x[k1].i);
        else acc[p][k1] = cnorm_acc(x[k1], acc[p][k1]);
      }
    }
  };

  auto run = [&](auto wide_range) {
    for (int pol = pol_lo; pol < pol_hi; ++pol) {
      // the lane's N-S positions a1 + 16 a2 = n + 64 g + 16 i, i < 4
      const uint32_t* src = a.volts + ((int64_t)chan * a.n_pol + pol) * N + n + 64 * g;
      const uint32_t* last = src + (t0 + a.block - 1) * frame_stride;
      uint32_t b0[4], b1[4];
      const uint32_t* q0 = src + t0 * frame_stride;
#pragma unroll
      for (int i = 0; i < 4; ++i) b0[i] = __builtin_nontemporal_load(q0 + 16 * i);
      // two frame buffers in turn; the load past the block's last frame
      // re-reads that frame (cached), so no load is conditional
      for (int s = 0; s < a.block; s += 2) {
        const uint32_t* q1 = (s + 1 < a.block) ? q0 + frame_stride : last;
#pragma unroll
        for (int i = 0; i < 4; ++i) b1[i] = __builtin_nontemporal_load(q1 + 16 * i);
        frame(wide_range, b0);
        if (s + 1 >= a.block) break;
        q0 = (s + 2 < a.block) ? q1 + frame_stride : last;
#pragma unroll
        for (int i = 0; i < 4; ++i) b0[i] = __builtin_nontemporal_load(q0 + 16 * i);
        frame(wide_range, b1);
      }
    }
  };
  if (TAN && wide) run(std::true_type{});
  else run(std::false_type{});

  // ---- block end: beams A = k2 + 32 k1 of E-W beam 2p + es, clamp, store ----
  float* lds_i = reinterpret_cast<float*>(lds_raw);
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int k1 = 0; k1 < 16; ++k1) lds_i[(2 * p + es) * M + k2s + 32 * k1] = acc[p][k1];
  wave_lds_sync();
  const int keep = a.n_keep;
  const int32_t* sel = a.sel ? a.sel + (int64_t)chan * keep : nullptr;
  float* o = a.out + (((int64_t)blk * a.n_chan + chan) * a.n_pg + pg) * 4 * keep;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    for (int j = lane; j < keep; j += 64) o[e * keep + j] = ldexpf(lds_i[e * M + (sel ? sel[j] : j)] * a.norm, 2 * ex);
}

}  // namespace

size_t mix256_table_bytes() { return kH256Bytes; }

hipError_t launch_mix256_tables(void* mat, hipStream_t s) {
  hipLaunchKernelGGL(k_mix256_tables, dim3(8), dim3(256), 0, s, mat);
  return hipGetLastError();
}

hipError_t launch_mix256(const MixArgs& a, bool fp32, int64_t n_wg, hipStream_t s) {
  if (n_wg == 0) return hipSuccess;
  if (n_wg > 0x7FFFFFFF) return hipErrorInvalidConfiguration;
  MixArgs b = a;
  b.n_wg = n_wg;
  const unsigned n2 = (unsigned)((n_wg + 1) / 2);
  if (a.gains) hipLaunchKernelGGL((k_mix256<true, true>), dim3(n2), dim3(128), 0, s, b);
  else if (fp32) hipLaunchKernelGGL((k_mix256<true, false>), dim3(n2), dim3(128), 0, s, b);
  else hipLaunchKernelGGL((k_mix256<false, false>), dim3((unsigned)n_wg), dim3(64), 0, s, b);
  return hipGetLastError();
}

}  // namespace fftbf
