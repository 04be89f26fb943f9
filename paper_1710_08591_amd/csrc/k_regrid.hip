// Intensity-domain regridding of FFT beams to arbitrary steering angles
// (eq. e:bp_max_arbitrary, Sec. "Redundancy-stacked visibilities"):
//
//   b_p(theta) = sum_A w^A_p b_A,  w^A_p = (1/M) sin((2n-1) pi y) / sin(pi y),
//   y = (d/lambda) sin(theta) - A/M,
//
// exact whenever M >= 2n - 1, which the zero-padded N-S axis (M = 2n)
// satisfies.  Applied per channel along N-S for every E-W FFT beam, so the
// targets can be the same sin(theta) in every channel (achromatic beams from
// the chromatic FFT grid of eq. e:theta_A).
//
// The weights are generated once in FP64 on the device (the removable
// singularity at integer y takes its limit (2n-1)/M), rounded to FP32 and
// stored as three BF16 terms each (dev_bf16.h): six bytes a weight, where FP32
// would take four, so that no workgroup splits them again.  The contraction
// Out[row][target] = sum_A I[row][A] W[target][A] (rows = (block, polarisation,
// E-W beam) of one channel) runs on v_mfma_f32_16x16x32_bf16, six products for
// one in FP32.  A workgroup of W wavefronts owns 256 targets (TG = 2 groups of
// wavefronts) or 64; a wavefront owns 16 RT rows against 128 or 64 targets, of
// which it skips the pairs of tiles of 16 that hold none.  The K axis (beams A)
// is walked in chunks of 32, KS of them between barriers:
//   * the intensities go straight from HBM to registers: lane (m, g) of a wave
//     feeds row m with the beams 4 g .. 4 g + 3 and 16 + 4 g .. of the chunk (two
//     16-byte loads, contiguous over g), splits them there and multiplies them
//     with every target tile;
//   * the weights are stored in the order the lanes read them, are copied to
//     LDS as they are (two buffers) and read back 16 bytes a lane;
//   * the global loads run two stages ahead for the intensities and one for the
//     weights (which the L2 holds), so their latency hides under the matrix work.
// The workgroups of one channel run on one XCD (its L2 then holds the
// channel's weights: 768 KB at M = 512 and 256 targets).
//
// 128 blocks, 64 channels, 2 polarisations, 8 E-W beams, M = 512, 256 2-D
// pointings (34 GFLOP): 196 us, from 351 on v_mfma_f32_16x16x4_f32, whose rate
// bounds it to 219.  Six BF16 products for one make that 206 GFLOP, 1050 TFLOP/s
// of the 1257 that a large BF16 matrix product reaches here.  64 targets: bound
// by the reads (268 MB of intensities in 70 us, 88 before).  The errors against
// 64 bits are less than half of the FP32 instructions' (2-norm 1.5e-7 against
// 3.6e-7 at M = 512): fewer roundings of the partial sums.

#include "dev_bf16.h"
#include "dev_common.h"
#include "kernels.h"

namespace fftbf {

namespace {

// Weight w^A of FFT beam A for the steering y (FP64).  coef == nullptr: the
// pointed kernel of eq. e:bp_max_arbitrary in closed form.  Otherwise the
// optimally windowed kernel (eq. e:w_opt mapped by eq. e:wA_from_wdelta):
// w^A = (1/M) [c_0 + 2 sum_{d=1}^{n-1} c_d cos(2 pi d (A/M - y))] with the
// window's lag coefficients c_d = R_d / ((n - d) N), summed with a
// unit-modulus recurrence.
__device__ double regrid_weight(int A, double y, int n, int m, const double* coef) {
  const double ya = y - (double)A / (double)m;
  if (!coef) {
    const double den = sinpi(ya);
    if (fabs(den) < 1e-12) return (double)(2 * n - 1) / m;
    return sinpi((double)(2 * n - 1) * ya) / den / m;
  }
  double s1, c1;
  sincospi(2.0 * ya, &s1, &c1);
  double er = c1, ei = s1, acc = coef[0];
  for (int d = 1; d < n; ++d) {
    acc += 2.0 * coef[d] * er;
    const double nr = er * c1 - ei * s1;
    ei = er * s1 + ei * c1;
    er = nr;
  }
  return acc / m;
}

// [chan][target / 16][chunk of 32 beams][term 3][lane 64][4]: dword q of lane
// (g, n) holds the BF16 terms of beams 2 q, 2 q + 1 of the lane's eight (4 g ..
// 4 g + 3, 16 + 4 g .. 16 + 4 g + 3) for target n of the tile
__global__ void k_regrid_weights(uint32_t* w, const double* dl, const double* sin_t, const double* coef, int n_chan,
                                 int n_target, int n_target_pad, int n, int m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)n_chan * n_target_pad * (m / 2);
  if (i >= total) return;
  const int q = (int)(i & 3), lane = (int)((i >> 2) & 63);
  int64_t r = i >> 8;
  const int kc = (int)(r % (m / 32));
  r /= m / 32;
  const int tile = (int)(r % (n_target_pad / 16)), c = (int)(r / (n_target_pad / 16));
  const int j = tile * 16 + (lane & 15);
  const int A = 32 * kc + 4 * (lane >> 4) + 2 * (q & 1) + 16 * (q >> 1);
  uint32_t h = 0, mid = 0, lo = 0;
  if (j < n_target) {
    const double y = dl[2 * c + 1] * sin_t[j];
    split3((float)regrid_weight(A, y, n, m, coef), (float)regrid_weight(A + 1, y, n, m, coef), h, mid, lo);
  }
  uint32_t* o = w + (i >> 8) * 768 + (i & 255);
  o[0] = h;
  o[256] = mid;
  o[512] = lo;
}

// E-W weights of 2-D pointings: w[chan][target][e], e < m (= 8), zero rows
// for padded targets; the pointed kernel of eq. e:bp_max_arbitrary on the
// (padded) E-W axis.
__global__ void k_regrid_ew_weights(float* w, const double* dl, const double* dircos_ew, int n_chan, int n_target,
                                    int n_target_pad, int n, int m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)n_chan * n_target_pad * m;
  if (i >= total) return;
  const int e = (int)(i % m);
  const int j = (int)((i / m) % n_target_pad);
  const int c = (int)(i / ((int64_t)m * n_target_pad));
  w[i] = j < n_target ? (float)regrid_weight(e, dl[2 * c] * dircos_ew[j], n, m, nullptr) : 0.f;
}

// Compact kernels: the k FFT beams nearest the steering on the circular beam
// grid, first = rint(y M) - (k-1)/2 (mod M), with their full-kernel weights.
// Layout: first[chan][target], tw[chan][tap][target].
__global__ void k_regrid_tap_table(int* first, float* tw, const double* dl, const double* sin_t, const double* coef,
                                   int n_chan, int n_target, int k, int n, int m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)n_chan * k * n_target;
  if (i >= total) return;
  const int t = (int)(i % n_target);
  const int j = (int)((i / n_target) % k);
  const int c = (int)(i / ((int64_t)n_target * k));
  const double y = dl[2 * c + 1] * sin_t[t];
  const int64_t f0 = (int64_t)rint(y * (double)m) - (k - 1) / 2;
  const int f = (int)(((f0 % m) + m) % m);
  if (j == 0) first[(int64_t)c * n_target + t] = f;
  tw[i] = (float)regrid_weight((f + j) % m, y, n, m, coef);
}

// One wavefront's sums on v_mfma_f32_16x16x4_f32, from the same operands: for
// values that are not finite, or too small for BF16 terms.
template <int RT, int NT>
__device__ __forceinline__ void regrid_f32(const float* const (&arow)[RT], const u32x4* wt,
                                        int tile_stride, int n_tile, int tile_step, int n_chunk, int lane,
                                        f32x4 (&acc)[RT][NT]) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[rt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int kc = 0; kc < n_chunk; ++kc) {
    f32x4 v[RT][2];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        v[rt][h] = *reinterpret_cast<const f32x4*>(arow[rt] + 32 * kc + 16 * h);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if (nt * tile_step >= n_tile) break;
      const u32x4* wp = wt + (int64_t)nt * tile_step * tile_stride + kc * 192 + lane;
      const u32x4 w0 = wp[0], w1 = wp[64], w2 = wp[128];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float wa = (bf16_lo(w0[q]) + bf16_lo(w1[q])) + bf16_lo(w2[q]);
        const float wb = (bf16_hi(w0[q]) + bf16_hi(w1[q])) + bf16_hi(w2[q]);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          acc[rt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[rt][q >> 1][2 * (q & 1)], wa, acc[rt][nt], 0, 0, 0);
          acc[rt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[rt][q >> 1][2 * (q & 1) + 1], wb, acc[rt][nt], 0, 0, 0);
        }
      }
    }
  }
}

// RT: tiles of 16 rows per wavefront.  TG: groups of wavefronts along the
// targets (2: 256 targets per workgroup, 1: 64).  EW2D: 2-D pointings on an
// E-W axis padded to 8 beams -- the 8 E-W rows of each (block, pol group)
// are combined with the E-W weights in the epilogue.
template <int W, int RT, int TG, int KS, bool ONE, bool EW2D>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(KS == 2 ? 3 : TG == 1 || ONE ? 4 : W / 4))) void k_regrid(RegridArgs a) {
  constexpr int NT = TG == 2 ? 8 : 4;     // target tiles per wavefront
  constexpr int TILES = NT * TG;          // target tiles per workgroup
  constexpr int RG = W / TG;              // groups of wavefronts along the rows
  constexpr int WV = (KS * TILES * 192 + 64 * W - 1) / (64 * W);   // 16-byte copies per thread and stage
  __shared__ u32x4 lds_w[ONE ? 1 : 2][WV * 64 * W];

  // workgroup -> (channel, target group, row group), a channel's on one XCD
  const int64_t per_xcd = gridDim.x >> 3;
  const int64_t task = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  const int n_tt = a.n_target_pad / (16 * TILES);
  const int n_rg = (a.rows_per_chan + 16 * RT * RG - 1) / (16 * RT * RG);
  if (task >= (int64_t)n_rg * n_tt * a.n_chan) return;
  const int rg = (int)(task % n_rg);
  const int tt = (int)(task / n_rg % n_tt);
  const int chan = (int)(task / ((int64_t)n_rg * n_tt));

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, g = lane >> 4;
  const int tg = wave % TG, wr = wave / TG;
  const int rows = a.rows_per_chan;
  const int t0 = tt * 16 * TILES;
  const int live = min(TILES, (a.n_target - t0 + 15) / 16);   // tiles with targets; the wave takes tg, tg + TG, ...
  const int used = min(TILES, (live + 2 * TG - 1) / (2 * TG) * (2 * TG));   // with the (zero) tiles that fill its pairs
  const int n_chunk = a.m_ns / 32, n_stage = ONE ? 1 : n_chunk / KS;
  const u32x4* const wt = reinterpret_cast<const u32x4*>(a.w) +
                          ((int64_t)chan * (a.n_target_pad / 16) + tt * TILES) * n_chunk * 192;

  // this lane's intensity rows (channel-local r -> global row through the
  // R = n_pg * m_ew rows of one block, R a power of two)
  const int row0 = (rg * RG + wr) * 16 * RT;
  const float* arow[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int r = row0 + rt * 16 + m;
    const int64_t grow = ((int64_t)(r >> a.log2_r) * a.n_chan + chan) * (1 << a.log2_r) + (r & ((1 << a.log2_r) - 1));
    arow[rt] = a.in + (r < rows ? grow : 0) * a.m_ns + 4 * g;
  }

  f32x4 acc[RT][NT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[rt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  // the next two stages' intensities and the next one's weights, in flight
  constexpr int D = ONE ? 1 : 2;
  f32x4 av[D][KS][RT][2];
  u32x4 wv[WV];
  // no load is conditional (rows and tiles past the end read the first row and
  // the last tile used): a branch around a load waits for those before it
  const u32x4* wp[WV];
#pragma unroll
  for (int it = 0; it < WV; ++it) {
    const int idx = min(tid + 64 * W * it, KS * TILES * 192 - 1);      // [chunk of the stage][tile][192]
    const int tile = min(idx / 192 % TILES, used - 1);
    wp[it] = wt + (int64_t)tile * n_chunk * 192 + idx / (192 * TILES) * 192 + idx % 192;
  }
  auto load_weights = [&](int st) {
    if (st >= n_stage) return;
#pragma unroll
    for (int it = 0; it < WV; ++it) wv[it] = wp[it][st * KS * 192];
  };
  auto load_rows = [&](int st, f32x4 (&to)[KS][RT][2]) {
    if (st >= n_stage) return;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          to[ks][rt][h] = *reinterpret_cast<const f32x4*>(arow[rt] + 32 * (st * KS + ks) + 16 * h);
  };
  auto stage = [&](int st, f32x4 (&v)[KS][RT][2]) {
    // the buffer written below was read in the stage before this barrier
    __syncthreads();
    const u32x4* wl = lds_w[ONE ? 0 : st & 1] + tg * 192 + lane;
    u32x4 at[KS][RT][3];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t h, mid, lo;
          split3(v[ks][rt][q >> 1][2 * (q & 1)], v[ks][rt][q >> 1][2 * (q & 1) + 1], h, mid, lo);
          at[ks][rt][0][q] = h;
          at[ks][rt][1][q] = mid;
          at[ks][rt][2][q] = lo;
        }
    if constexpr (!ONE) load_rows(st + D, v);
    // two target tiles at a time: 2 RT independent sums per term
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int nt = 0; nt < NT; nt += 2) {
        if (nt * TG + tg >= live) break;
        u32x4 w[2][3];
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int t = 0; t < 3; ++t) w[k][t] = wl[((ks * TILES + (nt + k) * TG) * 3 + t) * 64];
#pragma unroll
        for (int t = 0; t < 6; ++t) {
          constexpr int ta[6] = {1, 0, 2, 0, 1, 0}, tb[6] = {1, 2, 0, 1, 0, 0};
#pragma unroll
          for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
              acc[rt][nt + k] = mfma_bf16(at[ks][rt][ta[t]], w[k][tb[t]], acc[rt][nt + k]);
        }
      }
    if constexpr (!ONE) {
#pragma unroll
      for (int it = 0; it < WV; ++it) lds_w[~st & 1][tid + 64 * W * it] = wv[it];
      load_weights(st + 2);
    }
  };

  load_weights(0);
  load_rows(0, av[0]);
  if constexpr (D == 2) load_rows(1, av[1]);
#pragma unroll
  for (int it = 0; it < WV; ++it) lds_w[0][tid + 64 * W * it] = wv[it];
  if constexpr (ONE) {
    stage(0, av[0]);
  } else {
    load_weights(1);
#pragma unroll 1
    for (int st = 0; st < n_stage; st += 2) {           // n_stage is even (M >= 64 KS)
      stage(st, av[0]);
      stage(st + 1, av[D - 1]);
    }
  }
  {
    float bad = 0.f;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = acc[rt][nt][i];
          bad = fabsf(v) < 0x1p-90f && v != 0.f ? 1.f : fmaf(v, 0.f, bad);
        }
    if (!__all(bad == 0.f))
      regrid_f32<RT, NT>(arow, wt + (int64_t)tg * n_chunk * 192, n_chunk * 192, live - tg, TG, n_chunk, lane, acc);
  }

  // acc[rt][nt][i]: row row0 + 16 rt + 4 g + i, target t0 + 16 (TG nt + tg) + lane % 16
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    if constexpr (EW2D) {
      // rows [0, 8) and [8, 16) of the tile are two (block, pol group) groups of
      // 8 E-W beams: lane group g holds E-W beams 4 (g & 1) .. +3 of group g >> 1
      const int grp_row = row0 + rt * 16 + 8 * (g >> 1);
      const bool ok = grp_row < rows && (g & 1) == 0;
      const int gi = grp_row >> 3;
      const int blk = gi / a.n_pg, pg = gi - blk * a.n_pg;
      float* o = a.out + (((int64_t)blk * a.n_chan + chan) * a.n_pg + pg) * a.n_target;
      const float* wew = a.wew + ((int64_t)chan * a.n_target_pad + t0) * 8 + 4 * (g & 1);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int tl = 16 * (nt * TG + tg) + m;
        const f32x4 we = *reinterpret_cast<const f32x4*>(wew + tl * 8);
        float part = we[0] * acc[rt][nt][0];
        part = fmaf(we[1], acc[rt][nt][1], part);
        part = fmaf(we[2], acc[rt][nt][2], part);
        part = fmaf(we[3], acc[rt][nt][3], part);
        part += __shfl_xor(part, 16);
        if (ok && t0 + tl < a.n_target) o[t0 + tl] = part;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int ro = row0 + rt * 16 + 4 * g + i;
        if (ro >= rows) continue;
        const int64_t go =
            ((int64_t)(ro >> a.log2_r) * a.n_chan + chan) * (1 << a.log2_r) + (ro & ((1 << a.log2_r) - 1));
        float* o = a.out + go * a.n_target;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int t = t0 + 16 * (nt * TG + tg) + m;
          if (t < a.n_target) o[t] = acc[rt][nt][i];
        }
      }
    }
  }
}

// Few rows: one wavefront per 16 rows and 16 targets, its weights straight
// from memory, four chunks of both operands in flight; no LDS, no barrier.
__global__ __launch_bounds__(64) void k_regrid_few(RegridArgs a) {
  const int n_tile = (a.n_target + 15) / 16;
  const int tile = blockIdx.x % n_tile, rt = blockIdx.x / n_tile, chan = blockIdx.y;
  const int lane = threadIdx.x, m = lane & 15, g = lane >> 4;
  const int rows = a.rows_per_chan, n_chunk = a.m_ns / 32, rmask = (1 << a.log2_r) - 1;
  auto grow = [&](int r) -> int64_t { return ((int64_t)(r >> a.log2_r) * a.n_chan + chan) * (rmask + 1) + (r & rmask); };
  const int r = rt * 16 + m;
  const float* const arow[1] = {a.in + grow(r < rows ? r : 0) * a.m_ns + 4 * g};
  const u32x4* const wt = reinterpret_cast<const u32x4*>(a.w) +
                          ((int64_t)chan * (a.n_target_pad / 16) + tile) * n_chunk * 192;
  const int step = n_chunk < 4 ? n_chunk : 4;
  // terms of hi x hi, then the two pairs and the three smallest: three chains
  f32x4 acc[1][1] = {{f32x4{0.f, 0.f, 0.f, 0.f}}};
  f32x4 s1 = acc[0][0], s2 = acc[0][0];
#pragma unroll 1
  for (int k0 = 0; k0 < n_chunk; k0 += step) {
    f32x4 v[4][2];
    u32x4 w[4][3];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int kc = k0 + (k < step ? k : 0);
#pragma unroll
      for (int t = 0; t < 3; ++t) w[k][t] = wt[kc * 192 + t * 64 + lane];
#pragma unroll
      for (int h = 0; h < 2; ++h) v[k][h] = *reinterpret_cast<const f32x4*>(arow[0] + 32 * kc + 16 * h);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k >= step) break;
      u32x4 at[3];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t h, mid, lo;
        split3(v[k][q >> 1][2 * (q & 1)], v[k][q >> 1][2 * (q & 1) + 1], h, mid, lo);
        at[0][q] = h;
        at[1][q] = mid;
        at[2][q] = lo;
      }
      s2 = mfma_bf16(at[1], w[k][1], s2);
      s1 = mfma_bf16(at[0], w[k][1], s1);
      acc[0][0] = mfma_bf16(at[0], w[k][0], acc[0][0]);
      s2 = mfma_bf16(at[0], w[k][2], s2);
      s1 = mfma_bf16(at[1], w[k][0], s1);
      s2 = mfma_bf16(at[2], w[k][0], s2);
    }
  }
  acc[0][0] = acc[0][0] + (s1 + s2);
  float bad = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float v = acc[0][0][i];
    bad = fabsf(v) < 0x1p-90f && v != 0.f ? 1.f : fmaf(v, 0.f, bad);
  }
  if (!__all(bad == 0.f)) regrid_f32<1, 1>(arow, wt, 0, 1, 1, n_chunk, lane, acc);

  // acc[i]: row 16 rt + 4 g + i, target 16 tile + m
  const int t = 16 * tile + m;
  if (a.wew) {
    // rows [0, 8) and [8, 16): lane group g holds E-W beams 4 (g & 1) .. + 3 of (block, pol group) g >> 1
    const int grp_row = rt * 16 + 8 * (g >> 1), gi = grp_row >> 3;
    const int blk = gi / a.n_pg, pg = gi - blk * a.n_pg;
    const f32x4 we = *reinterpret_cast<const f32x4*>(a.wew + ((int64_t)chan * a.n_target_pad + t) * 8 + 4 * (g & 1));
    float part = we[0] * acc[0][0][0];
    part = fmaf(we[1], acc[0][0][1], part);
    part = fmaf(we[2], acc[0][0][2], part);
    part = fmaf(we[3], acc[0][0][3], part);
    part += __shfl_xor(part, 16);
    if (grp_row < rows && (g & 1) == 0 && t < a.n_target)
      a.out[(((int64_t)blk * a.n_chan + chan) * a.n_pg + pg) * a.n_target + t] = part;
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int ro = rt * 16 + 4 * g + i;
    if (ro < rows && t < a.n_target) a.out[grow(ro) * a.n_target + t] = acc[0][0][i];
  }
}

// Compact-kernel regridding (K taps per target): an HBM-bound gather.  A
// 256-thread workgroup stages kTapRows rows (all M beams) of one channel in LDS with
// float4 loads; each thread then takes targets t = tid, tid + 256, ... and
// forms sum_j tw[j][t] I[row][(first[t] + j) mod M] for those rows, writing
// each row's targets contiguously.
// rows per workgroup of the compact-tap kernel: 8 rows (16 KB of LDS at
// M = 512) let ten workgroups share a compute unit; 16 rows (32 KB, five
// workgroups) left the loads of one workgroup less to overlap with and
// were 10% slower at the CHIME shape, 4 rows no faster
constexpr int kTapRows = 8;

template <int K>
__global__ __launch_bounds__(256) void k_regrid_taps(RegridArgs a) {
  constexpr int RT = kTapRows;
  __shared__ __attribute__((aligned(16))) float lds[RT * 512];
  const int tid = threadIdx.x, chan = blockIdx.y;
  const int m = a.m_ns, mv = m >> 2;
  const int r0 = blockIdx.x * RT;
  const int nr = min(RT, a.rows_per_chan - r0);
  const int lr = a.log2_r, rmask = (1 << lr) - 1;
  auto grow = [&](int r) -> int64_t { return ((int64_t)(r >> lr) * a.n_chan + chan) * (1 << lr) + (r & rmask); };
  for (int idx = tid; idx < nr * mv; idx += 256) {
    const int rr = idx / mv, c4 = idx - rr * mv;
    *reinterpret_cast<f32x4*>(&lds[rr * m + 4 * c4]) =
        *reinterpret_cast<const f32x4*>(a.in + grow(r0 + rr) * m + 4 * c4);
  }
  __syncthreads();
  const int T = a.n_target;
  for (int t = tid; t < T; t += 256) {
    const int f = a.first[(int64_t)chan * T + t];
    float w[K];
    int ix[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      w[j] = a.tw[((int64_t)chan * K + j) * T + t];
      ix[j] = (f + j) & (m - 1);
    }
    for (int rr = 0; rr < nr; ++rr) {
      const float* row = &lds[rr * m];
      float acc = 0.f;
#pragma unroll
      for (int j = 0; j < K; ++j) acc = fmaf(w[j], row[ix[j]], acc);
      a.out[grow(r0 + rr) * T + t] = acc;
    }
  }
}

template <int W, int RT, int TG, int KS, bool ONE = false>
hipError_t launch_rt(const RegridArgs& a, hipStream_t s) {
  constexpr int RG = W / TG;
  const int64_t n_task = (int64_t)((a.rows_per_chan + 16 * RT * RG - 1) / (16 * RT * RG)) *
                         (a.n_target_pad / (TG == 2 ? 256 : 64)) * a.n_chan;
  if (n_task > 0x7FFFFFF0) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)((n_task + 7) / 8 * 8)), threads(64 * W);
  if (a.wew) hipLaunchKernelGGL((k_regrid<W, RT, TG, KS, ONE, true>), grid, threads, 0, s, a);
  else hipLaunchKernelGGL((k_regrid<W, RT, TG, KS, ONE, false>), grid, threads, 0, s, a);
  return hipGetLastError();
}

}  // namespace

// Targets are padded to the workgroup's target tile: 64 for up to 64
// targets, else a multiple of 256.
int regrid_target_pad(int n_target) {
  return n_target <= 64 ? 64 : (n_target + 255) / 256 * 256;
}

size_t regrid_weight_bytes(int n_chan, int n_target, int m) {
  return (size_t)n_chan * regrid_target_pad(n_target) * m * 6;
}

hipError_t launch_regrid_weights(uint32_t* w, const double* dl, const double* sin_t, const double* coef, int n_chan,
                                 int n_target, int n, int m, hipStream_t s) {
  const int pad = regrid_target_pad(n_target);
  const int64_t total = (int64_t)n_chan * pad * (m / 2);
  hipLaunchKernelGGL(k_regrid_weights, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, w, dl, sin_t, coef,
                     n_chan, n_target, pad, n, m);
  return hipGetLastError();
}

hipError_t launch_regrid_ew_weights(float* w, const double* dl, const double* dircos_ew, int n_chan, int n_target,
                                    int n, int m, hipStream_t s) {
  const int pad = regrid_target_pad(n_target);
  const int64_t total = (int64_t)n_chan * pad * m;
  hipLaunchKernelGGL(k_regrid_ew_weights, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, w, dl, dircos_ew,
                     n_chan, n_target, pad, n, m);
  return hipGetLastError();
}

hipError_t launch_regrid_tap_table(int* first, float* tw, const double* dl, const double* sin_t, const double* coef,
                                   int n_chan, int n_target, int k, int n, int m, hipStream_t s) {
  const int64_t total = (int64_t)n_chan * k * n_target;
  hipLaunchKernelGGL(k_regrid_tap_table, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, first, tw, dl, sin_t,
                     coef, n_chan, n_target, k, n, m);
  return hipGetLastError();
}

hipError_t launch_regrid(const RegridArgs& a_in, hipStream_t s) {
  RegridArgs a = a_in;
  if (a.m_ns < 32 || (a.m_ns & (a.m_ns - 1))) return hipErrorNotSupported;
  const int r_blk = a.n_pg * a.m_ew;
  if (r_blk <= 0 || (r_blk & (r_blk - 1))) return hipErrorNotSupported;
  a.log2_r = 0;
  while ((1 << a.log2_r) < r_blk) ++a.log2_r;
  const int64_t rows = a.n_blk * r_blk;
  if (rows == 0) return hipSuccess;
  if (rows > 0x7FFFFF00LL || a.n_chan > 65535) return hipErrorInvalidConfiguration;
  a.rows_per_chan = (int)rows;
  if (a.n_taps > 0) {
    if (a.n_taps > kRegridMaxTaps || a.m_ns > 512) return hipErrorNotSupported;
    const dim3 g((unsigned)((rows + kTapRows - 1) / kTapRows), (unsigned)a.n_chan);
    switch (a.n_taps) {
      case 1: hipLaunchKernelGGL(k_regrid_taps<1>, g, dim3(256), 0, s, a); break;
      case 2: hipLaunchKernelGGL(k_regrid_taps<2>, g, dim3(256), 0, s, a); break;
      case 3: hipLaunchKernelGGL(k_regrid_taps<3>, g, dim3(256), 0, s, a); break;
      case 4: hipLaunchKernelGGL(k_regrid_taps<4>, g, dim3(256), 0, s, a); break;
      case 5: hipLaunchKernelGGL(k_regrid_taps<5>, g, dim3(256), 0, s, a); break;
      case 6: hipLaunchKernelGGL(k_regrid_taps<6>, g, dim3(256), 0, s, a); break;
      case 7: hipLaunchKernelGGL(k_regrid_taps<7>, g, dim3(256), 0, s, a); break;
      default: hipLaunchKernelGGL(k_regrid_taps<8>, g, dim3(256), 0, s, a); break;
    }
    return hipGetLastError();
  }
  if (a.wew && a.m_ew != 8) return hipErrorNotSupported;
  const bool wide = a.n_target_pad > 64;
  // Few (row tile, target tile)s, eight wavefronts per CU or less: one wavefront
  // each without a workgroup's barriers; 64 rows in each of 16 channels, 60
  // targets, M = 512: 10.1 us against 15.7 (and 13.3 on the FP32 instructions).
  const int64_t few = (rows + 15) / 16 * ((a.n_target + 15) / 16) * a.n_chan;
  if (few <= 2048) {
    hipLaunchKernelGGL(k_regrid_few, dim3((unsigned)(few / a.n_chan), (unsigned)a.n_chan), dim3(64), 0, s, a);
    return hipGetLastError();
  }
  // 128 rows to a workgroup, 64 where that leaves CUs without one.  M = 32 is a
  // single chunk: one buffer, and no loads ahead of it.
  const int64_t wgs = (rows + 127) / 128 * (wide ? a.n_target_pad / 256 : 1) * a.n_chan;
  if (a.m_ns == 32) {
    if (wide) return launch_rt<8, 1, 2, 1, true>(a, s);
    return wgs >= 512 ? launch_rt<4, 2, 1, 1, true>(a, s) : launch_rt<4, 1, 1, 1, true>(a, s);
  }
  // 256 targets and 98 KB of LDS: sixteen wavefronts in the one workgroup that a
  // CU holds took 196 us where eight with two row tiles each took 215 (128
  // blocks, 64 channels, 256 pointings, M = 512)
  if (wide) return wgs >= 256 ? launch_rt<16, 1, 2, 1>(a, s) : launch_rt<8, 1, 2, 1>(a, s);
  if (wgs >= 256) return launch_rt<8, 1, 1, 1>(a, s);
  return a.m_ns < 128 ? launch_rt<4, 1, 1, 1>(a, s) : launch_rt<4, 1, 1, 2>(a, s);
}

}  // namespace fftbf
