// Tied-array beams from stored complex FFT beams, m_ns = 64 ... 512 (gfx950).
//
// Per (pointing p, sample t, channel, polarisation) the interpolation of
// k_tied.hip is a complex product over the N-S beams of each E-W beam,
//   Z[p][(t, e)] = sum_A c_A(y_ns,p) B[t][e][A],   B_p[t] = sum_e c_e(y_ew,p) Z[p][(t, e)].
// It runs on v_mfma_f32_16x16x32_bf16 with both operands as three BF16 terms
// (dev_bf16.h: FP32 operands, FP32 accumulation, six products): rows = 16
// pointings, columns = 4 samples x 4 E-W beams, K = 16 beams A as pairs
// (c_r, c_i).  Re Z takes the data pairs (b_r, -b_i) and Im Z the pairs
// (b_i, b_r), so the weights are held once.  Of the beams 16 kc + .. of chunk
// kc, lane group g takes A = 2 g, 2 g + 1, 8 + 2 g and 9 + 2 g: its two
// 16-byte loads are contiguous with its neighbours'.
//
// The weights of PT tiles of 16 pointings are generated once per workgroup in
// FP64 and stay in LDS, in the order the lanes read them; every wavefront
// walks its own output units (blocks of the intensity, or quads of samples)
// and reads, splits and multiplies each beam once for all PT tiles.
//
// 4 x 64, 32 channels, 2 polarisations, 2048 samples, 48 pointings: 537 MB of
// beams in 168 us (3.2 TB/s); the same contraction on v_mfma_f32_16x16x4_f32,
// one tile of 16 pointings per workgroup, took 404 us, bound by the FP32
// matrix rate (179 us) and by reading the beams three times.  The products
// take about 70 us here and the reads about 110: neither fills its unit, the
// splits (14 instructions per complex value) run between them.  Each chunk's
// products are summed by themselves before they join the running sum: 15 us,
// and errors against 64 bits a third of the FP32 instructions' (2-norm of the
// beams 0.84e-7 against 2.3e-7 at M = 128, 1.2e-7 against 4.4e-7 at 512; in one
// chain 2.2e-7 and 3.6e-7, larger than the FP32 instructions' on some inputs).

#include "dev_bf16.h"
#include "dev_common.h"
#include "kernels.h"

namespace fftbf {

namespace {

constexpr int kTsWaves = 8;

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// sum over the lane's quad
__device__ __forceinline__ float quad_sum(float v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  return v;
}

// (1/m) sum_{a<n} z^a for |z| = 1, n a power of two: (1 + z)(1 + z^2)(1 + z^4) ...
__device__ __forceinline__ void geom(double zr, double zi, int n, double inv_m, float* wr, float* wi) {
  double ar = 1.0 + zr, ai = zi;
  for (int k = 2; k < n; k <<= 1) {
    const double t = zr * zr - zi * zi;
    zi = 2.0 * zr * zi;
    zr = t;
    const double fr = 1.0 + zr;
    const double q = ar * fr - ai * zi;
    ai = ar * zi + ai * fr;
    ar = q;
  }
  *wr = (float)(ar * inv_m);
  *wi = (float)(ai * inv_m);
}

template <int M, int PT>
struct TsLds {
  u32x4 w[PT][M / 16][3][64];      // [tile][chunk][term][lane]: 4 pairs (c_r, c_i)
  float2 ew[PT * 16][4];           // c_e
  double2 ph[PT * 16];             // e^{-2 pi i y_ns}
  float part[kTsWaves][PT * 16];   // sums of the wavefronts that share a unit
};

// One output unit of the wavefront: `unit` samples from u * unit of
// polarisation group pg, of which it takes the quads sub, sub + split, ...;
// the sums go to `part` if the unit is split, else to the output.
// CPLX: complex output (units of one quad).  F32: the products on
// v_mfma_f32_16x16x4_f32.
// Returns whether every sum was finite and, for complex output, none was below
// 2^-90 (BF16 operands below 2^-126 count as zero, so there the low terms of
// the beams are lost; an intensity of such beams is zero in FP32 either way).
// The sums of a sample whose beams are all zero are right as they are: dead
// channels and zero-filled gaps cost no second pass (26 us against 44 to 52).
template <int M, int PT, bool CPLX, bool F32>
__device__ __forceinline__ bool tied_unit(const TiedArgs& a, const TsLds<M, PT>& lds, int lane, int64_t u, int unit,
                                          int pg, int chan, int cs, int p0, int sub, int split, float* part) {
  constexpr int NC = M / 16;
  const int n = lane & 15, g = lane >> 4;
  const int e = n & 3, s = n >> 2;
  const int pol_lo = a.pol_sum && !CPLX ? 0 : pg;
  const int pol_hi = a.pol_sum && !CPLX ? a.n_pol : pg + 1;
  const int64_t tstride = (int64_t)a.n_chan * a.n_pol * 4 * M;      // complex values per sample
  const float* beams = reinterpret_cast<const float*>(a.beams);
  auto quad_ptr = [&](int pol, int q) {
    const int64_t t = u * unit + q + s;
    const int64_t tc = t < a.n_time ? t : a.n_time - 1;
    return beams + 2 * (tc * tstride + (((int64_t)chan * a.n_pol + pol) * 4 + e) * M + 2 * g);
  };
  f32x4 acc[PT];
#pragma unroll
  for (int pt = 0; pt < PT; ++pt) acc[pt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float bad = 0.f;
  uint32_t any = 0;                // bits of the lane's beams
  constexpr int D = 2;             // chunks loaded ahead
  f32x4 ring[D + 1][2];
  static_assert(NC % 4 == 0, "chunks");
  const float* bp = quad_ptr(pol_lo, 4 * sub);
#pragma unroll
  for (int k = 0; k < D; ++k)
#pragma unroll
    for (int h = 0; h < 2; ++h) ring[k][h] = *reinterpret_cast<const f32x4*>(bp + 32 * k + 16 * h);

  for (int pol = pol_lo; pol < pol_hi; ++pol) {
    for (int q = 4 * sub; q < unit; q += 4 * split) {
      // the quad after this one (past the unit: this one again, cached)
      const float* bn = q + 4 * split < unit ? quad_ptr(pol, q + 4 * split)
                        : pol + 1 < pol_hi   ? quad_ptr(pol + 1, 4 * sub)
                                             : bp;
      f32x4 zr[PT], zi[PT];
#pragma unroll
      for (int pt = 0; pt < PT; ++pt) zr[pt] = zi[pt] = f32x4{0.f, 0.f, 0.f, 0.f};
      // (whole quads unrolled spill where four wavefronts share a SIMD, and with
      // complex output four chunks are slower as well; as it
      // is three and four tiles of pointings still spill 24 to 64 bytes a lane,
      // nearly all outside the innermost loop)
      constexpr int UN = NC > 4 ? (CPLX ? 2 : PT * M > 384 ? 8 : 4) : NC / 2;
#pragma unroll 1
      for (int k0 = 0; k0 < NC; k0 += UN) {
#pragma unroll
        for (int ku = 0; ku < UN; ++ku) {
          const int kc = k0 + ku;
          // the weights stay in LDS: without this they are read ahead of the
          // loops and held in (spilled) registers
          asm volatile("" : "+v"(lane));
          const float* np = kc + D < NC ? bp + 32 * (kc + D) : bn + 32 * (kc + D - NC);
          f32x4 v[2] = {ring[0][0], ring[0][1]};
          if constexpr (CPLX && !F32) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const u32x4 x = __builtin_bit_cast(u32x4, v[h]);
              any |= x[0] | x[1] | x[2] | x[3];
            }
          }
#pragma unroll
          for (int k = 0; k + 1 < D; ++k) {
            ring[k][0] = ring[k + 1][0];
            ring[k][1] = ring[k + 1][1];
          }
#pragma unroll
          for (int h = 0; h < 2; ++h) ring[D - 1][h] = *reinterpret_cast<const f32x4*>(np + 16 * h);
          if constexpr (F32) {
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) {
              const u32x4 w0 = lds.w[pt][kc][0][lane], w1 = lds.w[pt][kc][1][lane], w2 = lds.w[pt][kc][2][lane];
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const float cr = (bf16_lo(w0[j]) + bf16_lo(w1[j])) + bf16_lo(w2[j]);
                const float ci = (bf16_hi(w0[j]) + bf16_hi(w1[j])) + bf16_hi(w2[j]);
                const float br = v[j >> 1][2 * (j & 1)], bi = v[j >> 1][2 * (j & 1) + 1];
                zr[pt] = __builtin_amdgcn_mfma_f32_16x16x4f32(cr, br, zr[pt], 0, 0, 0);
                zr[pt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ci, -bi, zr[pt], 0, 0, 0);
                zi[pt] = __builtin_amdgcn_mfma_f32_16x16x4f32(cr, bi, zi[pt], 0, 0, 0);
                zi[pt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ci, br, zi[pt], 0, 0, 0);
              }
            }
          } else {
            u32x4 dr[3], di[3];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              float r = v[j >> 1][2 * (j & 1)], i = v[j >> 1][2 * (j & 1) + 1];
#pragma unroll
              for (int t = 0; t < 3; ++t) {
                const uint32_t w = pack_bf16(i, r);
                di[t][j] = w;                        // (b_i, b_r)
                dr[t][j] = pack_bf16(r, -i);         // (b_r, -b_i)
                if (t < 2) {
                  i -= bf16_lo(w);
                  r -= bf16_hi(w);
                }
              }
            }
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) {
              const u32x4 w[3] = {lds.w[pt][kc][0][lane], lds.w[pt][kc][1][lane], lds.w[pt][kc][2][lane]};
              // the chunk's products by themselves: two roundings of the running sum's size, not six
              const f32x4 none = {0.f, 0.f, 0.f, 0.f};
              const f32x4 cr = mfma_bf16x3(w, dr, none), ci = mfma_bf16x3(w, di, none);
              zr[pt] += cr;
              zi[pt] += ci;
            }
          }
        }
      }
      // E-W weights, the sum over the column quad's four E-W beams, |B_p|^2
      const int64_t t = u * unit + q + s;
      // whether the lane's sample holds anything: columns 4 s ... 4 s + 3 of every lane group
      const bool live = !CPLX || F32 || (__ballot((any & 0x7FFFFFFFu) != 0) & (0x000F000F000F000Full << (4 * s))) != 0;
#pragma unroll
      for (int pt = 0; pt < PT; ++pt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float2 c = lds.ew[pt * 16 + 4 * g + i][e];
          const cf b0 = cmul(cf{zr[pt][i], zi[pt][i]}, cf{c.x, c.y});
          const cf b{quad_sum(b0.r), quad_sum(b0.i)};
          if constexpr (CPLX) {
            const int p = p0 + pt * 16 + 4 * g + i;
            if (e == 0 && t < a.n_time && p < a.n_point)
              static_cast<float2*>(a.out)[((t * a.n_chan_sub + cs) * a.n_pol + pol) * (int64_t)a.n_point + p] =
                  make_float2(b.r, b.i);
            bad = live && fmaxf(fabsf(b.r), fabsf(b.i)) < 0x1p-90f ? 1.f : fmaf(b.r, 0.f, fmaf(b.i, 0.f, bad));
          } else {
            acc[pt][i] = cnorm_acc(b, acc[pt][i]);
          }
        }
      bp = bn;
    }
  }
  if constexpr (!CPLX) {
    const int n_pg = a.pol_sum ? 1 : a.n_pol;
    float* o = static_cast<float*>(a.out) + ((u * a.n_chan_sub + cs) * n_pg + pg) * (int64_t)a.n_point;
#pragma unroll
    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v = acc[pt][i];
        v += __shfl_xor(v, 4);
        v += __shfl_xor(v, 8);
        const int p = p0 + pt * 16 + 4 * g + i;
        if (n == 0) {
          if (split > 1) part[pt * 16 + 4 * g + i] = v;
          else if (p < a.n_point) o[p] = v;
        }
        bad = fmaf(v, 0.f, bad);
      }
  }
  return __all(bad == 0.f);
}

template <int M, int PT, bool CPLX>
__global__ __launch_bounds__(64 * kTsWaves) __attribute__((amdgpu_waves_per_eu(PT * M > 384 ? 2 : 4))) void k_tied_stored(TiedArgs a) {
  __shared__ TsLds<M, PT> lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_pt = (a.n_point + 16 * PT - 1) / (16 * PT);
  const int p0 = (int)(blockIdx.x % n_pt) * 16 * PT, run = blockIdx.x / n_pt;
  const int cs = blockIdx.y, chan = a.chan_lo + cs;
  const double dl_ew = a.dl[2 * chan], dl_ns = a.dl[2 * chan + 1];

  for (int i = tid; i < 16 * PT; i += 64 * kTsWaves) {
    const int p = min(p0 + i, a.n_point - 1);
    double sn, cs_;
    sincospi(-2.0 * (dl_ns * a.dircos[2 * p + 1]), &sn, &cs_);
    lds.ph[i] = make_double2(cs_, sn);
  }
  for (int i = tid; i < 64 * PT; i += 64 * kTsWaves) {
    const int p = min(p0 + (i >> 2), a.n_point - 1);
    double sn, cs_;
    sincospi(2.0 * (0.25 * (i & 3) - dl_ew * a.dircos[2 * p]), &sn, &cs_);
    float2 c;
    geom(cs_, sn, 4, 0.25, &c.x, &c.y);
    lds.ew[i >> 2][i & 3] = c;
  }
  __syncthreads();
  {
    // the thread's beam A stays the same over its pointings (M divides the workgroup)
    static_assert((64 * kTsWaves) % M == 0, "one beam per thread");
    const int A = tid % M;
    double ws, wc;
    sincospi(2.0 * (double)A / (double)M, &ws, &wc);
    const int kc = A >> 4, gg = (A & 7) >> 1, j = 2 * ((A >> 3) & 1) + (A & 1);
    for (int p = tid / M; p < 16 * PT; p += 64 * kTsWaves / M) {
      const double2 ph = lds.ph[p];
      float wr, wi;
      geom(wc * ph.x - ws * ph.y, wc * ph.y + ws * ph.x, a.n_ns, 1.0 / M, &wr, &wi);
      uint32_t h, m, l;
      split3(wr, wi, h, m, l);
      u32x4(*w)[64] = lds.w[p >> 4][kc];
      reinterpret_cast<uint32_t*>(&w[0][gg * 16 + (p & 15)])[j] = h;
      reinterpret_cast<uint32_t*>(&w[1][gg * 16 + (p & 15)])[j] = m;
      reinterpret_cast<uint32_t*>(&w[2][gg * 16 + (p & 15)])[j] = l;
    }
  }
  __syncthreads();

  const int n_pg = a.pol_sum && !CPLX ? 1 : a.n_pol;
  const int unit = CPLX ? 4 : a.block;
  const int64_t n_unit = (a.n_time + unit - 1) / unit * n_pg;
  const int64_t u0 = (int64_t)run * a.run_units;
  const int64_t u1 = u0 + a.run_units < n_unit ? u0 + a.run_units : n_unit;
  const int split = a.unit_split, slot = wave / split, sub = wave % split, slots = kTsWaves / split;
  for (int64_t ub = u0; ub < u1; ub += slots) {
    const int64_t u = ub + slot;
    const int64_t tu = u / n_pg;
    const int pg = (int)(u - tu * n_pg);
    if (u < u1 && !tied_unit<M, PT, CPLX, false>(a, lds, lane, tu, unit, pg, chan, cs, p0, sub, split, lds.part[wave]))
      tied_unit<M, PT, CPLX, true>(a, lds, lane, tu, unit, pg, chan, cs, p0, sub, split, lds.part[wave]);
    if (split > 1) {
      __syncthreads();
      if (u < u1 && sub == 0 && lane < 16 * PT && p0 + lane < a.n_point) {
        float v = lds.part[wave][lane];
        for (int k = 1; k < split; ++k) v += lds.part[wave + k][lane];
        static_cast<float*>(a.out)[((tu * a.n_chan_sub + cs) * n_pg + pg) * (int64_t)a.n_point + p0 + lane] = v;
      }
      __syncthreads();
    }
  }
}

template <int M, int PT>
hipError_t launch_mp(TiedArgs a, hipStream_t s) {
  const int n_pt = (a.n_point + 16 * PT - 1) / (16 * PT);
  const int n_pg = a.pol_sum && !a.complex_out ? 1 : a.n_pol;
  const int unit = a.complex_out ? 4 : a.block;
  const int64_t n_unit = (a.n_time + unit - 1) / unit * n_pg;
  const int64_t base = (int64_t)n_pt * a.n_chan_sub;
  // With fewer units than the chip has wavefronts in flight (two workgroups of
  // eight per CU), two or four wavefronts share a unit's quads of samples: 256
  // units of 16 samples at m_ns = 512 and 8 pointings took 79 us unsplit and 37 split.
  a.unit_split = 1;
  while (a.unit_split < 4 && 8 * a.unit_split <= unit && n_unit * base * a.unit_split < 4096) a.unit_split *= 2;
  const int slots = kTsWaves / a.unit_split;
  // The number of runs that ends soonest: rounds of resident workgroups times a
  // run's turns of its wavefronts, and the weights that each workgroup makes
  // first (about a third of a turn of whole units).  Only the most runs that fit
  // a number of rounds are worth a look.
  constexpr int kWgs = sizeof(TsLds<M, PT>) > 80 * 1024 ? 256 : 512;
  const int64_t max_runs = (n_unit + slots - 1) / slots;
  int64_t runs = 1;
  double best = 0.0;
  for (int k = 0; k < 5; ++k) {
    const int64_t rounds = (base + kWgs - 1) / kWgs + k;
    int64_t r = rounds * kWgs / base;
    if (r > max_runs) r = max_runs;
    const int64_t turns = ((n_unit + r - 1) / r + slots - 1) / slots;
    const double cost = (double)((base * r + kWgs - 1) / kWgs) * ((double)turns + 0.3 * a.unit_split);
    if (k == 0 || cost < best) {
      best = cost;
      runs = r;
    }
  }
  int64_t per = (n_unit + runs - 1) / runs;
  per = (per + slots - 1) / slots * slots;
  runs = (n_unit + per - 1) / per;
  if (per > 0x7FFFFFFF || n_pt * runs > 0x7FFFFFFF || a.n_chan_sub > 65535) return hipErrorInvalidConfiguration;
  a.run_units = (int)per;
  const dim3 grid((unsigned)(n_pt * runs), (unsigned)a.n_chan_sub), threads(64 * kTsWaves);
  if (a.complex_out) hipLaunchKernelGGL((k_tied_stored<M, PT, true>), grid, threads, 0, s, a);
  else hipLaunchKernelGGL((k_tied_stored<M, PT, false>), grid, threads, 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_tied_stored(const TiedArgs& a, hipStream_t s) {
  if (a.m_ew != 4 || a.n_ew != 4 || a.n_ns < 2 || (a.n_ns & (a.n_ns - 1)) ||
      (reinterpret_cast<uintptr_t>(a.beams) & 15) != 0)
    return hipErrorNotSupported;
  // Tiles of pointings per workgroup: as many as leave LDS for two workgroups
  // per CU (one at m_ns >= 256, where the weights take 50 KB a tile), fewer
  // where that would leave more of the last workgroup's tiles empty.
  const int pt = (a.n_point + 15) / 16;
  switch (a.m_ns) {
    case 64:
      if (pt <= 2) return pt == 1 ? launch_mp<64, 1>(a, s) : launch_mp<64, 2>(a, s);
      return pt == 3 || pt == 5 || pt == 6 ? launch_mp<64, 3>(a, s) : launch_mp<64, 4>(a, s);
    case 128:
      if (pt == 1) return launch_mp<128, 1>(a, s);
      return pt == 2 || pt == 4 ? launch_mp<128, 2>(a, s) : launch_mp<128, 3>(a, s);
    case 256: return pt == 1 ? launch_mp<256, 1>(a, s) : launch_mp<256, 2>(a, s);
    case 512: return launch_mp<512, 1>(a, s);
    default: return hipErrorNotSupported;
  }
}

}  // namespace fftbf
