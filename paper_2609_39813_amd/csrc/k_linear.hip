// E5M2-gradient Linear backward: residual operand planes of the policy biases and the
// coupling statistic between the two uses of a rounded incoming gradient.
#include "k_linear.h"

namespace bsp {

// Mean over the K trials of a use's new roundings minus the incoming gradient:
// E = s sign (lo + n_up step / K) - dY = s sign (mi K + n_up) step / K - dY, evaluated in
// fp64 (the integer and the power-of-two step are exact) and rounded once to fp32.
__device__ __forceinline__ float resid_value(float g, uint32_t n_up, int K, F8 f, float s, double rs) {
  const float y = div_scale(g, rs);
  const Bracket b = f8_bracket(fminf(fabsf(y), f.fmax), f);
  const double num = ((double)b.mi * K + (double)n_up) * (double)f8_step(b);
  double mv = num / K;
  if (signbit(y)) mv = -mv;
  return (float)((double)s * mv - (double)g);
}

// The residual planes of one use, the K new roundings drawn in the same pass (DRAW; else their
// counts are read): a block covers 64 rows x 64 columns, a thread 4 consecutive rows x 4 columns
// (one Philox call per row and trial). Bound by the draws; the planes' writes run under other
// blocks' draws. 16384 x 8192, 64 trials: 3.1 ms per use (one layout or both); counted by one kernel and
// formed by another, 2.80 + 0.51 ms. HI: the tensor has 2^32 or more groups of four elements (else the
// high counter word is a constant zero).
// The transposed planes pass through an LDS tile per term, a thread's four rows of a column as one
// 8-byte store; tile rows are 34 words apart, the words of row r rotated by 2 ((r >> 4) & 3), so
// that store and read passes are free of bank conflicts.
__device__ __forceinline__ int rp_word(int r, int w) { return r * 34 + ((w + 2 * ((r >> 4) & 3)) & 31); }

// Four waves per SIMD (128 registers) for the Philox latency.
template <bool DRAW, bool HI>
__global__ __launch_bounds__(256, 4) void resid_planes_kernel(ResidArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t tile[3][64 * 34];
  const int cg = threadIdx.x & 15, rg = threadIdx.x >> 4;
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  const int64_t tb = r0 + 4 * rg, cb = c0 + 4 * cg;  // first row, first column (n % 4 == 0)
  const float s = *a.scale;
  const double rs = 1.0 / (double)s;
  const bool v8 = ((uintptr_t)a.dY & 7) == 0;
  uint2 g2[4];  // four bf16 per row
  uint32_t cnt[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool ok = tb + i < a.M && cb < a.n;
    const u16* p = a.dY + (tb + i) * a.n + cb;
    g2[i] = make_uint2(0u, 0u);
    if (ok) {
      if (v8)
        g2[i] = *(const uint2*)p;
      else
        g2[i] = make_uint2((uint32_t)p[0] | ((uint32_t)p[1] << 16), (uint32_t)p[2] | ((uint32_t)p[3] << 16));
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) cnt[i][q] = 0;
    if (!DRAW && ok) {
      const uint2 c = *(const uint2*)(a.counts + (tb + i) * a.n + cb);
      cnt[i][0] = c.x & 0xFFFFu, cnt[i][1] = c.x >> 16, cnt[i][2] = c.y & 0xFFFFu, cnt[i][3] = c.y >> 16;
    }
  }
  auto elem = [&](int i, int q) {
    const uint32_t w = q < 2 ? g2[i].x : g2[i].y;
    return __uint_as_float(q & 1 ? w & 0xFFFF0000u : w << 16);
  };
  if constexpr (DRAW) {
    uint32_t F[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        F[i][q] = f8_bracket(fminf(fabsf(div_scale(elem(i, q), rs)), a.f.fmax), a.f).F;
        asm volatile("" : "+v"(F[i][q]));
      }
    for (int k0 = 0; k0 < a.K; k0 += 4) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int k = k0 + t;
        if (k >= a.K) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint64_t grp = (uint64_t)((tb + i) * a.n + cb) >> 2;
          const Philox4 p = philox4x32_10((uint32_t)grp, HI ? (uint32_t)(grp >> 32) : 0u, (uint32_t)(k + a.trial0), a.use,
                                          (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
#pragma unroll
          for (int q = 0; q < 4; ++q) cnt[i][q] += sr_up(F[i][q], philox_word(p, q));
        }
      }
    }
  }
  u16 o[3][4][4];  // [term][row][column]
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      split3(resid_value(elem(i, q), cnt[i][q], a.K, a.f, s, rs), o[0][i][q], o[1][i][q], o[2][i][q]);
    if (a.rows[0] && tb + i < a.M && cb < a.n) {
#pragma unroll
      for (int p = 0; p < 3; ++p)
        *(uint2*)(a.rows[p] + (tb + i) * a.n + cb) =
            make_uint2((uint32_t)o[p][i][0] | ((uint32_t)o[p][i][1] << 16),
                       (uint32_t)o[p][i][2] | ((uint32_t)o[p][i][3] << 16));
    }
  }
  if (!a.cols[0]) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int wd = rp_word(4 * cg + q, 2 * rg);
#pragma unroll
    for (int p = 0; p < 3; ++p)
      *(uint2*)&tile[p][wd] = make_uint2((uint32_t)o[p][0][q] | ((uint32_t)o[p][1][q] << 16),
                                         (uint32_t)o[p][2][q] | ((uint32_t)o[p][3][q] << 16));
  }
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int ch = threadIdx.x + 256 * pass, cc = ch >> 3, k8 = ch & 7;
    if (c0 + cc >= a.n) continue;
    const int w0 = rp_word(cc, 4 * k8), w1 = rp_word(cc, 4 * k8 + 2);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const uint2 x0 = *(const uint2*)&tile[p][w0], x1 = *(const uint2*)&tile[p][w1];
      *(uint4*)(a.cols[p] + (c0 + cc) * a.ldo + r0 + 8 * k8) = make_uint4(x0.x, x0.y, x1.x, x1.y);
    }
  }
}

bs_status launch_resid_planes(const ResidArgs& a, hipStream_t st) {
  if (a.n <= 0) return BS_OK;
  if ((a.n & 3) || (a.ldo & 63) || a.ldo < a.M) return BS_EINVAL;
  for (int p = 0; p < 3; ++p)
    if (((uintptr_t)a.rows[p] & 7) || ((uintptr_t)a.cols[p] & 15)) return BS_EINVAL;
  const int64_t rows = a.cols[0] ? a.ldo : a.M;
  if (rows <= 0) return BS_OK;
  const dim3 grid((unsigned)((a.n + 63) / 64), (unsigned)((rows + 63) / 64));
  ProfScope prof("fresh_count", st);
  if (a.counts)
    resid_planes_kernel<false, false><<<grid, 256, 0, st>>>(a);
  else if ((uint64_t)(round_up(a.M, 64) * a.n) >> 34)
    resid_planes_kernel<true, true><<<grid, 256, 0, st>>>(a);
  else
    resid_planes_kernel<true, false><<<grid, 256, 0, st>>>(a);
  BS_CHECK_LAUNCH();
  return BS_OK;
}

__global__ __launch_bounds__(256) void kappa_fixed_kernel(const u16* __restrict__ dY, const float* __restrict__ scale,
                                                          F8 f, int64_t n_el, const float* __restrict__ AW,
                                                          const float* __restrict__ XB, double* __restrict__ part) {
  const float s = *scale;
  const double rs = 1.0 / (double)s;
  double a0 = 0.0, b0 = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n_el; e += (int64_t)gridDim.x * 256) {
    const float g = bf16_to_f32(dY[e]);
    const float y = div_scale(g, rs);
    const Bracket b = f8_bracket(fminf(fabsf(y), f.fmax), f);
    double lo = (double)b.mi * (double)f8_step(b);
    if (signbit(y)) lo = -lo;
    const double r = (double)s * lo - (double)g;
    a0 += r * (double)AW[e];
    b0 += r * (double)XB[e];
  }
  __shared__ double red[2][4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  a0 = wave_sum_f64(a0);
  b0 = wave_sum_f64(b0);
  if (lane == 0) {
    red[0][w] = a0;
    red[1][w] = b0;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int i = threadIdx.x;
    part[(int64_t)blockIdx.x * 2 + i] = ((red[i][0] + red[i][1]) + red[i][2]) + red[i][3];
  }
}

__global__ void kappa_fixed_final(const double* __restrict__ part, int nblk, double* __restrict__ out) {
  if (threadIdx.x >= 2) return;
  double v = 0.0;
  for (int b = 0; b < nblk; ++b) v += part[b * 2 + threadIdx.x];
  out[threadIdx.x] = v;
}

bs_status launch_kappa_fixed(const u16* dY, const float* scale, int fmt, int64_t M, int64_t n, const float* AW,
                             const float* XB, double* part, double* out, hipStream_t st) {
  const int nblk = 1024;
  kappa_fixed_kernel<<<nblk, 256, 0, st>>>(dY, scale, f8_format(fmt), M * n, AW, XB, part);
  kappa_fixed_final<<<1, 64, 0, st>>>(part, nblk, out);
  BS_CHECK_LAUNCH();
  return BS_OK;
}

// one wave: trial sums of the block partials (blocks in order, per trial), then the mean
// of the per-trial products in trial order
__global__ void kappa_final_kernel(const double* __restrict__ fixed, const double* __restrict__ pa, int ia,
                                   const double* __restrict__ pb, int ib, int64_t nblk, int K,
                                   const float* __restrict__ scale, double* __restrict__ kappa) {
  __shared__ double prod[4096];
  const double s = *scale;
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    double sa = 0.0, sb = 0.0;
    const double* qa = pa + ((int64_t)k * 2 + ia) * nblk;
    const double* qb = pb + ((int64_t)k * 2 + ib) * nblk;
    for (int64_t b = 0; b < nblk; ++b) {
      sa += qa[b];
      sb += qb[b];
    }
    prod[k] = (fixed[0] + s * sa) * (fixed[1] + s * sb);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = 0.0;
    for (int k = 0; k < K; ++k) m += prod[k];
    *kappa = m / K;
  }
}

bs_status launch_kappa_final(const double* fixed, const double* pa, int ia, const double* pb, int ib, int64_t nblk,
                             int K, const float* scale, double* kappa, hipStream_t st) {
  if (K > 4096) return BS_EINVAL;
  kappa_final_kernel<<<1, 256, 0, st>>>(fixed, pa, ia, pb, ib, nblk, K, scale, kappa);
  BS_CHECK_LAUNCH();
  return BS_OK;
}

}  // namespace bsp
