// The paper's own normalization store (App. D.4): RMSNorm -> per-token b-bit uniform grid with
// stochastic rounding -> Linear, and the eight policies of its table (gain use first; the weight
// use may also read u_q + (u_f - u)). One new rounding u_f per trial feeds both uses.
//
// Per token t: s_t = fl32(max_j |u_tj| / M), M = 2^(b-1) - 1; y = fl32(u / s_t); a = min(|y|, M)
// (clamps counted); lo = floor(a), F = floor((a - lo) 2^32); the code rounds up iff R + F >= 2^32;
// u_q = fl32(q s_t). Every bias is a contraction (weight use) or an fp64 column sum (gain use) of
// a residual: e_U = u - u_q, e_e = mean_k u_f,k - u, e_N = mean_k u_f,k - u_q = e_U + e_e, where the mean
// over trials of the grid values is ((K - n) v_lo + n v_hi) / K from the element's up-count n.
#include <algorithm>

#include "bsp_kernels.h"
#include "k_fresh.h"
#include "k_norm.h"

#define BS_TRY(x)               \
  do {                          \
    const bs_status _s = (x);   \
    if (_s != BS_OK) return _s; \
  } while (0)

namespace bsp {

namespace {

struct GridBracket {
  float lo;     // floor(|y|), |y| clamped to M
  uint32_t F;   // floor(frac 2^32)
  bool neg;
  bool sat;
};

__device__ __forceinline__ GridBracket grid_bracket(float u, float s, float M) {
  GridBracket b;
  const float y = u / s;  // IEEE division (correctly rounded)
  const float a = fabsf(y);
  b.sat = a > M;
  const float ac = fminf(a, M);
  b.lo = floorf(ac);
  b.F = (uint32_t)((ac - b.lo) * 4294967296.0f);  // exact: ac - lo has at most 24 bits, < 1
  b.neg = signbit(y);
  return b;
}

// fl32(q s) of the code sign * m
__device__ __forceinline__ float grid_value(float m, bool neg, float s) {
#pragma clang fp contract(off)
  return (neg ? -m : m) * s;
}

// one wave per token: the step, the forward's codes (trial 0), u_q and e_U = u - u_q
__global__ __launch_bounds__(256) void grid_store_kernel(const float* __restrict__ u, int64_t T, int64_t d, int bits,
                                                         uint64_t seed, uint32_t use, int8_t* __restrict__ codes,
                                                         float* __restrict__ step, float* __restrict__ uq,
                                                         float* __restrict__ eU, bs_diag* __restrict__ diag) {
#pragma clang fp contract(off)  // e_U is u less the rounded q s, not a fused u - q s
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const float M = (float)((1 << (bits - 1)) - 1);
  const float* ur = u + t * d;
  float m = 0.0f;
  for (int64_t j = 4 * lane; j < d; j += 256) {
    const float4 v = *(const float4*)(ur + j);
    m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  const float s = m > 0.0f ? m / M : 1.0f;
  if (lane == 0) step[t] = s;
  uint32_t nsat = 0;
  for (int64_t j = 4 * lane; j < d; j += 256) {
    const float4 v = *(const float4*)(ur + j);
    const float uv[4] = {v.x, v.y, v.z, v.w};
    const Philox4 p = philox_group(seed, (uint64_t)(t * d + j) >> 2, 0u, use);
    const uint32_t R[4] = {p.w0, p.w1, p.w2, p.w3};
    float qv[4], ev[4];
    uint32_t cw = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const GridBracket b = grid_bracket(uv[r], s, M);
      nsat += b.sat ? 1u : 0u;
      const float mag = b.lo + (float)sr_up(b.F, R[r]);
      qv[r] = grid_value(mag, b.neg, s);
      ev[r] = (float)((double)uv[r] - (double)qv[r]);
      const int q = b.neg ? -(int)mag : (int)mag;
      cw |= ((uint32_t)(uint8_t)(int8_t)q) << (8 * r);
    }
    *(uint32_t*)(codes + t * d + j) = cw;
    *(float4*)(uq + t * d + j) = make_float4(qv[0], qv[1], qv[2], qv[3]);
    *(float4*)(eU + t * d + j) = make_float4(ev[0], ev[1], ev[2], ev[3]);
  }
  nsat = wave_sum_u32(nsat);
  if (lane == 0 && nsat) atomicAdd(&diag->n_saturated, nsat);
}

// up-counts of the new rounding over K trials (flat groups of 4 elements, k_fresh.h), then e_e =
// mean_k u_f,k - u (e_N = e_e + e_U, so the N bias is the sum of the R+e and U biases). 8192 x 1024,
// 256 trials: 740 us; one group per thread with every trial in its thread, 786 us.
template <int G, int TS>
__global__ __launch_bounds__(fresh_nt(TS)) void grid_fresh_kernel(const float* __restrict__ u,
                                                                  const float* __restrict__ step, int64_t T, int64_t d,
                                                                  int bits, uint64_t seed, uint32_t use, int K,
                                                                  float* __restrict__ eE) {
#pragma clang fp contract(off)  // the grid values are rounded
  const FreshBlock<G, TS> blk;
  const uint64_t ngroups = (uint64_t)(T * d) >> 2;
  const float M = (float)((1 << (bits - 1)) - 1);
  uint32_t F[G][4], cnt[G][4];
#pragma unroll
  for (int r = 0; r < G; ++r) {
    const uint64_t g = blk.group(r);
#pragma unroll
    for (int q = 0; q < 4; ++q) F[r][q] = 0;
    if (g < ngroups) {
      const float s = step[4 * g / d];
      const float4 v = *(const float4*)(u + 4 * g);
      const float uv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) F[r][q] = grid_bracket(uv[q], s, M).F;
    }
  }
  blk.count(F, cnt, K, 1, use, seed);
  uint2 n2[G];
  if (!blk.merge(cnt, n2)) return;
#pragma unroll
  for (int r = 0; r < G; ++r) {
    const uint64_t g = blk.group(r);
    if (g >= ngroups) continue;
    const float s = step[4 * g / d];
    const float4 v = *(const float4*)(u + 4 * g);
    const float uv[4] = {v.x, v.y, v.z, v.w};
    float o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t w = q < 2 ? n2[r].x : n2[r].y;
      const int n = (int)(q & 1 ? w >> 16 : w & 0xFFFFu);
      const GridBracket b = grid_bracket(uv[q], s, M);
      const double vlo = grid_value(b.lo, b.neg, s), vhi = grid_value(b.lo + 1.0f, b.neg, s);
      o[q] = (float)(((double)(K - n) * vlo + (double)n * vhi) / (double)K - (double)uv[q]);
    }
    *(float4*)(eE + 4 * g) = make_float4(o[0], o[1], o[2], o[3]);
  }
}

// gain use, fp64 column partials over token chunks of 256: [3][nchunk][d]
//   ref  sum z du;  R  sum (u/gain - z - eU/gain) du;  N  sum (u/gain - z + eE/gain) du
// rows per chunk of the gain use's column partial sums: T / 32 chunks (grid x) x d / 256 blocks
// (grid y); a lane takes 4 columns of its wave's 8 rows (16-byte loads, four rows in flight), the
// four waves' sums meet in LDS in wave order. 8192 x 1024: 35 us; one column and 32 rows per lane
// 61 us (few bytes in flight).
constexpr int GRID_GAIN_RT = 32;

__device__ __forceinline__ float4 load4(const float* p) { return *(const float4*)p; }
__device__ __forceinline__ float4 load4(const u16* p) {
  const uint2 v = *(const uint2*)p;
  return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16),
                     __uint_as_float(v.y & 0xFFFF0000u));
}

template <typename XT>
__global__ __launch_bounds__(256) void grid_gain_kernel(const XT* __restrict__ X, const float* __restrict__ rstd,
                                                        const float* __restrict__ gain, const float* __restrict__ u,
                                                        const float* __restrict__ du, const float* __restrict__ eU,
                                                        const float* __restrict__ eE, int64_t T, int64_t d,
                                                        double* __restrict__ part) {
#pragma clang fp contract(off)
  __shared__ double red[4][3][64][5];  // a lane's 4 columns and a pad word pair
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t j = (int64_t)blockIdx.y * 256 + 4 * lane;
  const int64_t c = blockIdx.x, nch = gridDim.x;
  const bool ok = j < d;  // d % 8 == 0
  const bool va = ((uintptr_t)X & (4 * sizeof(XT) - 1)) == 0 && ((uintptr_t)gain & 15) == 0;
  double acc[3][4] = {}, ig[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) ig[q] = ok ? 1.0 / (double)gain[j + q] : 0.0;
  const int64_t t0 = c * GRID_GAIN_RT + 8 * wave;
  if (ok) {
#pragma unroll 4
    for (int i = 0; i < 8; ++i) {
      const int64_t t = t0 + i;
      if (t >= T) break;
      const int64_t e = t * d + j;
      float4 xv;
      if (va)
        xv = load4(X + e);
      else
        xv = make_float4(load_f32(X, e), load_f32(X, e + 1), load_f32(X, e + 2), load_f32(X, e + 3));
      const float4 uv = load4(u + e), dv = load4(du + e), a = load4(eU + e), b = load4(eE + e);
      const float x4[4] = {xv.x, xv.y, xv.z, xv.w}, u4[4] = {uv.x, uv.y, uv.z, uv.w}, d4[4] = {dv.x, dv.y, dv.z, dv.w};
      const float a4[4] = {a.x, a.y, a.z, a.w}, b4[4] = {b.x, b.y, b.z, b.w};
      const float r = rstd[t];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double z = (double)(x4[q] * r), dd = d4[q], base = (double)u4[q] * ig[q] - z;
        acc[0][q] += z * dd;
        acc[1][q] += (base - (double)a4[q] * ig[q]) * dd;
        acc[2][q] += (base + (double)b4[q] * ig[q]) * dd;
      }
    }
  }
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) red[wave][p][lane][q] = acc[p][q];
  __syncthreads();
  // thread (column of the 256, each of the three sums)
  const int l = threadIdx.x >> 2, q = threadIdx.x & 3;
  const int64_t jo = (int64_t)blockIdx.y * 256 + threadIdx.x;
  if (jo >= d) return;
#pragma unroll
  for (int p = 0; p < 3; ++p)
    part[((int64_t)p * nch + c) * d + jo] = ((red[0][p][l][q] + red[1][p][l][q]) + red[2][p][l][q]) + red[3][p][l][q];
}

struct GridWs {
  float *u, *rstd, *du, *uq, *eU, *eE, *bias_rg, *bias_ng, *bias_w[2];  // weight biases: U, R+e
  u16 *dyT[3], *aT[3], *uq_rows[3], *wT[3], *dy_rows[3], *w_rows[3];
  double* gpart;
  float* gemm_part;
  int64_t gemm_part_cap;
};

GridWs carve_grid(Carver& c, int64_t T, int64_t d, int64_t n, bs_dtype wt, bs_dtype gt, bool want_y) {
  GridWs w{};
  const int64_t Tp = round_up(T > 0 ? T : 1, 64);
  const int nt = gt == BS_F32 ? 3 : 1, ntw = wt == BS_F32 ? 3 : 1;
  for (float** p : {&w.u, &w.du, &w.uq, &w.eU, &w.eE}) *p = c.take<float>(T * d);
  w.rstd = c.take<float>(T > 0 ? T : 1);
  for (int i = 0; i < nt; ++i) w.dyT[i] = c.take<u16>(n * Tp);
  for (int i = 0; i < 3; ++i) w.aT[i] = c.take<u16>(d * Tp);
  if (gt == BS_F32)
    for (int i = 0; i < 3; ++i) w.dy_rows[i] = c.take<u16>(T * n);
  if (wt == BS_F32)
    for (int i = 0; i < 3; ++i) w.w_rows[i] = c.take<u16>(d * n);
  if (want_y) {
    for (int i = 0; i < 3; ++i) w.uq_rows[i] = c.take<u16>(T * d);
    for (int i = 0; i < ntw; ++i) w.wT[i] = c.take<u16>(n * d);
  }
  w.bias_rg = c.take<float>(d);
  w.bias_ng = c.take<float>(d);
  for (int i = 0; i < 2; ++i) w.bias_w[i] = c.take<float>(d * n);
  w.gpart = c.take<double>(3 * ((T + GRID_GAIN_RT - 1) / GRID_GAIN_RT + 1) * d);
  w.gemm_part_cap = 4 * d * std::max<int64_t>(std::max<int64_t>(T, n), 64);
  w.gemm_part = c.take<float>(w.gemm_part_cap);
  return w;
}

}  // namespace

size_t grid_ws_size(int64_t T, int64_t d, int64_t n) {
  if (T < 0 || d < 8 || n < 8) return 0;
  Carver c;
  carve_grid(c, T, d, n, BS_F32, BS_F32, true);
  return c.used();
}

struct GridIO {
  const void *X, *W, *dY;
  const float* gain;
  bs_dtype dt;
  int64_t T, d, n;
  float eps;
  int bits;
  const bs_grid_policy* pol;
  int n_pol, K;
  uint64_t seed;
  uint32_t store_id;
  float* Y;
  int8_t* codes;
  float* step;
  float *dgain_ref, *dW_ref, *dX_ref;
  bs_est dgain, dW;
  bs_diag* diag;
};

bs_status grid_run(const GridIO& io, void* ws, size_t ws_bytes, hipStream_t st) {
  const int64_t T = io.T, d = io.d, n = io.n;
  if (!io.X || !io.W || !io.dY || !io.gain || !io.codes || !io.step || !io.dgain_ref || !io.dW_ref || !io.dX_ref ||
      !io.pol || !io.diag)
    return BS_EINVAL;
  if (io.dt != BS_F32 && io.dt != BS_BF16) return BS_EDTYPE;
  if (io.bits < 2 || io.bits > 8 || io.K < 1 || io.K > 4096 || io.n_pol < 1 || io.n_pol > 16 || !(io.eps >= 0.0f))
    return BS_EINVAL;
  if (T < 1 || d < 8 || d > 8192 || (d & 7) || n < 8 || (n & 7) || T > 65535LL * 256 || n > 0x7FFFFFFF)
    return BS_ESHAPE;
  if (io.dgain.se || io.dW.se) return BS_EUNSUPPORTED;
  for (int i = 0; i < io.n_pol; ++i) {
    if (io.pol[i].gain_use < BS_READ_U || io.pol[i].gain_use > BS_READ_N) return BS_EINVAL;
    if (io.pol[i].weight_use < BS_WREAD_U || io.pol[i].weight_use > BS_WREAD_R_EPS) return BS_EINVAL;
  }
  const bs_dtype wt = io.dt, gt = io.dt, xt = io.dt;
  Carver probe;
  carve_grid(probe, T, d, n, wt, gt, io.Y != nullptr);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < probe.used()) return BS_EWORKSPACE;
  Carver c(ws, ws_bytes);
  GridWs w = carve_grid(c, T, d, n, wt, gt, io.Y != nullptr);
  const int64_t Tp = round_up(T, 64);
  const int nt = gt == BS_F32 ? 3 : 1, ntw = wt == BS_F32 ? 3 : 1;
  const uint32_t base = io.store_id * 256u;

  // forward: RMSNorm (fixed fp32 order), the grid store
  BS_TRY(launch_init_diag(io.diag, st));
  BS_TRY(launch_rmsnorm_fwd(io.X, xt, io.gain, T, d, io.eps, w.u, w.rstd, io.diag, st));
  {
    ProfScope prof("grid_store", st);
    grid_store_kernel<<<(unsigned)((T + 3) / 4), 256, 0, st>>>(w.u, T, d, io.bits, io.seed, base, io.codes, io.step,
                                                               w.uq, w.eU, io.diag);
    BS_CHECK_LAUNCH();
  }
  // u_q and the residuals enter the contractions as three bf16 terms: the fp32 values at every
  // magnitude, against W and dY as given (bf16) or as three terms (fp32)
  // Y = u_q W
  if (io.Y) {
    BS_TRY(launch_planes(w.uq, BS_F32, T, d, d, false, w.uq_rows, 3, d, 1.0f, st));
    BS_TRY(launch_planes(io.W, wt, d, n, n, true, w.wT, ntw, d, 1.0f, st));
    GemmArgs g{};
    g.M = (int)T;
    g.N = (int)n;
    g.K = (int)d;
    g.lda = d;
    g.ldb = d;
    g.ldc = n;
    g.alpha = 1.0f;
    g.C = io.Y;
    gemm_add_products(g, w.uq_rows, 3, w.wT, ntw, 2, true);
    BS_TRY(launch_gemm(g, st));
  }
  // du = dY W^T
  {
    GemmArgs g{};
    g.M = (int)T;
    g.N = (int)d;
    g.K = (int)n;
    g.lda = n;
    g.ldb = n;
    g.ldc = d;
    g.alpha = 1.0f;
    g.C = w.du;
    g.part = w.gemm_part;
    g.part_cap = w.gemm_part_cap;
    u16* A0 = (u16*)io.dY;
    u16* B0 = (u16*)io.W;
    u16* const* Aops = &A0;
    u16* const* Bops = &B0;
    if (gt == BS_F32) {
      BS_TRY(launch_planes(io.dY, gt, T, n, n, false, w.dy_rows, 3, n, 1.0f, st));
      Aops = w.dy_rows;
    }
    if (wt == BS_F32) {
      BS_TRY(launch_planes(io.W, wt, d, n, n, false, w.w_rows, 3, n, 1.0f, st));
      Bops = w.w_rows;
    }
    gemm_add_products(g, Aops, nt, Bops, ntw);
    BS_TRY(launch_gemm(g, st));
  }
  // the new rounding's residual over K trials
  {
    ProfScope prof("grid_fresh", st);
    BS_TRY(launch_fresh_flat(T * d, io.K, [&](auto g, auto ts, unsigned blocks, int nt) {
      grid_fresh_kernel<decltype(g)::value, decltype(ts)::value><<<blocks, nt, 0, st>>>(
          w.u, io.step, T, d, io.bits, io.seed, base + 1, io.K, w.eE);
    }));
    BS_CHECK_LAUNCH();
  }
  // weight use: reference and the U and R+e biases, contractions of [d][Tp] planes with dY^T (the N
  // bias is their sum)
  BS_TRY(launch_planes(io.dY, gt, T, n, n, true, w.dyT, nt, Tp, 1.0f, st));
  const float* srcs[3] = {w.uq, w.eU, w.eE};
  float* dsts[3] = {io.dW_ref, w.bias_w[0], w.bias_w[1]};
  for (int i = 0; i < 3; ++i) {
    BS_TRY(launch_planes(srcs[i], BS_F32, T, d, d, true, w.aT, 3, Tp, 1.0f, st));
    GemmArgs g{};
    g.M = (int)d;
    g.N = (int)n;
    g.K = (int)Tp;
    g.lda = Tp;
    g.ldb = Tp;
    g.ldc = n;
    g.alpha = 1.0f;
    g.C = dsts[i];
    g.part = w.gemm_part;
    g.part_cap = w.gemm_part_cap;
    if (!gemm_add_products(g, w.aT, 3, w.dyT, nt, 2, true)) return BS_EINVAL;
    BS_TRY(launch_gemm(g, st));
  }
  // gain use: fp64 column sums
  {
    const int64_t nch = (T + GRID_GAIN_RT - 1) / GRID_GAIN_RT;
    const dim3 grid((unsigned)nch, (unsigned)((d + 255) / 256));
    if (xt == BS_F32)
      grid_gain_kernel<float><<<grid, 256, 0, st>>>((const float*)io.X, w.rstd, io.gain, w.u, w.du, w.eU, w.eE, T, d,
                                                   w.gpart);
    else
      grid_gain_kernel<u16><<<grid, 256, 0, st>>>((const u16*)io.X, w.rstd, io.gain, w.u, w.du, w.eU, w.eE, T, d,
                                                 w.gpart);
    BS_CHECK_LAUNCH();
    BS_TRY(launch_gain_final(w.gpart, nch, d, io.dgain_ref, w.bias_rg, w.bias_ng, st));
  }
  // the normalization input gradient with unrounded values
  if (xt == BS_F32) {
    DxArgs<float> da{(const float*)io.X, w.rstd, io.gain, w.du, nullptr, nullptr, F8{}, T, d, io.dX_ref, nullptr};
    BS_TRY(launch_dx_t(da, st));
  } else {
    DxArgs<u16> da{(const u16*)io.X, w.rstd, io.gain, w.du, nullptr, nullptr, F8{}, T, d, io.dX_ref, nullptr};
    BS_TRY(launch_dx_t(da, st));
  }
  // per-policy estimates
  // every policy's estimates, one pass per gradient over its reference
  CombineMulti cg{}, cw{};
  cg.ref = io.dgain_ref;
  cw.ref = io.dW_ref;
  cg.n_pol = cw.n_pol = io.n_pol;
  cg.mean = io.dgain.mean;
  cg.bias_out = io.dgain.bias;
  cw.mean = io.dW.mean;
  cw.bias_out = io.dW.bias;
  for (int i = 0; i < io.n_pol; ++i) {
    const bs_grid_policy& q = io.pol[i];
    cg.bias[i] = q.gain_use == BS_READ_R ? w.bias_rg : (q.gain_use == BS_READ_N ? w.bias_ng : nullptr);
    cw.bias[i] = q.weight_use == BS_WREAD_U       ? w.bias_w[0]
                 : q.weight_use == BS_WREAD_N     ? w.bias_w[0]
                 : q.weight_use == BS_WREAD_R_EPS ? w.bias_w[1]
                                                  : nullptr;
    if (q.weight_use == BS_WREAD_N) cw.bias2[i] = w.bias_w[1];
  }
  BS_TRY(launch_combine_multi(cg, d, cw, d * n, CombineMulti{}, 0, st));
  return BS_OK;
}

}  // namespace bsp

using namespace bsp;

extern "C" {

size_t bs_rmsnorm_linear_grid_workspace_size(int64_t T, int64_t d, int64_t n) { return grid_ws_size(T, d, n); }

bs_status bs_rmsnorm_linear_grid_fwd_bwd(const void* X, const float* gain, const void* W, const void* dY, bs_dtype dt,
                                         int64_t T, int64_t d, int64_t n, float eps, int bits,
                                         const bs_grid_policy* pol, int n_pol, int K, uint64_t seed,
                                         uint32_t store_id, float* Y, int8_t* u_codes, float* u_step,
                                         float* dgain_ref, float* dW_ref, float* dX_ref, bs_est dgain, bs_est dW,
                                         bs_diag* diag, void* ws, size_t ws_bytes, void* stream) {
  GridIO io{X, W, dY, gain, dt, T, d, n, eps, bits, pol, n_pol, K, seed, store_id, Y, u_codes, u_step, dgain_ref,
            dW_ref, dX_ref, dgain, dW, diag};
  return grid_run(io, ws, ws_bytes, (hipStream_t)stream);
}

}  // extern "C"
