// The log-softmax operator test (Sec. 4.3; App. C.5) on the GPU, in fp64 as the paper's test:
// the operator's backward h - exp(S) (1^T h) reads a saved output S = l + r (r_j = +-eps) under
// reuse, or l + r' with r' drawn anew; per trial the statistic is the mean over rows and classes
// of (g - g*) / p under the likelihood (h = -e_y) and the constructed loss (h = r).
//
// The four entry errors share their factors: with w_j(x) = (p_j - exp(l_j + x) / cal) / p_j for
// x = +eps or -eps, (g_j - g*_j) / p_j = (1^T h) w_j under either loss, so per (row, trial) the
// row sums of w under the two copies and the number of plus signs of r give all four. The
// preparation writes w_j(+eps) and w_j(-eps) once (the operator's exponentials and quotients in
// fp64, from the logits); a trial adds the one its sign picks. Per element and trial that leaves
// two Philox words (8.5 VALU each), a compare, a 64-bit select and an fp64 add per copy: 26 VALU,
// the bound. (Forming g and g* anew per trial took a third word for 1^T h and four fp64 quotients:
// 7.0 ms at 512 x 32768, 64 trials; now 0.78 ms of 0.93 for the call, 1.38 T element-trials/s against 1.46
// at the VALU ceiling; 0.90 ms in a trace of six calls, at the clock of an idle chip.)
//
// A wave takes one row and TK trials; a lane takes groups of 4 consecutive classes (one Philox
// call per group, draw and trial), the trials unrolled inside so that the element's part of the
// first two rounds is shared and the trial's runs on the scalar unit. A block's up to four waves
// share the row. A sum over the wave halves the trials each lane carries at each exchange.
#include <algorithm>

#include "bsp_kernels.h"

namespace bsp {

namespace {

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// l = z - max - log(sum exp(z - max)) per row, one block per row, then w(+eps) and w(-eps): four
// fp64 exponentials and two quotients per element (one wave per row left most of the chip idle:
// 694 us at 512 x 32768 with three exponentials, 136 us now)
__global__ __launch_bounds__(1024) void lsm_prep_kernel(const double* __restrict__ z, int C, double eps, double cal,
                                                        double* __restrict__ wp, double* __restrict__ wm) {
  const int64_t row = blockIdx.x;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
  const double* zr = z + row * C;
  __shared__ double red[16];
  double m = -INFINITY;
  for (int j = tid; j < C; j += nt) m = fmax(m, zr[j]);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) m = fmax(m, __shfl_xor(m, off, 64));
  if (lane == 0) red[wave] = m;
  __syncthreads();
  m = red[0];
  for (int i = 1; i < nw; ++i) m = fmax(m, red[i]);
  double se = 0.0;
  for (int j = tid; j < C; j += nt) se += exp(zr[j] - m);
  se = wsum(se);
  __syncthreads();
  if (lane == 0) red[wave] = se;
  __syncthreads();
  se = red[0];
  for (int i = 1; i < nw; ++i) se += red[i];
  const double lse = m + log(se);
  for (int j = tid; j < C; j += nt) {
    const double lj = zr[j] - lse, p = exp(lj);
    const int64_t e = row * C + j;
    wp[e] = (p - exp(lj + eps) / cal) / p;
    wm[e] = (p - exp(lj + -eps) / cal) / p;
  }
}

// v[t] summed over the L lanes of a lane group (L >= TK, powers of two): each exchange hands half
// of a lane's values over, so lane i of the group ends with value t(i) in v[0], t from its top
// bits; the remaining exchanges add whole. A fixed tree.
template <int H, typename V>
__device__ __forceinline__ void sum_halves(V* v, int lane, int off) {
  if constexpr (H >= 1) {
    const bool up = (lane & off) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const V lo = v[i], hi = v[i + H];
      const V send = up ? lo : hi, keep = up ? hi : lo;
      v[i] = keep + __shfl_xor(send, off, 64);
    }
    sum_halves<H / 2>(v, lane, off >> 1);
  }
}
template <int TK, typename V>
__device__ __forceinline__ void sum_trials(V* v, int lane, int L) {
  sum_halves<TK / 2>(v, lane, L >> 1);
  for (int off = L / (2 * TK); off >= 1; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
}

// per (row, trial): the row sums of the four entry errors, [4][K][rows]. SUB: rows of at most 32
// groups, L lanes (a power of two, at least TK) per trial and 64 / L trials side by side; else
// L = 64. MORE: the rows from row0 on (the launches after the first; the loop scheduled around that
// base takes 927 us for 912 at 512 x 32768).
template <int TK, bool SUB, bool MORE>
__global__ __launch_bounds__(256) void lsm_trial_kernel(const double* __restrict__ wp, const double* __restrict__ wm,
                                                        const int32_t* __restrict__ y, int64_t rows, int C, int L,
                                                        double eps, int K, uint64_t seed, uint32_t use_r,
                                                        uint32_t use_p, double* __restrict__ part, int64_t row0) {
  const int64_t row = MORE ? row0 + blockIdx.x : blockIdx.x;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nsub = SUB ? 64 / L : 1;
  const int nw = TK == 16 ? 4 : blockDim.x >> 6;        // (read at run time, 16 trials: 962 us for 927 at 512 x 32768)
  const int k0 = (blockIdx.y * nw + wave) * TK * nsub;  // trial index (trial k0 + 1) of the wave's first
  if (k0 >= K) return;                                 // wave-uniform; no barrier below
  const int sub = SUB ? lane / L : 0, gl = SUB ? lane % L : lane;
  const int ngroups = C / 4;
  double ar[TK], ap[TK];
  int n[TK];
#pragma unroll
  for (int t = 0; t < TK; ++t) ar[t] = ap[t] = 0.0, n[t] = 0;
  for (int gi = gl; gi < ngroups; gi += L) {
    const int64_t e = row * C + 4 * gi;
    const uint64_t grp = (uint64_t)e / 4;
    double vp[4], vm[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) vp[q] = wp[e + q], vm[q] = wm[e + q];
#pragma unroll
    for (int t = 0; t < TK; ++t) {
      const uint32_t trial = (uint32_t)(k0 + t * nsub + sub + 1);  // past K: computed, not stored
      const Philox4 pr = philox_group(seed, grp, trial, use_r);
      const Philox4 pp = philox_group(seed, grp, trial, use_p);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool ur = (int32_t)philox_word(pr, q) < 0, up = (int32_t)philox_word(pp, q) < 0;  // words >= 2^31
        ar[t] += ur ? vp[q] : vm[q];
        ap[t] += up ? vp[q] : vm[q];
        n[t] += ur;
      }
    }
  }
  sum_trials<TK>(ar, lane, L);
  sum_trials<TK>(ap, lane, L);
  sum_trials<TK>(n, lane, L);
  int t = 0;
  for (int h = TK / 2, off = L >> 1; h >= 1; h >>= 1, off >>= 1) t += (lane & off) ? h : 0;
  const int k = k0 + t * nsub + sub;
  if ((gl & (L / TK - 1)) == 0 && k < K) {
    const int yt = y[row];
    const double sh = (yt >= 0 && yt < C) ? -1.0 : 0.0;  // likelihood: 1^T h
    const double sr = eps * (double)(2 * n[0] - C);      // constructed: 1^T r
    const int64_t o = (int64_t)k * rows + row, stride = (int64_t)K * rows;
    part[o] = sh * ar[0];
    part[o + stride] = sh * ap[0];
    part[o + 2 * stride] = sr * ar[0];
    part[o + 3 * stride] = sr * ap[0];
  }
}

// per statistic: t_k = sum over rows (row order) / (rows C); mean and se over trials
// trials per block of the first reduction stage: one per wave while the second stage's single
// blocks stay short (the stage is latency: 66 us with 64 trials per block at 512 rows, 64 trials,
// now 8 us), 64 beyond
inline int lsm_rt(int K) { return K <= 4096 ? 4 : 64; }
// blocks of that stage that the workspace has room for: those of the largest smaller K too (a workspace
// query grows with every size)
inline int lsm_blocks_max(int K) { return std::max((K + 63) / 64, std::min((K + 3) / 4, 1024)); }

// mean over rows and classes of statistic c in trial k: one wave, rows lane-strided, combined by
// a fixed xor tree (every lane ends with the total)
__device__ __forceinline__ double lsm_trial_mean(const double* __restrict__ part, int64_t rows, int C, int K, int c,
                                                 int k) {
  const int lane = threadIdx.x & 63;
  double t = 0.0;
  for (int64_t i = lane; i < rows; i += 64) t += part[((int64_t)c * K + k) * rows + i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
  return t / ((double)rows * C);
}

// first stage: block (j, c) takes trials rt j .. rt j + rt - 1 of statistic c and writes their sums of
// d_k = m_k - m_0 and d_k^2 (shifted by trial 0's mean m_0, which block (0, c) also writes)
__global__ __launch_bounds__(256) void lsm_reduce_kernel(const double* __restrict__ part, int64_t rows, int C, int K,
                                                         int rt, double* __restrict__ acc, double* __restrict__ m0) {
  const int c = blockIdx.y, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double t0 = lsm_trial_mean(part, rows, C, K, c, 0);
  double s1 = 0.0, s2 = 0.0;
  for (int j = w; j < rt; j += 4) {
    const int k = blockIdx.x * rt + j;
    if (k >= K) break;  // wave-uniform
    const double d = lsm_trial_mean(part, rows, C, K, c, k) - t0;
    s1 += d;
    s2 += d * d;
  }
  __shared__ double red[2][4];
  if (lane == 0) {
    red[0][w] = s1;
    red[1][w] = s2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double* o = acc + 2 * ((int64_t)c * gridDim.x + blockIdx.x);
    o[0] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    o[1] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    if (blockIdx.x == 0) m0[c] = t0;
  }
}

// second stage: block c sums its nb partials (thread-strided, then a fixed tree) into the mean
// and its standard error over the K trials
__global__ __launch_bounds__(256) void lsm_final_kernel(const double* __restrict__ acc, const double* __restrict__ m0,
                                                        int nb, int K, double* __restrict__ stats) {
  const int c = blockIdx.x;
  __shared__ double red[2][256];
  double s1 = 0.0, s2 = 0.0;
  for (int j = threadIdx.x; j < nb; j += 256) {
    s1 += acc[2 * ((int64_t)c * nb + j)];
    s2 += acc[2 * ((int64_t)c * nb + j) + 1];
  }
  red[0][threadIdx.x] = s1;
  red[1][threadIdx.x] = s2;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) {
      red[0][threadIdx.x] += red[0][threadIdx.x + off];
      red[1][threadIdx.x] += red[1][threadIdx.x + off];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double S1 = red[0][0], S2 = red[1][0];
    const double var = K > 1 ? fmax(S2 - S1 * S1 / K, 0.0) / (K - 1) : 0.0;
    stats[2 * c] = m0[c] + S1 / K;
    stats[2 * c + 1] = sqrt(var / K);
  }
}

}  // namespace

// rows per launch: a launch holds fewer than 2^32 threads in a grid dimension, and a row takes up to 1024
constexpr int64_t LSM_ROWS = (int64_t)1 << 21;

size_t lsm_ws_size(int64_t rows, int C, int K) {
  if (rows < 1 || C < 4 || (C & 3) || K < 1) return 0;
  Carver c;
  for (int i = 0; i < 2; ++i) c.take<double>(rows * C);
  c.take<double>((int64_t)4 * K * rows);
  c.take<double>((int64_t)8 * lsm_blocks_max(K));
  c.take<double>(4);
  return c.used();
}

}  // namespace bsp

using namespace bsp;

extern "C" {

size_t bs_logsoftmax_check_workspace_size(int64_t rows, int C, int K) { return lsm_ws_size(rows, C, K); }

bs_status bs_logsoftmax_reuse_check(const double* logits, const int32_t* target, int64_t rows, int C, double eps,
                                    int K, uint64_t seed, uint32_t store_id, int calibrate, double* stats, void* ws,
                                    size_t ws_bytes, void* stream) {
  if (!logits || !target || !stats) return BS_EINVAL;
  if (rows < 1 || K < 1 || K > (1 << 20) || !(eps > 0.0) || !(eps < 1.0)) return BS_EINVAL;
  if (C < 4 || (C & 3) || rows > 0x7FFFFFFF) return BS_ESHAPE;
  const size_t need = lsm_ws_size(rows, C, K);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need) return BS_EWORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  Carver c(ws, ws_bytes);
  double* wp = c.take<double>(rows * C);
  double* wm = c.take<double>(rows * C);
  double* part = c.take<double>((int64_t)4 * K * rows);
  const int rt = lsm_rt(K), nb = (K + rt - 1) / rt;
  double* acc = c.take<double>((int64_t)8 * lsm_blocks_max(K));
  double* m0 = c.take<double>(4);
  {
    ProfScope prof("lsm_prep", st);
    // a row's fp64 exponentials bound it: as many waves per row as its length fills
    const int nt = C >= 4096 ? 1024 : (C >= 512 ? 256 : 64);
    for (int64_t r0 = 0; r0 < rows; r0 += LSM_ROWS) {
      lsm_prep_kernel<<<(unsigned)std::min(LSM_ROWS, rows - r0), nt, 0, st>>>(
          logits + r0 * C, C, eps, calibrate ? cosh(eps) : 1.0, wp + r0 * C, wm + r0 * C);
      BS_CHECK_LAUNCH();
    }
  }
  const uint32_t base = store_id * 256u;
  {
    ProfScope prof("lsm_trial", st);
    // L lanes per trial (short rows put several trials side by side). Trials per lane group: as many as
    // leave two waves of a row work (trials past K cost what others do: 4096 x 1000, one trial, 72 us
    // with 1, 78 with 4, 112 with 16; 64 trials 325, 277, 268) and give every SIMD two waves (512 x
    // 32768, 16 trials: 350 us with 2, 378 with 4, 613 with 16). As many waves per block as have trials.
    int L = 64;
    while (L > 16 && C / 4 <= L / 2) L /= 2;
    const int nsub = 64 / L;
    int tk = 1;
    while (tk < 16 && 4 * tk * nsub <= K && rows * ((K + 2 * tk * nsub - 1) / (2 * tk * nsub)) >= 2048) tk *= 2;
    const int nw = tk == 16 ? 4 : std::min(4, (K + tk * nsub - 1) / (tk * nsub)), per = nw * tk * nsub;
    for (int64_t r0 = 0; r0 < rows; r0 += LSM_ROWS) {
      const dim3 grid((unsigned)std::min(LSM_ROWS, rows - r0), (unsigned)((K + per - 1) / per));
      auto go = [&](auto n) {
        constexpr int TK = decltype(n)::value;
        auto run = [&](auto kernel) {
          kernel<<<grid, 64 * nw, 0, st>>>(wp, wm, target, rows, C, L, eps, K, seed, base, base + 1, part, r0);
        };
        if (r0 == 0)
          L == 64 ? run(lsm_trial_kernel<TK, false, false>) : run(lsm_trial_kernel<TK, true, false>);
        else
          L == 64 ? run(lsm_trial_kernel<TK, false, true>) : run(lsm_trial_kernel<TK, true, true>);
      };
      switch (tk) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 4: go(std::integral_constant<int, 4>{}); break;
        case 8: go(std::integral_constant<int, 8>{}); break;
        default: go(std::integral_constant<int, 16>{});
      }
      BS_CHECK_LAUNCH();
    }
  }
  {
    ProfScope prof("lsm_reduce", st);
    lsm_reduce_kernel<<<dim3((unsigned)nb, 4), 256, 0, st>>>(part, rows, C, K, rt, acc, m0);
    lsm_final_kernel<<<4, 256, 0, st>>>(acc, m0, nb, K, stats);
    BS_CHECK_LAUNCH();
  }
  return BS_OK;
}

}  // extern "C"
