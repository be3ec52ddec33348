// The trial loop of the new-rounding counters over flat groups of four elements, shared by the FP8
// and the grid store's kernels.
//
// A block of FRESH_NT(TS) threads takes LN x G consecutive groups (LN = threads per trial part, G
// groups per thread), an aligned power-of-two range, so the high counter word is uniform. The trials
// of one element are independent, so a tensor with too few elements to fill the chip splits its
// trials over TS parts of the block's threads (part p takes trials p, p + TS, ...); the counts of the
// parts meet in LDS (integers: any order gives the same sum).
#pragma once
#include "bsp_kernels.h"

namespace bsp {

constexpr int fresh_nt(int TS) { return TS > 4 ? 64 * TS : 256; }

template <int G, int TS>
struct FreshBlock {
  static constexpr int NT = fresh_nt(TS), LN = NT / TS;
  int part, ln;
  uint64_t base;  // the block's first group
  __device__ __forceinline__ FreshBlock() {
    const int tid = threadIdx.x;
    part = TS > 1 ? __builtin_amdgcn_readfirstlane(tid / LN) : 0;
    ln = TS > 1 ? tid % LN : tid;
    base = (uint64_t)blockIdx.x * (LN * G);
  }
  __device__ __forceinline__ uint64_t group(int r) const { return base + r * LN + ln; }

  // cnt[r][q] = trials (trial0 .. trial0 + K - 1) of group r's element q that round up (threshold F)
  __device__ __forceinline__ void count(uint32_t (&F)[G][4], uint32_t (&cnt)[G][4], int K, int trial0, uint32_t use,
                                        uint64_t seed) const {
    constexpr int TB = 4;
    const uint32_t g_hi = (uint32_t)(base >> 32);
#pragma unroll
    for (int r = 0; r < G; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        cnt[r][q] = 0;
        asm volatile("" : "+v"(F[r][q]));  // opaque: keeps validity tests out of the trial loop
      }
    for (int k0 = part; k0 < K; k0 += TB * TS) {
#pragma unroll
      for (int i = 0; i < TB; ++i) {
        const int k = k0 + i * TS;
        if (k >= K) break;
#pragma unroll
        for (int r = 0; r < G; ++r) {
          const Philox4 p = philox4x32_10((uint32_t)base + r * LN + ln, g_hi, (uint32_t)(k + trial0), use, (uint32_t)seed,
                                          (uint32_t)(seed >> 32));
#pragma unroll
          for (int q = 0; q < 4; ++q) cnt[r][q] += sr_up(F[r][q], philox_word(p, q));
        }
      }
    }
  }

  // out[r] = the group's four counts over all parts, 16 bits each (K <= 4096: no carry between
  // them); false for the threads of the other parts, whose work is done (all threads call it)
  __device__ __forceinline__ bool merge(const uint32_t (&cnt)[G][4], uint2 (&out)[G]) const {
#pragma unroll
    for (int r = 0; r < G; ++r) out[r] = make_uint2(cnt[r][0] | (cnt[r][1] << 16), cnt[r][2] | (cnt[r][3] << 16));
    if constexpr (TS > 1) {
      __shared__ uint32_t red[2][LN * G];
      for (int i = threadIdx.x; i < 2 * LN * G; i += NT) (&red[0][0])[i] = 0;
      __syncthreads();
#pragma unroll
      for (int r = 0; r < G; ++r) {
        atomicAdd(&red[0][r * LN + ln], out[r].x);
        atomicAdd(&red[1][r * LN + ln], out[r].y);
      }
      __syncthreads();
      if (part != 0) return false;
#pragma unroll
      for (int r = 0; r < G; ++r) out[r] = make_uint2(red[0][r * LN + ln], red[1][r * LN + ln]);
    }
    return true;
  }
};

// Groups per thread and trial parts of n elements and K trials, and the launch of kernel<G, TS>. In
// waves of one group per thread on the chip's 1024 SIMDs: 8 groups per thread (the set-up paid once
// for all of them) while that leaves two waves each; fewer groups per thread, then 4 and 16 trial
// parts, below. (256 x 64, 64 trials: 4.9 us with 16 parts, 56 with one; 1111 x 520, 24 trials: 9.6
// with 4, 27 with one.)
template <typename Launch>
bs_status launch_fresh_flat(int64_t n, int K, Launch go) {
  const int64_t groups = n / 4, waves = groups / 64;
  auto run = [&](auto g, auto ts) -> bs_status {
    constexpr int G = decltype(g)::value, TS = decltype(ts)::value;
    const int64_t per = (int64_t)FreshBlock<G, TS>::LN * G, blocks = (groups + per - 1) / per;
    if (blocks > 0x7FFFFFFF) return BS_ESHAPE;
    go(g, ts, (unsigned)blocks, fresh_nt(TS));
    return BS_OK;
  };
  using std::integral_constant;
  if (waves >= 8 * 2048) return run(integral_constant<int, 8>{}, integral_constant<int, 1>{});
  if (waves >= 2 * 2048 || K < 4) return run(integral_constant<int, 2>{}, integral_constant<int, 1>{});
  if (waves >= 512 || K < 16) return run(integral_constant<int, 2>{}, integral_constant<int, 4>{});
  return run(integral_constant<int, 1>{}, integral_constant<int, 16>{});
}

}  // namespace bsp
