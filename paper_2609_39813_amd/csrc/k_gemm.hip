// bf16 MFMA contraction for gfx950: C[M,N] = alpha * sum_seg A_seg[M,K] B_seg[N,K]^T (+ C).
//
// Both operands are K-contiguous ("NT"): every contraction of the backward is brought to
// this layout by the kernels that produce its operands (transposed planes are written
// once, in the layout the contraction reads). Several (A, B) segments over the same K
// are summed in one pass: that is how fp32-valued operands enter as a sum of exact bf16
// terms. Products of bf16 values are exact in the fp32 accumulator.
//
// Three kernels. The pipelined kernel moves operand tiles straight from
// global memory into LDS (buffer_load_dwordx4 ... lds, no register staging) in 64-deep
// chunks, so that every operand row of a chunk is one full 128-byte line; two LDS stages
// (128 KB for a 256 x 256 tile) hold the chunk being computed and the next one. A 256 x 256
// block tile is split over 8 wave64s of 128 x 64 (8 x 4 MFMA 16x16x32 tiles, accumulators in
// AGPRs): at 128 accumulator registers a wave fits twice per SIMD, so one wave's MFMAs run
// while the other waits on a load issue or the barrier. The 16-byte unit u of row r sits at unit u ^ (r & 7) of its LDS row, so the
// rows one ds_read_b128 serves together fall on distinct banks. The operand loads go through
// buffer resources that end with the tile's last valid row (rows past M or N read as zero).
// The instruction order of the main loop is fixed in source (scheduling barriers): LDS reads
// of the next k-step and the global loads of the chunk after next are spread between the
// MFMAs, one barrier per chunk. Shapes with fewer tiles than CUs split K over blocks into
// fp32 partials that one more kernel sums in a fixed order (the result does not depend on
// timing). The small-output kernel (32 x 32 tiles, K split over a block's waves) serves outputs that
// even 128 x 128 tiles leave on a few CUs; plan_gemm chooses. The register-staged kernel below
// serves operands that are not 16-byte aligned or whose rows are too long for buffer offsets.
//
// Register-staged kernel: tile 128 x 128 x 64, 256 threads (4 wave64s in
// 2 x 2), double-buffered LDS with a 16-byte row pad (row stride 144 B keeps the 16 rows read
// by one ds_read_b128 on distinct banks).
//
// All renumber workgroups so that the tiles of one XCD are contiguous in row-major tile order
// (shared A panels in that XCD's L2).
#include <algorithm>
#include <cmath>

#include "bsp_kernels.h"

namespace bsp {

constexpr int GBK = 64, GPAD = 72;

// Block tile BM x BN, 256 threads as a WGM x WGN grid of wave64s; each wave owns a
// (BM / WGM) x (BN / WGN) tile of 16 x 16 MFMA results.
template <int BM, int BN, int WGM, int WGN, bool F16>
__global__ __launch_bounds__(256) void gemm_nt_kernel(GemmArgs g) {
  static_assert(WGM * WGN == 4, "four waves");
  constexpr int TM = BM / WGM, TN = BN / WGN, FM = TM / 16, FN = TN / 16;
  constexpr int LA = BM / 32, LB = BN / 32;  // 16-byte loads per thread per chunk
  __shared__ __attribute__((aligned(16))) u16 sA[2][BM][GPAD];
  __shared__ __attribute__((aligned(16))) u16 sB[2][BN][GPAD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int tiles_n = (g.N + BN - 1) / BN;
  const int nblk = gridDim.x;
  int bid = blockIdx.x;
  if ((nblk & 7) == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);  // XCD-contiguous tiles
  const int bm = (bid / tiles_n) * BM, bn = (bid % tiles_n) * BN;

  const int nch = (g.K + GBK - 1) / GBK;
  const int total = nch * g.nseg;

  const int lrow = tid >> 3, lk = (tid & 7) * 8;
  uint4 ra[LA], rb[LB];
  auto gload = [&](int c) {
    const int seg = c / nch;
    const int k0 = (c - seg * nch) * GBK + lk;
    const u16* A = g.A[seg];
    const u16* B = g.B[seg];
    const bool ka = k0 < g.K;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int r = lrow + 32 * i;
      ra[i] = (bm + r < g.M && ka) ? *(const uint4*)(A + (int64_t)(bm + r) * g.lda + k0) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int r = lrow + 32 * i;
      rb[i] = (bn + r < g.N && ka) ? *(const uint4*)(B + (int64_t)(bn + r) * g.ldb + k0) : make_uint4(0, 0, 0, 0);
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < LA; ++i) *(uint4*)&sA[buf][lrow + 32 * i][lk] = ra[i];
#pragma unroll
    for (int i = 0; i < LB; ++i) *(uint4*)&sB[buf][lrow + 32 * i][lk] = rb[i];
  };

  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  if (total > 0) {
    gload(0);
    sstore(0);
  }
  __syncthreads();
  const int fr = lane & 15, fk = (lane >> 4) * 8;
  for (int c = 0; c < total; ++c) {
    const int buf = c & 1;
    if (c + 1 < total) gload(c + 1);
#pragma unroll
    for (int kk = 0; kk < GBK; kk += 32) {
      bf16x8 af[FM], bfr[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) af[i] = *(const bf16x8*)&sA[buf][wm * TM + i * 16 + fr][kk + fk];
#pragma unroll
      for (int j = 0; j < FN; ++j) bfr[j] = *(const bf16x8*)&sB[buf][wn * TN + j * 16 + fr][kk + fk];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          if constexpr (F16)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, af[i]),
                                                               __builtin_bit_cast(halfx8, bfr[j]), acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
        }
    }
    if (c + 1 < total) sstore(buf ^ 1);
    __syncthreads();
  }

  // D[i][j] of a 16x16 tile sits in lane (j + 16 * (i / 4)), register i % 4.
  const int oc = lane & 15, orow = (lane >> 4) * 4;
  const float alpha = gemm_alpha(g);
#pragma unroll
  for (int i = 0; i < FM; ++i) {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = bn + wn * TN + j * 16 + oc;
      if (n >= g.N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = bm + wm * TM + i * 16 + orow + r;
        if (m < g.M) {
          float* p = g.C + (int64_t)m * g.ldc + n;
          const float v = alpha * acc[i][j][r];
          *p = g.accumulate ? *p + v : v;
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// pipelined kernel
// ------------------------------------------------------------------------------------
// A stage holds a 64-deep K chunk: every operand row is one 128-byte line. The 16-byte unit u
// of row r sits at unit u ^ swz(r) of its LDS row, so that the rows one ds_read_b128 serves
// together fall on distinct banks.
constexpr int LBK = 64, LNST = 2;
__device__ __forceinline__ int swz_of(int r) { return r & 7; }
__device__ __forceinline__ int lds_swz(int r, int u) { return r * 128 + ((u ^ swz_of(r)) << 4); }

// Block tile BM x BN, WGM x WGN wave64s, each owning a (BM / WGM) x (BN / WGN) tile. F16: the
// operands hold fp16 values (v_mfma_f32_16x16x32_f16), else bf16.
template <int BM, int BN, int WGM, int WGN, bool F16>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_lds_kernel(GemmArgs g, int cps) {
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN, FM = WM / 16, FN = WN / 16;
  constexpr int AI = BM / (8 * NW), BI = BN / (8 * NW), LPC = AI + BI;  // 1-KB loads (8 rows) per wave per chunk
  static_assert(AI * 8 * NW == BM && BI * 8 * NW == BN, "loads cover the tile");
  constexpr int STAGE = (BM + BN) * 128;
  __shared__ __attribute__((aligned(1024))) char smem[LNST * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN, ntile = tiles_m * tiles_n;
  const int nblk = gridDim.x;
  int bid = blockIdx.x;
  if ((nblk & 7) == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);
  const int zs = bid / ntile, tile = bid - zs * ntile;
  // a batched launch's member z (batched launches do not split K), else the split
  const int zb = g.batch > 1 ? zs : 0, split = g.batch > 1 ? 0 : zs;
  const int64_t oA = (int64_t)zb * g.sA, oB = (int64_t)zb * g.sB;
  // groups of GM tile rows: consecutive tiles (one XCD's share) form a GM-row patch, so the
  // A and B panels they read overlap in that XCD's L2
  constexpr int GM = 4;
  const int group = tile / (GM * tiles_n), in_group = tile - group * GM * tiles_n;
  const int first_m = group * GM, gsz = min(tiles_m - first_m, GM);
  const int bm = (first_m + in_group % gsz) * BM, bn = (in_group / gsz) * BN;
  const int nch = (g.K + LBK - 1) / LBK, total = nch * g.nseg;
  const int c0 = split * cps;
  const int n = min(total, c0 + cps) - c0;

  // Operand tiles are read through buffer resources whose range ends with the tile's last
  // valid row: rows past M (N) read as zero (their products are never stored) and cost no
  // memory traffic. Load i of this wave fills rows (wave * AI + i) * 8 .. +7 of A (then B):
  // lane l writes row l / 8 at unit position l % 8, which holds logical unit (l % 8) ^ swz(row);
  // swz(row) = swz(l / 8) because the row's other terms are multiples of 8. One per-lane byte
  // offset per operand; the load index and the k position enter as scalar offsets.
  const int rows_a = min(g.M - bm, BM), rows_b = min(g.N - bn, BN);
  const uint32_t lane_a = (uint32_t)(((wave * AI * 8 + (lane >> 3)) * g.lda + (((lane & 7) ^ swz_of(lane >> 3)) << 3)) * 2);
  const uint32_t lane_b = (uint32_t)(((wave * BI * 8 + (lane >> 3)) * g.ldb + (((lane & 7) ^ swz_of(lane >> 3)) << 3)) * 2);
  const uint32_t step_a = (uint32_t)(8 * g.lda * 2), step_b = (uint32_t)(8 * g.ldb * 2);
  auto rsrc = [](const u16* base, int64_t row0, int rows, int64_t ld) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(base + row0 * ld), (short)0, (int)(rows * ld * 2), 0x00020000);
  };
  // The next chunk to load: segment, k offset and the segment's resources (wave-uniform).
  // Past the last chunk of the contraction the position wraps to the start of the last
  // segment: the loop body is branch-free, and the surplus loads land in a stage that is
  // never read again.
  int iss_seg = c0 / nch, iss_k = (c0 - iss_seg * nch) * LBK;
  __amdgpu_buffer_rsrc_t ra = rsrc(g.A[iss_seg] + oA, bm, rows_a, g.lda);
  __amdgpu_buffer_rsrc_t rb = rsrc(g.B[iss_seg] + oB, bn, rows_b, g.ldb);
  // A segment's last chunk may be ragged (K any multiple of 8): lanes whose unit lies past K take
  // an offset past every resource (< 2^31 bytes) and read zero.
  const int unit_k = ((lane & 7) ^ swz_of(lane >> 3)) << 3;
  uint32_t va = 0, vb = 0;
  auto place = [&]() {
    const bool in = iss_k + unit_k < g.K;
    va = in ? lane_a : 0x7FFFFFF0u;
    vb = in ? lane_b : 0x7FFFFFF0u;
  };
  place();
  auto issue_one = [&](int st, int i) {
    char* base = smem + st * STAGE;
    if (i < AI)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (void __attribute__((address_space(3)))*)(base + (wave * AI + i) * 1024),
                                               16, va, (uint32_t)iss_k * 2 + i * step_a, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rb, (void __attribute__((address_space(3)))*)(base + BM * 128 + (wave * BI + i - AI) * 1024), 16, vb,
          (uint32_t)iss_k * 2 + (i - AI) * step_b, 0, 0);
  };
  // Kept out of the MFMA regions: the rare segment switch is a branch with scalar loads.
  auto advance = [&]() {
    iss_k += LBK;
    if (iss_k >= g.K) {
      iss_k = 0;
      if (++iss_seg < g.nseg) {
        ra = rsrc(g.A[iss_seg] + oA, bm, rows_a, g.lda);
        rb = rsrc(g.B[iss_seg] + oB, bn, rows_b, g.ldb);
      }
    }
    place();
  };

  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int fr = lane & 15, fc = lane >> 4;
  bf16x8 fa[2][FM], fb[2][FN];
  // MFMA t of a k-step, in row-major (i, j) order
  auto mfma_t = [&](int buf, int t) {
    const int i = t / FN, j = t % FN;
    if constexpr (F16)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, fa[buf][i]),
                                                         __builtin_bit_cast(halfx8, fb[buf][j]), acc[i][j], 0, 0, 0);
    else
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[buf][i], fb[buf][j], acc[i][j], 0, 0, 0);
  };
  // read q of a k-step's fragments: B first (the first MFMAs use every B fragment), then A
  auto read_q = [&](int st, int s, int q, bf16x8* a, bf16x8* b) {
    const char* base = smem + st * STAGE;
    if (q < FN)
      b[q] = *(const bf16x8*)(base + BM * 128 + lds_swz(wn * WN + q * 16 + fr, fc + 4 * s));
    else
      a[q - FN] = *(const bf16x8*)(base + lds_swz(wm * WM + (q - FN) * 16 + fr, fc + 4 * s));
  };
  // wait until at most vm of this wave's loads are pending and its fragment reads are done,
  // then a barrier without a memory fence (a fence would drain the prefetch too)
#define BS_LAND(vm)                                                                             \
  do {                                                                                          \
    __builtin_amdgcn_s_waitcnt(((vm) & 15) | (((vm) >> 4) << 14) | (7 << 4)); /* lgkmcnt(0) */ \
    asm volatile("s_barrier" ::: "memory");                                                     \
  } while (0)
  static_assert(LPC < 64, "vmcnt range");

  // Prologue: chunks 0 and 1 in flight; chunk 0 landed; its first k-step in registers.
#pragma unroll
  for (int st = 0; st < 2; ++st) {
#pragma unroll
    for (int i = 0; i < LPC; ++i) issue_one(st, i);
    advance();
  }
  BS_LAND(LPC);
#pragma unroll
  for (int q = 0; q < FM + FN; ++q) read_q(0, 0, q, fa[0], fb[0]);

  // Chunk c (stage c & 1), two k-steps of 32; the fragments alternate between two register
  // sets (k-step 0 computes from set 0 and fills set 1, k-step 1 the reverse).
  // k-step 0: its MFMAs, with the fragments of k-step 1 (same stage, landed) read in between.
  // k-step 1: the MFMAs of the first PA fragment rows; then chunk c + 1 is awaited and every
  //   wave has finished reading chunk c; the loads of chunk c + 2 go into chunk c's stage and
  //   the first fragments of chunk c + 1 are read, both between the remaining MFMAs: one read
  //   per MFMA, one load per LSP MFMAs, evenly over all of them (a burst of loads stalls the
  //   wave at issue and with it its MFMAs).
  // The instruction order is fixed in source: a scheduling barrier closes every MFMA's group
  // (its load, its read), so reads are issued well before their use. The last iteration reads
  // a stage of surplus data that is never used.
  constexpr int NM = FM * FN;                  // MFMAs per k-step
  constexpr int RD = FM + FN;                  // fragment reads per k-step
  constexpr int PA = FM >= 4 ? FM / 4 : 1;     // rows before the barrier
  constexpr int NA = PA * FN, NB = NM - NA;    // MFMAs before / after the barrier
  constexpr int M0 = NM / RD >= 2 ? 2 : 1;     // k-step 0: one read per M0 MFMAs
  constexpr int LSP = NB / LPC > 0 ? NB / LPC : 1;  // k-step 1: one load per LSP MFMAs
  static_assert(RD <= NB && LPC <= NB, "k-step 1 holds the reads and loads");
  for (int c = 0; c < n; ++c) {
    const int st = c & 1;
#pragma unroll
    for (int q = 0; q < RD; ++q) {
      read_q(st, 1, q, fa[1], fb[1]);
#pragma unroll
      for (int t = q * M0; t < (q + 1) * M0; ++t) mfma_t(0, t);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int t = RD * M0; t < NM; ++t) mfma_t(0, t);
    __builtin_amdgcn_sched_barrier(0);

#pragma unroll
    for (int t = 0; t < NA; ++t) mfma_t(1, t);
    __builtin_amdgcn_sched_barrier(0);
    BS_LAND(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      if (p % LSP == 0 && p / LSP < LPC) issue_one(st, p / LSP);
      if (p < RD) read_q(st ^ 1, 0, p, fa[0], fb[0]);
      mfma_t(1, NA + p);
      __builtin_amdgcn_sched_barrier(0);
    }
    advance();
  }
  // no load into LDS may outlive the block (the CU hands its LDS to the next block)
  __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));  // vmcnt(0)
#undef BS_LAND

  // D[i][j] of a 16x16 tile sits in lane (j + 16 * (i / 4)), register i % 4.
  const int oc = lane & 15, orow = (lane >> 4) * 4;
  float* out = g.part ? g.part + (int64_t)split * g.M * g.N : g.C + (int64_t)zb * g.sC;
  const int64_t ldo = g.part ? g.N : g.ldc;
  const float alpha = g.part ? 1.0f : gemm_alpha(g, zb);
  const bool acc_in = !g.part && g.accumulate;
  float mx = 0.0f;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int nn = bn + wn * WN + j * 16 + oc;
      if (nn >= g.N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = bm + wm * WM + i * 16 + orow + r;
        if (m < g.M) {
          float* p = out + (int64_t)m * ldo + nn;
          const float v = alpha * acc[i][j][r];
          *p = acc_in ? *p + v : v;
          mx = fmaxf(mx, fabsf(v));
        }
      }
    }
  }
  if (g.amax && !g.part) wave_amax_to_slot(mx, g.amax + zb * g.s_amax);  // split partials: the split sum takes it
}

// C = alpha * sum_s part[s] (+ C), splits summed in order
__global__ __launch_bounds__(256) void gemm_split_sum_kernel(GemmArgs g, int splits) {
  const int64_t mn = (int64_t)g.M * g.N;
  const float alpha = gemm_alpha(g);
  float mx = 0.0f;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < mn; i += (int64_t)gridDim.x * blockDim.x) {
    float v = g.part[i];
    for (int s = 1; s < splits; ++s) v += g.part[(int64_t)s * mn + i];
    const int64_t m = i / g.N, nn = i - m * g.N;
    float* p = g.C + m * g.ldc + nn;
    *p = g.accumulate ? *p + alpha * v : alpha * v;
    mx = fmaxf(mx, fabsf(alpha * v));
  }
  if (g.amax) block_amax_to_slot(mx, g.amax);
}

template <int BM, int BN, int WGM, int WGN, bool F16>
static bs_status launch_gemm_lds(const GemmArgs& g0, int splits, hipStream_t st) {
  GemmArgs g = g0;
  const int64_t tiles = (int64_t)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  const int total = (g.K + LBK - 1) / LBK * g.nseg;
  const int cps = (total + splits - 1) / splits;
  splits = (total + cps - 1) / cps;
  if (splits == 1) g.part = nullptr;
  const int64_t nblocks = tiles * (g.batch > 1 ? g.batch : splits);
  if (nblocks > 0x7FFFFFFF) return BS_ESHAPE;
  {
    ProfScope prof("gemm", st, gemm_flops(g), gemm_exec_flops(g));
    gemm_lds_kernel<BM, BN, WGM, WGN, F16><<<(unsigned)nblocks, 64 * WGM * WGN, 0, st>>>(g, cps);
    BS_CHECK_LAUNCH();
  }
  if (splits > 1) {
    const int64_t mn = (int64_t)g.M * g.N;
    const unsigned blocks = (unsigned)std::min<int64_t>((mn + 255) / 256, 8192);
    ProfScope prof("gemm_split_sum", st);
    gemm_split_sum_kernel<<<blocks, 256, 0, st>>>(g, splits);
    BS_CHECK_LAUNCH();
  }
  return BS_OK;
}

template <int BM, int BN, int WGM, int WGN, bool F16>
static bs_status launch_gemm_cfg(const GemmArgs& g, hipStream_t st) {
  const int64_t tiles = (int64_t)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  if (tiles > 0x7FFFFFFF) return BS_ESHAPE;
  ProfScope prof("gemm", st, gemm_flops(g), gemm_exec_flops(g));
  gemm_nt_kernel<BM, BN, WGM, WGN, F16><<<(unsigned)tiles, 256, 0, st>>>(g);
  BS_CHECK_LAUNCH();
  return BS_OK;
}

// ------------------------------------------------------------------------------------
// small-output kernel
// ------------------------------------------------------------------------------------
// A block computes one (16 FM) x (16 FN) tile; its NW waves split the 64-deep k steps of all the
// segments (wave w takes steps w, w + NW, ...), read their fragments straight from global memory
// (a lane's eight k values are 16 contiguous bytes; no LDS staging, no barrier in the loop, the
// next step's loads in flight during a step's MFMAs) and meet once in LDS, where the partial tiles
// are added in wave order. Outputs too small to fill the chip with staged tiles are bound by the
// serial chain of a tile's k steps: this takes the chain apart inside the block, without
// partials in global memory and without a second launch. K any multiple of 8 (the tail reads zero).
template <int FM, int FN, int NW, bool F16>
__global__ __launch_bounds__(64 * NW) void gemm_wave_kernel(GemmArgs g) {
  constexpr int NF = FM * FN;
  __shared__ floatx4 red[NW][NF][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles_n = (g.N + 16 * FN - 1) / (16 * FN), ntile = (g.M + 16 * FM - 1) / (16 * FM) * tiles_n;
  const int nblk = gridDim.x;
  int bid = blockIdx.x;
  if ((nblk & 7) == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);  // XCD-contiguous tiles
  const int zb = bid / ntile, tile = bid - zb * ntile;
  const int bm = tile / tiles_n * (16 * FM), bn = tile % tiles_n * (16 * FN);
  const int ks = (g.K + 63) / 64, total = ks * g.nseg;
  const int fr = lane & 15, fk = (lane >> 4) * 8;
  // rows past the edge read the last row (their products are not stored)
  int64_t ra[FM], rb[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) ra[i] = (int64_t)zb * g.sA + (int64_t)min(bm + i * 16 + fr, g.M - 1) * g.lda;
#pragma unroll
  for (int j = 0; j < FN; ++j) rb[j] = (int64_t)zb * g.sB + (int64_t)min(bn + j * 16 + fr, g.N - 1) * g.ldb;

  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  bf16x8 fa[2][2][FM], fb[2][2][FN];  // [stage][32-deep half][fragment]
  auto load = [&](int st, int s) {
    const int seg = s / ks;
    const u16 *A = g.A[seg], *B = g.B[seg];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = (s - seg * ks) * 64 + 32 * h + fk;
      const bool ok = k < g.K;
#pragma unroll
      for (int i = 0; i < FM; ++i) fa[st][h][i] = ok ? *(const bf16x8*)(A + ra[i] + k) : bf16x8{};
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[st][h][j] = ok ? *(const bf16x8*)(B + rb[j] + k) : bf16x8{};
    }
  };
  auto mma = [&](int st) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          if constexpr (F16)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, fa[st][h][i]),
                                                               __builtin_bit_cast(halfx8, fb[st][h][j]), acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[st][h][i], fb[st][h][j], acc[i][j], 0, 0, 0);
        }
  };
  if (wave < total) load(0, wave);
  for (int s = wave; s < total; s += 2 * NW) {
    if (s + NW < total) load(1, s + NW);
    mma(0);
    if (s + NW < total) {
      if (s + 2 * NW < total) load(0, s + 2 * NW);
      mma(1);
    }
  }
  if (wave < total) {
#pragma unroll
    for (int f = 0; f < NF; ++f) red[wave][f][lane] = acc[f / FN][f % FN];
  }
  __syncthreads();
  // wave w finishes fragments w, w + NW, ...; D[i][j] of a 16 x 16 tile sits in lane
  // (j + 16 (i / 4)), register i % 4
  const int np = min(NW, total);
  const int oc = lane & 15, orow = (lane >> 4) * 4;
  const float alpha = gemm_alpha(g, zb);
  float* out = g.C + (int64_t)zb * g.sC;
  float mx = 0.0f;
#pragma unroll
  for (int f0 = 0; f0 < NF; f0 += NW) {
    const int f = f0 + wave;
    if (f >= NF) break;
    floatx4 v = red[0][f][lane];
    for (int w = 1; w < np; ++w) v += red[w][f][lane];
    const int n = bn + f % FN * 16 + oc;
    if (n >= g.N) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = bm + f / FN * 16 + orow + r;
      if (m < g.M) {
        float* p = out + (int64_t)m * g.ldc + n;
        const float o = alpha * v[r];
        *p = g.accumulate ? *p + o : o;
        mx = fmaxf(mx, fabsf(o));
      }
    }
  }
  if (g.amax) wave_amax_to_slot(mx, g.amax + zb * g.s_amax);
}

template <int FM, int FN, int NW, bool F16>
static bs_status launch_gemm_wave(const GemmArgs& g, hipStream_t st) {
  const int64_t blocks = (int64_t)((g.M + 16 * FM - 1) / (16 * FM)) * ((g.N + 16 * FN - 1) / (16 * FN)) * g.batch;
  if (blocks > 0x7FFFFFFF) return BS_ESHAPE;
  ProfScope prof("gemm", st, gemm_flops(g), gemm_exec_flops(g));
  gemm_wave_kernel<FM, FN, NW, F16><<<(unsigned)blocks, 64 * NW, 0, st>>>(g);
  BS_CHECK_LAUNCH();
  return BS_OK;
}

// Which kernel, and how many splits of K: the least estimated time of the pipelined kernel's 256 x 256
// and 128 x 128 tiles (one and two blocks per CU) and the small-output kernel's 32 x 32 tiles.
// The times (us) are fitted to launches of 141 shapes from 64 x 64 x 64 to 8192 x 8192 x 2048: a fixed
// part, and per 64-deep chunk of a block a part that grows as more blocks load and multiply at once (n
// chunks per block, f the share of the blocks the CUs hold, r rounds of them):
//   256 x 256   13 + n (0.95 + 0.6 f)     4096^2 x 1024: 38 measured, 38 estimated
//     rounds    each 12.5 + n (0.98 + 0.38 f^4), the first 2.5 more   8192 x 4096 x 1024: 72 and 71
//   128 x 128   6.5 + n (0.42 + 0.6 f)    2048 x 4096 x 1024: 24 and 23; 640^2 x 2816: 25 and 26
//     rounds    each 3 + 3 f + n (0.4 + 0.44 f), the first 4.7 more   16384 x 1024 x 512: 30 and 30
//   32 x 32     2.4 + 1.9 n/8 r           512^2 x 1536: 8.7 and 8.1 (its 8 waves share the chunks; the rounds
//               of a few chunks overlap, of more count whole: 768^2 x 2048 24 and 25)
//   split sum   4 + s M N 1e-6 (the partials out and in, and the launch)
// (By output size alone, 256 x 256 from M N = 2^20, these took 33.3, 19.3 with 128 x 128, at 4160 x
// 776 x 1152; 28.6, now 14.4, at 4096 x 512 x 1024; 16.3, now 8.7, at 512^2 x 1536. With every round
// counted by its fraction and no fixed part 16384 x 1024 x 512 took 28.5 with 128 x 128, 25.1 with 256 x
// 256, and 768^2 x 2048 24.0 with 32 x 32, 20.1 with 128 x 128.)
struct GemmPlan {
  int kind = 0;  // 0: 256 x 256, 1: 128 x 128, 2: 32 x 32
  int splits = 1;
};
// kind's time for `blocks` blocks of n chunks each
static double gemm_estimate(int kind, double blocks, int n) {
  const double cap = kind == 1 ? 512 : 256, r = blocks / cap;
  if (kind == 2) return 2.4 + 1.9 * ((n + 7) / 8) * std::max(1.0, n < 24 ? r : std::ceil(r));
  if (r <= 1.0) return (kind == 0 ? 13.0 : 6.5) + n * ((kind == 0 ? 0.95 : 0.42) + 0.6 * r);
  auto round = [&](double f) {
    return kind == 0 ? 12.5 + n * (0.98 + 0.38 * f * f * f * f) : 3.0 + 3.0 * f + n * (0.4 + 0.44 * f);
  };
  const double full = std::floor(r);
  return (kind == 0 ? 2.5 : 4.7) + full * round(1.0) + (r > full ? round(r - full) : 0.0);
}
static GemmPlan plan_gemm(const GemmArgs& g) {
  const int total = (int)std::min<int64_t>((int64_t)((g.K + LBK - 1) / LBK) * g.nseg, 1 << 30);
  const int top = g.part && g.batch == 1 ? (int)std::min<int64_t>(16, std::min<int64_t>(total / 2, g.part_cap / ((int64_t)g.M * g.N))) : 1;
  GemmPlan best;
  double tb = 1e300;
  for (int kind = 0; kind < 3; ++kind) {
    const int bt = kind == 0 ? 256 : (kind == 1 ? 128 : 32);
    const double tiles = (double)((g.M + bt - 1) / bt) * ((g.N + bt - 1) / bt) * g.batch;
    for (int s = 1; s <= (kind == 2 ? 1 : std::max(1, top)); ++s) {
      if (s > 1 && tiles * s > (kind == 0 ? 256 : 512)) break;  // more blocks than the CUs hold gain nothing
      double t = gemm_estimate(kind, tiles * s, (total + s - 1) / s);
      if (s > 1) t += 4.0 + s * (double)g.M * g.N * 1e-6;
      if (t < tb) tb = t, best.kind = kind, best.splits = s;
    }
  }
  return best;
}

template <bool F16>
static bs_status launch_gemm_planned(const GemmArgs& g, hipStream_t st) {
  const GemmPlan p = plan_gemm(g);
  if (p.kind == 2) return launch_gemm_wave<2, 2, 8, F16>(g, st);
  return p.kind == 0 ? launch_gemm_lds<256, 256, 2, 4, F16>(g, p.splits, st)
                     : launch_gemm_lds<128, 128, 2, 2, F16>(g, p.splits, st);
}

bs_status launch_gemm(const GemmArgs& g, hipStream_t st) {
  if (g.M <= 0 || g.N <= 0) return BS_OK;
  if (g.nseg < 1 || g.nseg > GEMM_MAX_SEG) return BS_EINVAL;
  if ((g.K & 7) || (g.lda & 7) || (g.ldb & 7) || g.lda < g.K || g.ldb < g.K) return BS_ESHAPE;
  if (g.amax && g.accumulate) return BS_EINVAL;
  if (g.batch < 1 || (g.batch > 1 && (g.sA < 0 || g.sB < 0 || g.sC < 0 || g.s_alpha2 < 0))) return BS_EINVAL;
  if (g.K == 0) return g.accumulate ? BS_OK : launch_fill2d(g.C, g.M, g.N, g.ldc, 0.0f, st);
  // buffer offsets of one 256-row tile fit in 31 bits
  bool lds_ok = g.lda < (1 << 21) && g.ldb < (1 << 21);
  for (int i = 0; i < g.nseg; ++i) lds_ok = lds_ok && ((uintptr_t)g.A[i] & 15) == 0 && ((uintptr_t)g.B[i] & 15) == 0;
  if (lds_ok) return g.f16 ? launch_gemm_planned<true>(g, st) : launch_gemm_planned<false>(g, st);
  if (g.amax || g.batch > 1) return BS_EINVAL;  // maxima, batches: aligned operands only
  return g.f16 ? launch_gemm_cfg<128, 128, 2, 2, true>(g, st) : launch_gemm_cfg<128, 128, 2, 2, false>(g, st);
}

}  // namespace bsp
