// Gradient path, a stage of radix 9 .. 48 whose stride is a multiple of 16 (the leftover prime of a schedule, 43 of
// 11008) on the matrix cores, one launch: dK[c] = sum over rows of x^T g and g K^T of the same rows.
//
// A workgroup owns 16 neighbouring blocks (runs of 64 bytes of a row) and a chunk of rows, 16 rows a step: x and g
// come in 16-byte pieces into LDS tiles [j][block][row], wave w multiplies blocks w and 8 + w with
// v_mfma_f32_16x16x4_f32 (float32 operands: x^T g over the rows, one value j per lane; g K^T with the block's
// values in registers for the whole launch), and what is passed back leaves through the places that g came in.  The sums of
// a step are made from zero and then added to the chunk's.  They leave block by block, in the order dK has.
// Rows step by step: x and the product share a tile with nobody, g has two, so that a step's last pieces leave while the
// next step's rows arrive; two barriers a step.
//
// Two launches, each with 16 waves, read g twice and wrote partial sums of 64 rows through LDS.  1537 x 11008 float32
// (8, 8, 4, 43): 84 us (sums) + 42 (passed back) + 22 (reduction) -> 88 + 6; whole calls 302 -> 242 us, 64 rows bf16 82 -> 53.
// What is left: 233 MB at 2.6 TB/s, as every kernel does that takes 64-byte pieces a kilobyte apart (the matrix instructions are busy
// 37 % of the time).  Without effect: the block's values read again every step from the L2 (88 us either way), stores without
// conditions, the next rows asked for earlier or later in a step.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "harp_internal.h"
#include "harp_mfma4.h"

namespace harp {
namespace {

constexpr int kBigThreads = 512, kBigWaves = kBigThreads / 64, kBigRows = 16;
// Place of (j, block, row) in a tile: blocks k, 4 + k, 8 + k, 12 + k of 16 rows, which a wave moves together, are 64
// neighbouring places, and 4 kBigJ = 16 mod 64 spreads a wave's operands and 16-byte pieces over the banks.
constexpr int kBigJ = 16 * kBigRows + 4, kBigStep = 4 * kBigRows;
__device__ __forceinline__ int big_slot(int block) { return (4 * (block & 3) + (block >> 2)) * kBigRows; }

template <int KT, typename TG>
__global__ __launch_bounds__(kBigThreads, 2) void harp_grad_big_bwd_kernel(
    const float *__restrict__ X, const TG *__restrict__ G, int64_t ldg, float *__restrict__ Gout, int64_t d, int64_t n,
    int rows, int S, int b, int gx, int share, const f4v *__restrict__ operands, float *__restrict__ partial) {
  constexpr int TILE = 16 * KT * kBigJ, MAXG = (kBigRows * 16 * KT * 4 + kBigThreads - 1) / kBigThreads;
  __shared__ __attribute__((aligned(16))) float lds[3 * TILE];
  const int tid = (int)threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6) & 7;
  const int l = tid & 63, g = l >> 4, c16 = l & 15;
  unsigned wg = blockIdx.x;
  if (share > 1) {   // block tiles that share lines go to one XCD
    const unsigned xcd = wg & 7u, k = wg >> 3;
    wg = ((k / share) * 8u + xcd) * share + k % share;
  }
  const int q0 = (int)(wg % (unsigned)gx) * 16, chunk = (int)(wg / (unsigned)gx);
  const int base = (q0 / S) * b * S + q0 % S;
  const int64_t r0 = (int64_t)chunk * rows, r1 = r0 + rows < n ? r0 + rows : n;

  // This thread's pieces: blocks 4 lo4 .. 4 lo4 + 3 of one row and values j = w, w + 8 .. (past the radix the last one once
  // more: the same places, the same values).
  const int lo4 = tid & 3, row = (tid >> 2) % kBigRows;
  const int col = base + 4 * lo4, place = big_slot(4 * lo4) + row;
  auto value = [&](int u) { return w + kBigWaves * u < b ? w + kBigWaves * u : b - 1; };
  typedef typename std::conditional<sizeof(TG) == 2, uint2, f4v>::type raw_t;   // four elements of G as loaded
  f4v px[MAXG];
  raw_t pg[MAXG];
  auto fetch = [&](int64_t first) {   // rows past the end repeat the last one
    const int64_t r = first < r1 ? first : r1 - 1;
    const int last = (int)(r1 - 1 - r);
    const uint32_t at = (uint32_t)(row < last ? row : last);
    const float *xr = X + r * d;
    const TG *gr = G + r * ldg;
#pragma unroll
    for (int u = 0; u < MAXG; ++u) {
      px[u] = *reinterpret_cast<const f4v *>(xr + value(u) * S + (at * (uint32_t)d + (uint32_t)col));
      pg[u] = *reinterpret_cast<const raw_t *>(gr + value(u) * S + (at * (uint32_t)ldg + (uint32_t)col));
    }
  };
  fetch(r0);
  const BlockValues<1024> val = {__builtin_amdgcn_make_buffer_rsrc(const_cast<f4v *>(operands + (size_t)q0 * (KT * KT * 64)), 0,
                                                              16 * KT * KT * 1024, 0x00020000),
                                 l * 16};
  f4v K[2][KT][KT];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int t = 0; t < KT * KT; ++t) K[h][t / KT][t % KT] = val.piece((w + 8 * h) * KT * KT, t);
  f4v sum[2][KT][KT];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int t = 0; t < KT * KT; ++t) sum[h][t / KT][t % KT] = (f4v){0.f, 0.f, 0.f, 0.f};
  float *tx = lds, *tg = lds + TILE, *tother = lds + 2 * TILE;

  for (int64_t r = r0; r < r1; r += kBigRows) {
    const int left = (int)(r1 - r < kBigRows ? r1 - r : kBigRows);
#pragma unroll
    for (int u = 0; u < MAXG; ++u) {
      f4v gv;
      if constexpr (sizeof(TG) == 2)
        gv = (f4v){__uint_as_float(pg[u].x << 16), __uint_as_float(pg[u].x & 0xffff0000u), __uint_as_float(pg[u].y << 16),
                   __uint_as_float(pg[u].y & 0xffff0000u)};
      else
        gv = pg[u];
#pragma unroll
      for (int k = 0; k < 4; ++k) {   // rows past the end enter as zeros
        tx[value(u) * kBigJ + place + k * kBigStep] = row < left ? px[u][k] : 0.f;
        tg[value(u) * kBigJ + place + k * kBigStep] = row < left ? gv[k] : 0.f;
      }
    }
    fetch(r + kBigRows);
    lds_barrier();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int slot = big_slot(w + 8 * h);
      f4v gv[KT];   // rows 4 g .. 4 g + 3 of value 16 t + c16 (past the radix: whatever lies there)
#pragma unroll
      for (int t = 0; t < KT; ++t) gv[t] = *reinterpret_cast<const f4v *>(tg + (16 * t + c16) * kBigJ + slot + 4 * g);
#pragma unroll
      for (int m = 0; m < KT; ++m) {
        const f4v xv = *reinterpret_cast<const f4v *>(tx + (16 * m + c16) * kBigJ + slot + 4 * g);
        f4v few[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) few[t] = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i)   // row 4 g + i: every row once
#pragma unroll
          for (int t = 0; t < KT; ++t) few[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[i], gv[t][i], few[t], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < KT; ++t) {
          sum[h][m][t] += few[t];
          asm volatile("" : "+v"(sum[h][m][t]));   // here, not all at the end of the step
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      f4v back[KT];
#pragma unroll
      for (int t = 0; t < KT; ++t) back[t] = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int m = 0; m < KT; ++m) {
        float a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = tg[(16 * m + 4 * g + i) * kBigJ + slot + c16];
          a[i] = 16 * m + 4 * g + i < b ? v : 0.f;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int t = 0; t < KT; ++t) back[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], K[h][m][t][i], back[t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      wave_fence();   // (no other wave touches this block's places)
#pragma unroll
      for (int t = 0; t < KT; ++t)
        if (16 * t + c16 < b) *reinterpret_cast<f4v *>(tg + (16 * t + c16) * kBigJ + slot + 4 * g) = back[t];
      __builtin_amdgcn_sched_barrier(0);
    }
    lds_barrier();
    if (row < left) {
      float *out = Gout + r * d;
      const uint32_t own = (uint32_t)row * (uint32_t)d + (uint32_t)col;
#pragma unroll
      for (int u = 0; u < MAXG; ++u) {
        const float *t = tg + value(u) * kBigJ + place;
        *reinterpret_cast<f4v *>(out + value(u) * S + own) = (f4v){t[0], t[kBigStep], t[2 * kBigStep], t[3 * kBigStep]};
      }
    }
    float *const swap = tg;   // its pieces leave under the next step
    tg = tother;
    tother = swap;
  }
  // sums of the chunk: [block][value]
  const int bb = b * b, D = (int)(d / b);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float *out = partial + ((size_t)chunk * D + q0 + w + 8 * h) * bb;
#pragma unroll
    for (int m = 0; m < KT; ++m)
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int j = 16 * m + 4 * g + i, j2 = 16 * t + c16;
          if (j < b && j2 < b) out[j * b + j2] = sum[h][m][t][i];
        }
  }
}

// dK = the chunks' sums in ascending order within each eight, then the eights in ascending order; with SL slices of the
// chunks, the slices in ascending order behind that.  A thread's eights follow one another, so few blocks with many chunks
// want slices: 144 x 9 values leave two workgroups a serial walk over 250 chunks (4000 x 144 float32 (4, 4, 9), whole call 65 -> 49 us;
// 100000 x 528 (4, 4, 33), 782 chunks, 1628 -> 1572).  (dK is the caller's: four stores where it is not on a boundary of 16 bytes.)
constexpr int kBigSumThreads = 256;
template <int SL>
__global__ __launch_bounds__(kBigSumThreads) void harp_grad_big_sum_kernel(const f4v *__restrict__ partial, int nchunks,
                                                                           size_t total, int aligned, float *__restrict__ dK) {
  constexpr int Q = kBigSumThreads / SL;   // quads of a workgroup
  const int slice = (int)threadIdx.x / Q;
  const size_t own = (size_t)blockIdx.x * Q + threadIdx.x % Q, e = own < total ? own : total - 1;
  const int per = ((nchunks + SL - 1) / SL + 7) / 8 * 8, k0 = slice * per, k1 = k0 + per < nchunks ? k0 + per : nchunks;
  f4v s = {0.f, 0.f, 0.f, 0.f};
  for (int k = k0; k < k1; k += 8) {
    f4v v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = partial[(size_t)(k + u < k1 ? k + u : k) * total + e];
    f4v part = v[0];
#pragma unroll
    for (int u = 1; u < 8; ++u)
      if (k + u < k1) part += v[u];
    s += part;
  }
  if constexpr (SL > 1) {
    __shared__ f4v sums[kBigSumThreads];
    sums[threadIdx.x] = s;
    __syncthreads();
    if (slice > 0) return;
#pragma unroll
    for (int i = 1; i < SL; ++i) s += sums[i * Q + threadIdx.x];
  }
  if (own >= total) return;
  if (aligned) {
    *reinterpret_cast<f4v *>(dK + 4 * e) = s;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) dK[4 * e + i] = s[i];
  }
}

// Chunks of rows that fill the chip once, one workgroup per compute unit, and how often that is done so that no workgroup has
// more than 128 rows.
int64_t big_round(const harp_plan *plan, int64_t gx) { return std::max<int64_t>(1, (plan->num_cu > 0 ? plan->num_cu : 256) / gx); }
int64_t big_rounds(const harp_plan *plan, int64_t n, int64_t gx) {
  return std::max<int64_t>(1, ((n + 127) / 128 + big_round(plan, gx) - 1) / big_round(plan, gx));
}
// Rows of a workgroup, in whole steps: the rounds share them evenly (128 each left a last round nearly empty: 33000 x 528
// float32 (4, 4, 33), 258 workgroups, whole call 497 -> 459 us).
int big_rows(const harp_plan *plan, int64_t n, int64_t gx) {
  const int64_t chunks = big_rounds(plan, n, gx) * big_round(plan, gx), rows = (n + chunks - 1) / chunks;
  return (int)((rows + kBigRows - 1) / kBigRows * kBigRows);
}

}  // namespace

// The stage at t runs here (the choice depends on the plan alone; X and Gout must then lie on boundaries of 16 bytes, G on
// boundaries of four elements).
bool grad_big_stage(const harp_plan *plan, int t) {
  const int b = plan->radices[t];
  return b >= 9 && b <= 48 && plan->grad_mfma[1].size() > (size_t)t && plan->grad_mfma[1][t].aux != nullptr &&
         (size_t)3 * 16 * ((b + 15) / 16) * kBigJ * 4 <= (size_t)plan->lds_bytes;
}
// (at least as many chunks as there are, and never fewer for more rows)
size_t grad_big_partial_floats(const harp_plan *plan, int t, int64_t n) {
  const int64_t b = plan->radices[t], gx = plan->d / b / 16;
  const int64_t chunks = std::min<int64_t>((n + kBigRows - 1) / kBigRows, big_rounds(plan, n, gx) * big_round(plan, gx));
  return (size_t)std::max<int64_t>(chunks, 1) * (size_t)(plan->d * b);
}

harp_status_t launch_grad_big(const harp_plan *plan, int t, const float *X, const void *G, int64_t ldg, bool bf, float *Gout,
                              int64_t n, float *partial, float *dK, hipStream_t st) {
  const PassDesc &pd = plan->grad_mfma[1][t];
  const int b = pd.b, KT = (b + 15) / 16;
  const int64_t d = plan->d, D = d / b, gx = D / 16;
  const int rows = big_rows(plan, n, gx);
  const int64_t chunks = (n + rows - 1) / rows, total = gx * chunks;
  if (total > 0x7fffffff) return HARP_ERR_UNSUPPORTED;
  const int share = gx % 4 == 0 && total % 32 == 0 ? 4 : 1;
  // the float32 operand tiles follow the bf16 ones of all blocks
  const f4v *operands = reinterpret_cast<const f4v *>(static_cast<const uint16_t *>(pd.aux) + (size_t)pd.nqp * KT * KT * 2 * 64 * 4);
#define HARP_BIG_T(T, TG)                                                                                              \
  hipLaunchKernelGGL((harp_grad_big_bwd_kernel<T, TG>), dim3((unsigned)total), dim3(kBigThreads), 0, st, X, (const TG *)G, \
                     ldg, Gout, d, n, rows, (int)pd.S, b, (int)gx, share, operands, partial)
#define HARP_BIG(T)                     \
  do {                                  \
    if (bf) HARP_BIG_T(T, uint16_t);    \
    else HARP_BIG_T(T, float);          \
  } while (0)
  if (KT == 1) HARP_BIG(1);
  else if (KT == 2) HARP_BIG(2);
  else HARP_BIG(3);
#undef HARP_BIG
#undef HARP_BIG_T
  const size_t quads = (size_t)(d * b / 4);   // D is a multiple of 16
#define HARP_BIG_SUM(SL)                                                                                                   \
  hipLaunchKernelGGL((harp_grad_big_sum_kernel<SL>), dim3((unsigned)((quads * SL + kBigSumThreads - 1) / kBigSumThreads)), \
                     dim3(kBigSumThreads), 0, st, reinterpret_cast<const f4v *>(partial), (int)chunks, quads,              \
                     (uintptr_t)dK % 16 == 0 ? 1 : 0, dK)
  // (16 chunks are two steps of a thread, and 65536 quads a workgroup per compute unit)
  if (chunks <= 16 || quads >= 65536) HARP_BIG_SUM(1);
  else if (chunks <= 64) HARP_BIG_SUM(4);
  else HARP_BIG_SUM(16);
#undef HARP_BIG_SUM
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

}  // namespace harp
