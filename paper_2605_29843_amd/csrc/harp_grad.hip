// Backward of Y = X U with respect to the block kernels and to X -- the gradient that the
// update of the layerwise fitting procedure (Algorithm 3) needs, by the chain rule through
// Algorithm 1.  With x_0 = X diag(sigma), x_{t+1} = stage_t(x_t) and g_m = G = dL/dY:
//     dK_t[c] = sum over rows of x_t[idx]^T g_{t+1}[idx],     g_t[idx] = g_{t+1}[idx] K_t[c]^T,
// idx = the b_t coordinates alpha b s + r s + beta of block c = alpha s + beta, and dX = g_0
// diag(sigma).  Nothing is assumed about the blocks (they need not be orthogonal).
//
// Segment by segment through device memory: the forward pass keeps the input of every segment
// (float32 copies of the batch in the workspace; the first segment, and the last one on the way
// back, use the caller's rows where their kernel can), the backward pass runs one kernel per segment
// that passes g back and leaves per-row-chunk partial sums of dK, and a reduction kernel adds the
// chunks in a fixed order (no atomics: results are reproducible).  The segments:
//   - the stages of the first 64 coordinates together (radix 2 or 8, orthogonal), and behind them eight
//     coordinates and up to eight more in one launch (harp_grad_pair.hip; harp_grad_seg.hip, forward);
//   - up to three consecutive radix-2 stages: a thread owns the 2^k coordinates base + e s and the
//     k 2^(k-1) blocks that act on them, the forward kernel stores only the run's output, and the
//     backward kernel recomputes the run's inner activations in registers;
//   - one stage of radix up to 8: a thread owns one block for a chunk of rows, its b*b values and b*b
//     accumulators in registers, g in place;
//   - one stage of radix 9 .. 64, g out of place: on the matrix cores where the stride is a multiple
//     of 16 (up to 48 in one launch, harp_grad_big.hip), else one value per thread.
// All read the plan's dense per-stage image with the signs folded into stage 0 (the one the
// column-mode passes use).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "harp_internal.h"
#include "harp_mfma4.h"

namespace harp {
namespace {

constexpr int kGradThreads = 256;

// Element i of a row of fewer than 2^24: a scalar row address and a 32-bit byte offset per lane.
template <typename T>
__device__ __forceinline__ T *grad_at(T *row, int i) {
  typedef typename std::conditional<std::is_const<T>::value, const char, char>::type byte_t;
  return reinterpret_cast<T *>(reinterpret_cast<byte_t *>(row) + (uint32_t)i * (uint32_t)sizeof(T));
}

__device__ __forceinline__ float grad_widen(float v) { return v; }
__device__ __forceinline__ float grad_widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ void grad_narrow(float v, float *p) { *p = v; }
__device__ __forceinline__ void grad_narrow(float v, uint16_t *p) {
  const uint32_t u = __float_as_uint(v);
  const uint32_t rounded = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  const uint32_t quiet = (u >> 16) | 0x40u;
  *p = (uint16_t)(((u & 0x7fffffffu) > 0x7f800000u) ? quiet : rounded);
}

// dst[r, c] = convert(src[r, c]); VEC: eight elements per thread with 16-byte accesses on the
// two-byte side (d a multiple of 8, rows and pointers on 16-byte boundaries)
template <typename TS, typename TD, bool VEC>
__global__ __launch_bounds__(kGradThreads) void harp_grad_convert_kernel(
    const TS *__restrict__ src, int64_t lds_, TD *__restrict__ dst, int64_t ldd, int64_t n, int d) {
  const int64_t row = blockIdx.y;
  if (VEC) {
    for (int c = 8 * (blockIdx.x * kGradThreads + threadIdx.x); c < d; c += 8 * gridDim.x * kGradThreads) {
      float v[8];
      const TS *sp = src + row * lds_ + c;
      TD *dp = dst + row * ldd + c;
      if (sizeof(TS) == 2) {
        const uint4 raw = *reinterpret_cast<const uint4 *>(sp);
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[2 * i] = __uint_as_float(w[i] << 16);
          v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
      } else {
        const float4 a = *reinterpret_cast<const float4 *>(sp), b = *reinterpret_cast<const float4 *>(sp + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
      }
      if (sizeof(TD) == 2) {
        uint16_t h[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) grad_narrow(v[i], reinterpret_cast<uint16_t *>(&h[i]));
        *reinterpret_cast<uint4 *>(dp) =
            make_uint4(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16),
                       h[4] | ((uint32_t)h[5] << 16), h[6] | ((uint32_t)h[7] << 16));
      } else {
        *reinterpret_cast<float4 *>(dp) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(dp) + 4) = make_float4(v[4], v[5], v[6], v[7]);
      }
    }
  } else {
    for (int c = blockIdx.x * kGradThreads + threadIdx.x; c < d; c += gridDim.x * kGradThreads)
      grad_narrow(grad_widen(src[row * lds_ + c]), dst + row * ldd + c);
  }
  (void)n;
}

// y[idx] = x[idx] K[c] for every row of the chunk blockIdx.y
template <int B>
__global__ __launch_bounds__(kGradThreads) void harp_grad_fwd_kernel(
    const float *__restrict__ X, float *__restrict__ Y, int64_t ld, int64_t n, int rows,
    const float *__restrict__ blocks, int D, int s) {
  const int c = blockIdx.x * kGradThreads + threadIdx.x;
  if (c >= D) return;
  float K[B * B];
#pragma unroll
  for (int v = 0; v < B * B; ++v) K[v] = blocks[(size_t)c * (B * B) + v];
  const int base = (c / s) * B * s + c % s;
  const int64_t r0 = (int64_t)blockIdx.y * rows;
  const int64_t r1 = (r0 + rows < n) ? r0 + rows : n;
  for (int64_t row = r0; row < r1; ++row) {
    const float *x = X + row * ld + base;
    float *y = Y + row * ld + base;
    float v[B];
#pragma unroll
    for (int r = 0; r < B; ++r) v[r] = x[(size_t)r * s];
#pragma unroll
    for (int r2 = 0; r2 < B; ++r2) {
      float acc = 0.f;
#pragma unroll
      for (int r = 0; r < B; ++r) acc = fmaf(v[r], K[r * B + r2], acc);
      y[(size_t)r2 * s] = acc;
    }
  }
}

// Backward kernels: a workgroup is 128 items x four groups of rows.  The partial sums of a stage's block
// gradients are a fifth of the bytes such a kernel moves when every 8 rows write theirs; the four groups
// add theirs in LDS first, in a fixed order (2048 x 4096 bf16 radix 2: a run of three stages 20 -> 18 - 19 us, its
// reduction 5.7 -> 4.5; 1537 x 11008 float32: radix-4 stage 45 -> 38 us, reduction 8.0 -> 5.2).
constexpr int kSumItems = 128, kSumGroups = 4, kSumThreads = kSumItems * kSumGroups;
struct SumRows {
  int item, group;
  int64_t r0, r1;   // rows of this group
};
__device__ __forceinline__ SumRows sum_rows(int64_t n, int rows) {
  SumRows sr;
  sr.item = (int)threadIdx.x % kSumItems;
  sr.group = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kSumItems);   // whole waves: row addresses are scalar
  const int per = (rows + kSumGroups - 1) / kSumGroups;
  const int64_t w0 = (int64_t)blockIdx.y * rows, w1 = (w0 + rows < n) ? w0 + rows : n;
  sr.r0 = w0 + (int64_t)sr.group * per;
  sr.r1 = (sr.r0 + per < w1) ? sr.r0 + per : w1;
  return sr;
}
// acc of group 0 <- (group 0 + group 2) + (group 1 + group 3); every thread of the workgroup takes part
// (red: 2 NV kSumItems floats of LDS that nobody uses any more)
template <int NV>
__device__ __forceinline__ void sum_groups(float (&acc)[NV], const SumRows &sr, float *red) {
  auto at = [&](int half, int v) -> float & { return red[(half * NV + v) * kSumItems + sr.item]; };
  if (sr.group >= 2) {
#pragma unroll
    for (int v = 0; v < NV; ++v) at(sr.group - 2, v) = acc[v];
  }
  __syncthreads();
  if (sr.group < 2) {
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] += at(sr.group, v);
  }
  if (sr.group == 1) {   // into the slots that this thread alone has read
#pragma unroll
    for (int v = 0; v < NV; ++v) at(1, v) = acc[v];
  }
  __syncthreads();
  if (sr.group == 0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] += at(1, v);
  }
}

// For the rows of chunk blockIdx.y: acc[r][r2] += x[idx_r] g[idx_r2];  g[idx_r] <- sum_r2
// g[idx_r2] K[r][r2] (in place).  Partial sums go to partial[(chunk * B*B + v) * D + c].
// The blocks of a workgroup lie one after the other in memory.  From radix 5 on they enter by whole lines
// through LDS (odd pitch: 64 blocks spread over the banks) under the first rows' way: with each lane
// fetching its own block, 64 lines a load, the kernel of 4096 radix 8 took 14.6 instead of 9.1 us at 256
// rows and 21.5 instead of 19.5 us at 2048.  Smaller blocks are fetched by their lanes (radix 4: 1.5 % faster).
template <int B>
__global__ __launch_bounds__(kSumThreads) void harp_grad_bwd_kernel(
    const float *__restrict__ X, float *__restrict__ Gm, int64_t ld, int64_t n, int rows,
    const float *__restrict__ blocks, int D, int s, float *__restrict__ partial) {
  const SumRows sr = sum_rows(n, rows);
  const int c0 = blockIdx.x * kSumItems + sr.item, c = c0 < D ? c0 : D - 1;
  constexpr int BB = B * B, PITCH = BB | 1, NK = (kSumItems * BB + kSumThreads - 1) / kSumThreads;
  constexpr bool STAGED = B > 4;
  static_assert(PITCH <= 2 * BB, "the blocks fit in the space of the sums");
  __shared__ float red[2 * BB * kSumItems];
  const int first = (int)blockIdx.x * kSumItems;
  const int left = (D - first < kSumItems ? D - first : kSumItems) * BB;   // block values of the workgroup
  float K[BB], acc[BB], kk[NK], nx[B], ng[B];
  if constexpr (STAGED) {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int at = (int)threadIdx.x + i * kSumThreads;
      kk[i] = blocks[(size_t)first * BB + (at < left ? at : 0)];
    }
  } else {
#pragma unroll
    for (int v = 0; v < BB; ++v) K[v] = blocks[(size_t)c * BB + v];
  }
  const int base = (c / s) * B * s + c % s;
  const int64_t r1 = c0 < D ? sr.r1 : sr.r0;   // threads past the last block have no rows
  auto request = [&](int64_t row) {
#pragma unroll
    for (int r = 0; r < B; ++r) {
      nx[r] = *grad_at(X + row * ld, base + r * s);
      ng[r] = *grad_at(Gm + row * ld, base + r * s);
    }
  };
  if (sr.r0 < r1) request(sr.r0);
  if constexpr (STAGED) {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int at = (int)threadIdx.x + i * kSumThreads;
      if (at < left) red[at / BB * PITCH + at % BB] = kk[i];
    }
    lds_barrier();   // the first rows stay on their way
#pragma unroll
    for (int v = 0; v < BB; ++v) K[v] = red[(c - first) * PITCH + v];
  }
#pragma unroll
  for (int v = 0; v < BB; ++v) acc[v] = 0.f;
  for (int64_t row = sr.r0; row < r1; ++row) {
    float *g = Gm + row * ld;
    float xv[B], gv[B];
#pragma unroll
    for (int r = 0; r < B; ++r) {
      xv[r] = nx[r];
      gv[r] = ng[r];
    }
    if (row + 1 < r1) request(row + 1);   // (nobody but this thread writes its g)
#pragma unroll
    for (int r = 0; r < B; ++r) {
      float back = 0.f;
#pragma unroll
      for (int r2 = 0; r2 < B; ++r2) {
        acc[r * B + r2] = fmaf(xv[r], gv[r2], acc[r * B + r2]);
        back = fmaf(gv[r2], K[r * B + r2], back);
      }
      *grad_at(g, base + r * s) = back;
    }
  }
  if constexpr (STAGED) __syncthreads();   // everyone has its block
  sum_groups<BB>(acc, sr, red);
  if (sr.group == 0 && c0 < D) {
#pragma unroll
    for (int v = 0; v < B * B; ++v)
      partial[((size_t)blockIdx.y * (B * B) + v) * D + c] = acc[v];
  }
}

// Radix 9..64 (the leftover prime of a schedule): a block no longer fits one thread's registers,
// so thread (c, j) owns one column or row of it.  TR false: y[j] = sum_r x[r] K[r][j] (the stage
// itself); TR true: y[j] = sum_r x[r] K[j][r] (the gradient passed back through it).  Out of
// place.  Workgroup = 64 consecutive blocks c x 4 values of j; blockIdx.z covers the other j.
// BMAX = the radix rounded up to a multiple of 16: the loads of a row are unconditional (index
// clamped to the last coordinate of the block, value replaced by zero), so that all of them are
// in flight together; under a per-load condition each one was waited for before the next was
// issued and the three launches of the radix-43 stage of 11008 took 1 ms each.
template <int BMAX, bool TR>
__global__ __launch_bounds__(kGradThreads) void harp_grad_apply_big_kernel(
    const float *__restrict__ X, float *__restrict__ Y, int64_t ld, int64_t n, int rows,
    const float *__restrict__ blocks, int D, int s, int b) {
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int j = blockIdx.z * 4 + (threadIdx.x >> 6);
  if (c >= D || j >= b) return;
  float kv[BMAX];
  const float *kb = blocks + (size_t)c * b * b;
#pragma unroll
  for (int r = 0; r < BMAX; ++r) {
    const int rc = r < b ? r : b - 1;
    const float v = TR ? kb[j * b + rc] : kb[rc * b + j];
    kv[r] = r < b ? v : 0.f;
  }
  const int base = (c / s) * b * s + c % s;
  const int64_t r0 = (int64_t)blockIdx.y * rows;
  const int64_t r1 = (r0 + rows < n) ? r0 + rows : n;
  for (int64_t row = r0; row < r1; ++row) {
    const float *x = X + row * ld + base;
    float xv[BMAX];
#pragma unroll
    for (int r = 0; r < BMAX; ++r) xv[r] = x[(size_t)(r < b ? r : b - 1) * s];
    float acc = 0.f;
#pragma unroll
    for (int r = 0; r < BMAX; ++r) acc = fmaf(r < b ? xv[r] : 0.f, kv[r], acc);
    Y[row * ld + base + (size_t)j * s] = acc;
  }
}

// Thread (c, r2) accumulates column r2 of dK[c] over the rows of chunk blockIdx.y:
// acc[r] += x[idx_r] g[idx_r2]; partial sums in the layout of the small-radix kernel.
template <int BMAX>
__global__ __launch_bounds__(kGradThreads) void harp_grad_dk_big_kernel(
    const float *__restrict__ X, const float *__restrict__ Gm, int64_t ld, int64_t n, int rows,
    int D, int s, int b, float *__restrict__ partial) {
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int r2 = blockIdx.z * 4 + (threadIdx.x >> 6);
  if (c >= D || r2 >= b) return;
  float acc[BMAX];
#pragma unroll
  for (int r = 0; r < BMAX; ++r) acc[r] = 0.f;
  const int base = (c / s) * b * s + c % s;
  const int64_t r0 = (int64_t)blockIdx.y * rows;
  const int64_t r1 = (r0 + rows < n) ? r0 + rows : n;
  for (int64_t row = r0; row < r1; ++row) {
    const float *x = X + row * ld + base;
    const float gv = Gm[row * ld + base + (size_t)r2 * s];
    float xv[BMAX];
#pragma unroll
    for (int r = 0; r < BMAX; ++r) xv[r] = x[(size_t)(r < b ? r : b - 1) * s];
#pragma unroll
    for (int r = 0; r < BMAX; ++r) acc[r] = fmaf(xv[r], gv, acc[r]);   // r >= b: never stored
  }
#pragma unroll
  for (int r = 0; r < BMAX; ++r)
    if (r < b) partial[((size_t)blockIdx.y * (b * b) + r * b + r2) * D + c] = acc[r];
}

// Radix 49 .. 64: the same sums on the matrix cores: dK[c] = sum over rows of x[idx]^T g[idx] is a b x rows x b
// product per block (v_mfma_f32_16x16x4_f32, unsplit float32 operands: the k index is the row).
// Needs 16 consecutive blocks to be 16 consecutive coordinates (s a multiple of 16).  A workgroup
// of 16 waves owns 16 consecutive blocks and one row chunk and walks down its rows 8 at a time:
// coalesced 16-byte loads of x and g (next step prefetched in registers) -> two LDS tiles
// [r][block][row] -> wave w multiplies the tiles of its block, KT x KT accumulator tiles in
// registers for the whole chunk.  At the end the accumulators pass through LDS tile by tile
// so that the partial sums leave in runs of 16 consecutive blocks (64 bytes).  Rows past the end
// of the chunk enter as zeros.  Workgroups that share 128-byte lines (two neighbouring block
// tiles) are numbered onto one XCD.
constexpr int kDkRows = 8;                  // rows per step (16 measured 1 % faster at 2048 x 11008 for twice the LDS)
constexpr int kDkLS = kDkRows + 1;          // LDS stride between consecutive blocks
constexpr int kDkJS = 16 * kDkLS + 4;       // LDS stride between consecutive r

__global__ __launch_bounds__(1024) void harp_grad_dk_mfma_kernel(
    const float *__restrict__ X, int64_t ldx, const float *__restrict__ Gm, int64_t ldg, int64_t n, int rows,
    int D, int s, int b, int gx, int paired, float *__restrict__ partial) {
  typedef float f4v __attribute__((ext_vector_type(4)));
  constexpr int KT = 4;   // operand tiles of 16: radix 49 .. 64
  constexpr int MAXG = (kDkRows * 16 * KT * 4 + 1023) / 1024;
  constexpr int TILE = 16 * KT * kDkJS;
  __shared__ float lds[2 * TILE];
  float *tx = lds, *tg = lds + TILE;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63, g = l >> 4, c16 = l & 15;
  unsigned wg = blockIdx.x;
  if (paired) {
    const unsigned xcd = wg & 7u, k = wg >> 3;
    wg = ((k >> 1) * 8u + xcd) * 2u + (k & 1u);
  }
  const int qx = (int)(wg % (unsigned)gx), chunk = (int)(wg / (unsigned)gx);
  const int q0 = qx * 16;
  const int64_t base = (int64_t)(q0 / s) * b * s + q0 % s;
  const int64_t r_begin = (int64_t)chunk * rows;
  const int64_t r_end = (r_begin + rows < n) ? r_begin + rows : n;

  const int ngroups = kDkRows * b * 4;   // (row, r, quarter of the 16 blocks) per step
  unsigned off[MAXG], offg[MAXG];
  int grow[MAXG], slot[MAXG];
#pragma unroll
  for (int u = 0; u < MAXG; ++u) {
    const int gi = (tid + u * 1024) % ngroups;
    const int lo4 = gi & 3, rem = gi >> 2;
    const int row = rem & (kDkRows - 1), j = rem / kDkRows;
    grow[u] = row;
    off[u] = (unsigned)(row * (int)ldx + j * s + lo4 * 4);
    offg[u] = (unsigned)(row * (int)ldg + j * s + lo4 * 4);
    slot[u] = j * kDkJS + (lo4 * 4) * kDkLS + row;
  }
  float4 px[MAXG], pg[MAXG];
  auto fetch = [&](int64_t r0, int left) {
    const float *xc = X + r0 * ldx + base, *gc = Gm + r0 * ldg + base;
    if (left >= kDkRows) {
#pragma unroll
      for (int u = 0; u < MAXG; ++u) {
        px[u] = *reinterpret_cast<const float4 *>(xc + off[u]);
        pg[u] = *reinterpret_cast<const float4 *>(gc + offg[u]);
      }
    } else {
#pragma unroll
      for (int u = 0; u < MAXG; ++u) {
        px[u] = pg[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (grow[u] < left) {
          px[u] = *reinterpret_cast<const float4 *>(xc + off[u]);
          pg[u] = *reinterpret_cast<const float4 *>(gc + offg[u]);
        }
      }
    }
  };
  auto commit = [&]() {
#pragma unroll
    for (int u = 0; u < MAXG; ++u) {
      float *a = tx + slot[u], *c = tg + slot[u];
      a[0] = px[u].x; a[kDkLS] = px[u].y; a[2 * kDkLS] = px[u].z; a[3 * kDkLS] = px[u].w;
      c[0] = pg[u].x; c[kDkLS] = pg[u].y; c[2 * kDkLS] = pg[u].z; c[3 * kDkLS] = pg[u].w;
    }
  };
  f4v acc[KT][KT];
#pragma unroll
  for (int mt = 0; mt < KT; ++mt)
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) acc[mt][nt] = (f4v){0.f, 0.f, 0.f, 0.f};

  if (r_begin < r_end) {
    fetch(r_begin, (int)(r_end - r_begin));
    for (int64_t r0 = r_begin; r0 < r_end; r0 += kDkRows) {
      commit();
      __syncthreads();
      const int64_t rn = r0 + kDkRows;
      if (rn < r_end) fetch(rn, (int)(r_end - rn));
#pragma unroll
      for (int ks = 0; ks < kDkRows / 4; ++ks) {
        float a[KT], bv[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) {
          const int j = 16 * t + c16;
          const int at = (j < b ? j : 0) * kDkJS + w * kDkLS + 4 * ks + g;
          a[t] = (j < b) ? tx[at] : 0.f;
          bv[t] = (j < b) ? tg[at] : 0.f;
        }
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
          for (int nt = 0; nt < KT; ++nt)
            acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mt], bv[nt], acc[mt][nt], 0, 0, 0);
      }
      __syncthreads();   // every wave has read its operands: the tiles are free again
    }
  }
  // accumulator tile (mt, nt) of all 16 blocks -> LDS [m][n][block] -> 64-byte runs
  float *so = lds;
  const int e = tid >> 2, quarter = tid & 3;
  const int em = e >> 4, en = e & 15;
#pragma unroll
  for (int mt = 0; mt < KT; ++mt)
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
#pragma unroll
      for (int i = 0; i < 4; ++i) so[((4 * g + i) * 16 + c16) * 16 + w] = acc[mt][nt][i];
      __syncthreads();
      const int r = 16 * mt + em, r2 = 16 * nt + en;
      if (r < b && r2 < b) {
        const float4 v = *reinterpret_cast<const float4 *>(so + e * 16 + 4 * quarter);
        *reinterpret_cast<float4 *>(partial + ((size_t)chunk * (b * b) + r * b + r2) * D + q0 + 4 * quarter) = v;
      }
      __syncthreads();
    }
}

static void launch_dk_mfma(const float *X, int64_t ldx, const float *Gm, int64_t ldg, int64_t n, int rows, int nchunks,
                           int D, int s, int b, float *partial, hipStream_t st) {
  const int gx = D / 16;
  const int64_t total = (int64_t)gx * nchunks;
  const int paired = (gx % 2 == 0) && (total % 16 == 0);
  hipLaunchKernelGGL(harp_grad_dk_mfma_kernel, dim3((unsigned)total), dim3(1024), 0, st, X, ldx, Gm, ldg, n,
                     rows, D, s, b, gx, paired, partial);
}

static bool dk_mfma_supported(int b, int s, int D, const void *X, int64_t ldx, const void *Gm, int64_t ldg,
                              const void *partial, int64_t nchunks) {
  if (b < 49 || b > 64 || s % 16 != 0 || D % 16 != 0) return false;
  if (ldx % 4 || ldg % 4 || ldx >= ((int64_t)1 << 26) || ldg >= ((int64_t)1 << 26)) return false;
  if ((uintptr_t)X % 16 || (uintptr_t)Gm % 16 || (uintptr_t)partial % 16) return false;
  return (int64_t)(D / 16) * nchunks <= 0x7fffffff;
}

// the instantiation whose BMAX covers radix b
#define HARP_GRAD_BIG(b, CALL)            \
  do {                                    \
    if ((b) <= 16) { CALL(16); }          \
    else if ((b) <= 32) { CALL(32); }     \
    else if ((b) <= 48) { CALL(48); }     \
    else { CALL(64); }                    \
  } while (0)

// Run of K radix-2 stages with strides s, 2s, .., 2^(K-1) s.  Item q = hi s + lo owns the
// coordinates base + e s, e < 2^K, base = hi 2^K s + lo.  Stage i pairs e0 (bit i clear) with e0 + 2^i.
// Pair p (e0 with bit i taken out) is block hi 2^(K-1) s + lo + p s of its stage, whatever the stage.
struct GradRun {
  const float *blocks[3];
};

// c0: the item's block of pair 0
template <int K>
__device__ __forceinline__ void grad_run_blocks(const GradRun &run, int c0, int s, float (&kv)[K][1 << (K - 1)][4]) {
#pragma unroll
  for (int i = 0; i < K; ++i)
#pragma unroll
    for (int p = 0; p < (1 << (K - 1)); ++p) {
      const float4 f = *reinterpret_cast<const float4 *>(run.blocks[i] + (size_t)(c0 + p * s) * 4);
      kv[i][p][0] = f.x; kv[i][p][1] = f.y; kv[i][p][2] = f.z; kv[i][p][3] = f.w;
    }
}

// The E coordinates x[e s] of an item, float32 or bf16 (the caller's own rows in the first and
// last run, so that no separate conversion pass is needed); vec: stride 1 and aligned rows, the
// item is contiguous and moves with 16-byte accesses.
template <int E, typename T>
__device__ __forceinline__ void grad_load_item(const T *row, int base, int s, bool vec, float (&v)[E]) {
  if (vec) {
    const T *x = grad_at(row, base);
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int q = 0; q < E / 4; ++q) {
        const float4 f = *reinterpret_cast<const float4 *>(x + 4 * q);
        v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
      }
    } else if constexpr (E == 8) {
      const uint4 r = *reinterpret_cast<const uint4 *>(x);
      const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
      }
    } else {
      const uint2 r = *reinterpret_cast<const uint2 *>(x);
      v[0] = __uint_as_float(r.x << 16); v[1] = __uint_as_float(r.x & 0xffff0000u);
      v[2] = __uint_as_float(r.y << 16); v[3] = __uint_as_float(r.y & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = grad_widen(*grad_at(row, base + e * s));
  }
}
template <int E, typename T>
__device__ __forceinline__ void grad_store_item(T *row, int base, int s, bool vec, const float (&v)[E]) {
  if (vec) {
    T *y = grad_at(row, base);
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int q = 0; q < E / 4; ++q)
        *reinterpret_cast<float4 *>(y + 4 * q) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    } else {
      uint16_t h[E];
#pragma unroll
      for (int e = 0; e < E; ++e) grad_narrow(v[e], &h[e]);
      if constexpr (E == 8)
        *reinterpret_cast<uint4 *>(y) = make_uint4(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16),
                                                    h[4] | ((uint32_t)h[5] << 16), h[6] | ((uint32_t)h[7] << 16));
      else
        *reinterpret_cast<uint2 *>(y) = make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) grad_narrow(v[e], grad_at(row, base + e * s));
  }
}

// TX: element type of the run's input rows (leading dimension ldx)
template <int K, typename TX = float>
__global__ __launch_bounds__(kGradThreads) void harp_grad_fwd_run_kernel(
    const TX *__restrict__ X, int64_t ldx, float *__restrict__ Y, int64_t ld, int64_t n, int rows,
    GradRun run, int nitems, int s, int aligned) {
  constexpr int E = 1 << K, H = E / 2;
  const int q = blockIdx.x * kGradThreads + threadIdx.x;
  if (q >= nitems) return;
  const int base = (q / s) * E * s + q % s;
  float kv[K][H][4];
  grad_run_blocks<K>(run, (q / s) * H * s + q % s, s, kv);
  const int64_t r0 = (int64_t)blockIdx.y * rows;
  const int64_t r1 = (r0 + rows < n) ? r0 + rows : n;
  // the next row is requested before the work on the current one
  // stride 1: the item's coordinates are contiguous (16-byte accesses when the row allows it)
  const bool vec = aligned && (s == 1) && (E % 4 == 0) && (ld % 4 == 0);
  const bool vecx = vec && ldx % (16 / (int)sizeof(TX)) == 0 && (uintptr_t)X % 16 == 0;
  auto load_item = [&](const TX *row_, float (&v)[E]) { grad_load_item<E, TX>(row_, base, s, vecx, v); };
  float nx[E];
#pragma unroll
  for (int e = 0; e < E; ++e) nx[e] = 0.f;
  if (r0 < r1) load_item(X + r0 * ldx, nx);
  for (int64_t row = r0; row < r1; ++row) {
    float *y = Y + row * ld + base;
    float v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = nx[e];
    if (row + 1 < r1) load_item(X + (row + 1) * ldx, nx);
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
      for (int p = 0; p < H; ++p) {
        const int eh = p >> i, el = p & ((1 << i) - 1);
        const int e0 = (eh << (i + 1)) | el, e1 = e0 | (1 << i);
        const float a = v[e0], b = v[e1];
        v[e0] = fmaf(b, kv[i][p][2], a * kv[i][p][0]);
        v[e1] = fmaf(b, kv[i][p][3], a * kv[i][p][1]);
      }
    if (vec) {
#pragma unroll
      for (int q = 0; q < E / 4; ++q)
        *reinterpret_cast<float4 *>(y + 4 * q) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) y[(size_t)e * s] = v[e];
    }
  }
}

// partial sums of sub-stage i go to partial[i * pstride + (chunk * 4 + v) * D + c], D = d / 2
// TX: element type of the run's input rows X; the gradient is read from Gin (TGI) and the
// gradient passed back is written to Gout (TGO): the same float32 matrix in place, or the
// caller's G on the way in (last run) and the caller's dX on the way out (first run).  A thread
// reads its item of a row (X and gradient) before it writes it, and no other thread touches that item:
// dX may be X or G.
template <int K, typename TX = float, typename TGI = float, typename TGO = float>
__global__ __launch_bounds__(kSumThreads) void harp_grad_bwd_run_kernel(
    const TX *X, int64_t ldx, const TGI *Gin, int64_t ldgi, TGO *Gout, int64_t ldgo,
    int64_t ld, int64_t n, int rows, GradRun run, int nitems, int s, int D,
    float *__restrict__ partial, size_t pstride, int aligned) {
  constexpr int E = 1 << K, H = E / 2;
  const SumRows sr = sum_rows(n, rows);
  const int q0 = blockIdx.x * kSumItems + sr.item, q = q0 < nitems ? q0 : nitems - 1;
  const int base = (q / s) * E * s + q % s;
  float kv[K][H][4], acc[K * H * 4];
  const int c0 = (q / s) * H * s + q % s;
  grad_run_blocks<K>(run, c0, s, kv);
#pragma unroll
  for (int v = 0; v < K * H * 4; ++v) acc[v] = 0.f;
  const int64_t r0 = sr.r0, r1 = q0 < nitems ? sr.r1 : sr.r0;   // threads past the last item have no rows
  const bool vec = aligned && (s == 1) && (E % 4 == 0) && (ld % 4 == 0);
  const bool vecx = vec && ldx % (16 / (int)sizeof(TX)) == 0 && (uintptr_t)X % 16 == 0;
  const bool vecgi = vec && ldgi % (16 / (int)sizeof(TGI)) == 0 && (uintptr_t)Gin % 16 == 0;
  const bool vecgo = vec && ldgo % (16 / (int)sizeof(TGO)) == 0 && (uintptr_t)Gout % 16 == 0;
  float nx[E], ng[E];
#pragma unroll
  for (int e = 0; e < E; ++e) nx[e] = ng[e] = 0.f;
  if (r0 < r1) {
    grad_load_item<E, TX>(X + r0 * ldx, base, s, vecx, nx);
    grad_load_item<E, TGI>(Gin + r0 * ldgi, base, s, vecgi, ng);
  }
  for (int64_t row = r0; row < r1; ++row) {
    float xs[K][E], gv[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      xs[0][e] = nx[e];
      gv[e] = ng[e];
    }
    if (row + 1 < r1) {   // the next row (its g is not written by anyone before this thread does)
      grad_load_item<E, TX>(X + (row + 1) * ldx, base, s, vecx, nx);
      grad_load_item<E, TGI>(Gin + (row + 1) * ldgi, base, s, vecgi, ng);
    }
    // inputs of the inner stages, recomputed
#pragma unroll
    for (int i = 0; i + 1 < K; ++i) {
#pragma unroll
      for (int p = 0; p < H; ++p) {
        const int eh = p >> i, el = p & ((1 << i) - 1);
        const int e0 = (eh << (i + 1)) | el, e1 = e0 | (1 << i);
        const float a = xs[i][e0], b = xs[i][e1];
        xs[i + 1][e0] = fmaf(b, kv[i][p][2], a * kv[i][p][0]);
        xs[i + 1][e1] = fmaf(b, kv[i][p][3], a * kv[i][p][1]);
      }
    }
#pragma unroll
    for (int i = K - 1; i >= 0; --i) {
#pragma unroll
      for (int p = 0; p < H; ++p) {
        const int eh = p >> i, el = p & ((1 << i) - 1);
        const int e0 = (eh << (i + 1)) | el, e1 = e0 | (1 << i);
        const float x0 = xs[i][e0], x1 = xs[i][e1], g0 = gv[e0], g1 = gv[e1];
        acc[(i * H + p) * 4 + 0] = fmaf(x0, g0, acc[(i * H + p) * 4 + 0]);
        acc[(i * H + p) * 4 + 1] = fmaf(x0, g1, acc[(i * H + p) * 4 + 1]);
        acc[(i * H + p) * 4 + 2] = fmaf(x1, g0, acc[(i * H + p) * 4 + 2]);
        acc[(i * H + p) * 4 + 3] = fmaf(x1, g1, acc[(i * H + p) * 4 + 3]);
        gv[e0] = fmaf(g1, kv[i][p][1], g0 * kv[i][p][0]);   // g K^T, row 0: k00 g0 + k01 g1
        gv[e1] = fmaf(g1, kv[i][p][3], g0 * kv[i][p][2]);
      }
    }
    grad_store_item<E, TGO>(Gout + row * ldgo, base, s, vecgo, gv);
  }
  __shared__ float red[2 * K * H * 4 * kSumItems];
  sum_groups<K * H * 4>(acc, sr, red);
  if (sr.group != 0 || q0 >= nitems) return;
#pragma unroll
  for (int i = 0; i < K; ++i)
#pragma unroll
    for (int p = 0; p < H; ++p)
#pragma unroll
      for (int w = 0; w < 4; ++w)
        partial[(size_t)i * pstride + ((size_t)blockIdx.y * 4 + w) * D + c0 + p * s] = acc[(i * H + p) * 4 + w];
}

// dK[c][v] = sum over the chunks of partial[(chunk * BB + v) * D + c], in a fixed order: eight
// threads per value each add a contiguous eighth of the chunks (ascending), then the eight
// sums are added in ascending order.  For stage 0 the image holds diag(sigma) K_0, so row r of
// its gradient takes the sign of coordinate c b + r.
// blockIdx.y = sub-stage of a run (its partial sums start pstride floats further on).
struct GradReduceOut {
  float *dK[3];
  const int8_t *signs[3];
};
__global__ __launch_bounds__(kGradThreads) void harp_grad_reduce_kernel(
    const float *__restrict__ partial_all, size_t pstride, int nchunks, int D, int b,
    GradReduceOut out) {
  __shared__ float part[8][32];
  const float *__restrict__ partial = partial_all + (size_t)blockIdx.y * pstride;
  const int8_t *__restrict__ signs = out.signs[blockIdx.y];
  float *__restrict__ dK = out.dK[blockIdx.y];
  const int bb = b * b;
  const int64_t total = (int64_t)D * bb;
  const int lane = threadIdx.x & 31, slice = threadIdx.x >> 5;
  const int per = (nchunks + 7) / 8;
  const int k0 = slice * per, k1 = (k0 + per < nchunks) ? k0 + per : nchunks;
  const size_t step = (size_t)bb * D;
  for (int64_t i0 = (int64_t)blockIdx.x * 32; i0 < total; i0 += (int64_t)gridDim.x * 32) {
    const int64_t i = i0 + lane;
    const int v = (int)(i / D), c = (int)(i % D);     // consecutive lanes: consecutive c
    float sum = 0.f;
    if (i < total) {
      const float *p = partial + (size_t)v * D + c;
      int k = k0;
      for (; k + 8 <= k1; k += 8) {
        float t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = p[(size_t)(k + u) * step];
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += t[u];
      }
      for (; k < k1; ++k) sum += p[(size_t)k * step];
    }
    part[slice][lane] = sum;
    __syncthreads();
    if (slice == 0 && i < total) {
      float tot = part[0][lane];
#pragma unroll
      for (int u = 1; u < 8; ++u) tot += part[u][lane];
      if (signs) tot *= (float)signs[(size_t)c * b + v / b];
      dK[(size_t)c * bb + v] = tot;
    }
    __syncthreads();
  }
}

template <int B>
void launch_fwd(const float *X, float *Y, int64_t ld, int64_t n, int rows, int nchunks,
                const float *blocks, int D, int s, hipStream_t st) {
  hipLaunchKernelGGL((harp_grad_fwd_kernel<B>), dim3((D + kGradThreads - 1) / kGradThreads, nchunks),
                     dim3(kGradThreads), 0, st, X, Y, ld, n, rows, blocks, D, s);
}
template <int B>
void launch_bwd(const float *X, float *G, int64_t ld, int64_t n, int rows, int nchunks,
                const float *blocks, int D, int s, float *partial, hipStream_t st) {
  hipLaunchKernelGGL((harp_grad_bwd_kernel<B>), dim3((D + kSumItems - 1) / kSumItems, nchunks),
                     dim3(kSumThreads), 0, st, X, G, ld, n, rows, blocks, D, s, partial);
}

#define HARP_GRAD_SWITCH(b, CALL)  \
  switch (b) {                     \
    case 2: CALL(2); break;        \
    case 3: CALL(3); break;        \
    case 4: CALL(4); break;        \
    case 5: CALL(5); break;        \
    case 6: CALL(6); break;        \
    case 7: CALL(7); break;        \
    default: CALL(8); break;       \
  }

template <typename TS, typename TD>
void launch_convert(const TS *src, int64_t lds_, TD *dst, int64_t ldd, int64_t n, int64_t d,
                    hipStream_t st) {
  const bool vec = (d % 8 == 0) && (lds_ % 8 == 0) && (ldd % 8 == 0) && ((uintptr_t)src % 16 == 0) &&
                   ((uintptr_t)dst % 16 == 0);
  const int64_t per = vec ? 8 * kGradThreads : kGradThreads;
  // the row index is blockIdx.y (at most 65535 per launch)
  for (int64_t r0 = 0; r0 < n; r0 += 65535) {
    const int64_t nr = std::min<int64_t>(65535, n - r0);
    const unsigned gx = (unsigned)std::min<int64_t>((d + per - 1) / per, 64);
    if (vec)
      hipLaunchKernelGGL((harp_grad_convert_kernel<TS, TD, true>), dim3(gx, (unsigned)nr),
                         dim3(kGradThreads), 0, st, src + r0 * lds_, lds_, dst + r0 * ldd, ldd, nr, (int)d);
    else
      hipLaunchKernelGGL((harp_grad_convert_kernel<TS, TD, false>), dim3(gx, (unsigned)nr),
                         dim3(kGradThreads), 0, st, src + r0 * lds_, lds_, dst + r0 * ldd, ldd, nr, (int)d);
  }
}

}  // namespace

// Row chunks per launch: a fused run of three stages has only d / 8 threads per row, so the
// rows have to supply the parallelism (d = 4096: 2 workgroups x 256 chunks).
int grad_chunks(int64_t n) {
  const int64_t c = (n + 7) / 8;
  return (int)std::max<int64_t>(1, std::min<int64_t>(c, 256));
}

// Row chunks of the backward kernel of a stage (or run) with `items` blocks (or items) per row.  A workgroup
// of four groups takes 4, 8 or 16 rows as long as the launch then has no more than 64, 128 or 256 workgroups,
// else 32 (more beyond 8192 rows).  The rows of a group follow one another, so few rows want many
// workgroups, while each workgroup costs its block values and a set of partial sums, which the reduction
// reads again.  4096 radix 8 (four workgroups wide), kernel + reduction, us, at 4 / 8 / 16 / 32 rows each:
// 128 rows 12.2 / 11.4 / 11.6 / 14.8, 256 rows 15.2 / 13.6 / 13.3 / 16.3, 1024 rows 34 / 22.5 / 17.6 / 17.6,
// 2048 rows 38 / 38 / 27.7 / 24.1.  Whole calls against 32 rows each throughout, us: 60 rows 132 -> 79,
// 256 rows 149 -> 104 (radix 8, generic blocks), 512 rows 94 -> 77 (radix 2).
int grad_sum_chunks(int64_t n, int64_t items) {
  const int64_t wide = (items + kSumItems - 1) / kSumItems;
  for (int64_t rows = kSumGroups; rows <= 4 * kSumGroups; rows *= 2)
    if ((n + rows - 1) / rows * wide <= 16 * rows) return (int)std::max<int64_t>(1, (n + rows - 1) / rows);
  return (int)std::min<int64_t>((n + 8 * kSumGroups - 1) / (8 * kSumGroups), 256);
}
// At least grad_sum_chunks(n, items), and never less for more rows.
static int64_t grad_sum_chunks_bound(int64_t n, int64_t items) {
  const int64_t wide = (items + kSumItems - 1) / kSumItems;
  const int64_t few = std::min<int64_t>((n + kSumGroups - 1) / kSumGroups, std::max<int64_t>(16 * 4 * kSumGroups / wide, 1));
  return std::max<int64_t>(1, std::max(few, std::min<int64_t>((n + 8 * kSumGroups - 1) / (8 * kSumGroups), 256)));
}

// Segments of the backward pass: the first `lead` stages as one segment of 64 coordinates and pairs of
// passes behind it (harp_grad_pair.hip), then runs of up to three radix-2 stages, single stages otherwise.
struct GradSegment {
  int t0, k;
  bool pair;
};
static std::vector<GradSegment> grad_segments(const std::vector<int32_t> &radices, int lead) {
  std::vector<GradSegment> seg;
  const int m = (int)radices.size();
  if (lead > 0) seg.push_back(GradSegment{0, lead, false});
  int t = lead;
  while (t < m) {
    int k = lead > 0 ? grad_pair_stages(radices, t) : 0;
    const bool pair = k > 0;
    if (!pair) {
      k = 1;
      if (radices[t] == 2)
        while (k < 3 && t + k < m && radices[t + k] == 2) ++k;
    }
    seg.push_back(GradSegment{t, k, pair});
    t += k;
  }
  return seg;
}
static std::vector<GradSegment> grad_segments(const harp_plan *plan, int lead) { return grad_segments(plan->radices, lead); }

extern "C" int32_t harp_internal_grad_sides(int32_t m, const int32_t *radices, int32_t *room) {
  const std::vector<int32_t> r(radices, radices + m);
  const int lead = grad_seg_stages(r);
  int sides = lead > 0 ? 2 : 0;
  if (lead > 0)
    for (const GradSegment &sg : grad_segments(r, lead)) sides += sg.pair ? 2 : 0;
  *room = kGradMostSides;
  return sides;
}

// Stages of radix above 8 take longer row chunks: blockIdx.z already supplies parallelism, and a
// chunk costs one read of the block column per thread and b * b partial sums per block.
static int grad_big_rows(int64_t n) {
  const int nchunks = grad_chunks(n);
  return std::max((int)((n + nchunks - 1) / nchunks), 64);
}
static int grad_big_chunks(int64_t n) {
  const int rb = grad_big_rows(n);
  return (int)std::max<int64_t>(1, (n + rb - 1) / rb);
}
// At least grad_big_chunks(n), and never less for more rows (longer chunks can mean fewer of them).
static int64_t grad_big_chunks_bound(int64_t n) {
  return std::max<int64_t>(1, std::min<int64_t>((n + 63) / 64, 256));
}

// Does not fall as n grows: a workspace for n rows serves every smaller batch (every count of chunks
// in it is one that never falls, and the plan without the leading segment keeps one matrix more, so
// neither end of that segment's range of n is a step down).
static size_t grad_partial_floats(const harp_plan *plan, int64_t n) {   // the most partial sums of one launch of this file
  size_t per_row = 0;   // times 1 / d: chunks * b of a stage, chunks * 2 k of a run
  for (int32_t b : plan->radices) {
    if (b > 8) per_row = std::max(per_row, (size_t)grad_big_chunks_bound(n) * b);
    else per_row = std::max(per_row, (size_t)grad_sum_chunks_bound(n, plan->d / b) * b);
  }
  // (the segments behind the leading one are among these, or shorter runs with fewer chunks)
  for (const GradSegment &sg : grad_segments(plan, 0))
    if (sg.k > 1) per_row = std::max(per_row, (size_t)grad_sum_chunks_bound(n, plan->d >> sg.k) * 2 * sg.k);
  size_t most = per_row * (size_t)plan->d;
  for (int t = 0; t < plan->m; ++t)
    if (grad_big_stage(plan, t)) most = std::max(most, grad_big_partial_floats(plan, t, n));
  return (most + 3) / 4 * 4;
}
size_t grad_workspace_bytes(const harp_plan *plan, int64_t n) {
  int bbig = 0;
  for (int32_t b : plan->radices) bbig = std::max(bbig, (int)b);
  if (bbig <= 8) bbig = 0;
  const int lead = grad_seg_stages(plan, n);
  const size_t mat = (size_t)n * (size_t)plan->d * 4;
  const size_t partial = grad_partial_floats(plan, n) * 4;
  // a stage of radix above 8 passes the gradient back out of place: one more matrix
  const size_t extra = 1 + (bbig > 0 ? 1 : 0);
  size_t need = (grad_segments(plan, 0).size() + extra) * mat + partial;
  if (lead > 0) {
    size_t sums = partial + grad_lead_partial_bytes(plan, n);
    const std::vector<GradSegment> seg = grad_segments(plan, lead);
    for (const GradSegment &sg : seg)
      if (sg.pair) sums += grad_pair_partial_bytes(plan, sg.t0, n);
    need = std::max(need, (seg.size() + extra) * mat + sums);
  }
  return need + 16;   // launch_grad starts at the next multiple of 16 bytes
}

harp_status_t launch_grad(const harp_plan *plan, const void *X, int64_t ldx, const void *G,
                          int64_t ldg, int64_t n, harp_dtype_t dt, float *const *dK, void *dX,
                          int64_t lddx, void *ws, hipStream_t st) {
  const std::vector<ColStage> &stages = plan->col[DIR_FWD];
  // The path follows from the plan and n alone, never from where the matrices lie: kernels sum in
  // different orders, and the same numbers are to give the same bits.
  ws = (void *)(((uintptr_t)ws + 15) & ~(uintptr_t)15);
  const int lead = grad_seg_stages(plan, n);
  const std::vector<GradSegment> seg = grad_segments(plan, lead);
  const int nseg = (int)seg.size();
  const int64_t d = plan->d;
  const int nchunks = grad_chunks(n);
  const int rows = (int)((n + nchunks - 1) / nchunks);
  const int rows_big = grad_big_rows(n);
  const int nchunks_big = grad_big_chunks(n);
  const size_t mat = (size_t)n * (size_t)d;
  int bmax = 0;
  for (int32_t b : plan->radices) bmax = std::max(bmax, (int)b);
  float *act = (float *)ws;                 // act[i] = input of segment i
  float *g = act + (size_t)nseg * mat;      // gradient, updated in place (radix <= 8) ...
  float *g2 = g + mat;                      // ... or into the other of two matrices (radix >= 9)
  float *partial = g + (bmax > 8 ? 2 : 1) * mat;
  float *sums_at = partial + grad_partial_floats(plan, n);   // of harp_grad_pair.hip, all until the end of the call
  GradSums sums{};
  // 16-byte accesses of the stride-1 runs need the float32 copies on 16-byte boundaries
  const int aligned = (mat % 4 == 0);
  auto run_of = [&](const GradSegment &sg) {
    GradRun run;
    for (int i = 0; i < 3; ++i) run.blocks[i] = stages[sg.t0 + std::min(i, sg.k - 1)].blocks;
    return run;
  };
  // A run of radix-2 stages at the start reads the caller's X itself (forward and backward), one
  // at the end reads the caller's G, and the first run writes dX: no separate conversion pass.
  const bool bf = (dt == HARP_BF16);
  const bool first_run = seg[0].k > 1;
  const GradSegment &behind = seg[nseg - 1];
  const bool last_run = behind.k > 1 && (!behind.pair || grad_pair_reads(plan, behind.t0, ldg, bf));
  const bool dx_direct = first_run && dX != nullptr;
  // A stage of radix above 8 at the end passes the gradient back out of place, so its matrix-core kernels read the caller's G
  // where it lies (1537 x 11008 float32, last radix 43: 348 -> 311 us for the whole call; 2048 x 11008 bf16 in one launch:
  // a conversion of 26 us less), radix 49 and up float32 rows only.  Their plain fallbacks take one leading dimension and
  // keep the copy.
  const int tlast = seg[nseg - 1].t0;
  const ColStage &last = stages[tlast];
  const bool g_direct =
      last.b > 8 && (uintptr_t)G % (bf ? 8 : 16) == 0 && ldg % 4 == 0 && ldg < ((int64_t)1 << 25) &&
      (grad_big_stage(plan, tlast) ||
       (!bf && mfma_pass_supported(plan->grad_mfma[1][tlast], G, ldg, g2, d) &&
        dk_mfma_supported(last.b, last.s, (int)(d / last.b), act + (size_t)(nseg - 1) * mat, d, G, ldg, partial,
                          nchunks_big)));
  if (n > 0) {
    if (!first_run) {
      if (bf) launch_convert((const uint16_t *)X, ldx, act, d, n, d, st);
      else launch_convert((const float *)X, ldx, act, d, n, d, st);
    }
    if (!last_run && !g_direct) {
      if (bf) launch_convert((const uint16_t *)G, ldg, g, d, n, d, st);
      else launch_convert((const float *)G, ldg, g, d, n, d, st);
    }
    for (int i = 0; i + 1 < nseg; ++i) {
      const ColStage &cs = stages[seg[i].t0];
      const float *in = act + (size_t)i * mat;
      float *out = act + (size_t)(i + 1) * mat;
      if (i == 0 && lead > 0) {
        const harp_status_t rc = launch_grad_seg_fwd(plan, lead, X, ldx, bf, out, n, st);
        if (rc != HARP_OK) return rc;
      } else if (seg[i].pair) {
        const harp_status_t rc = launch_grad_pair_fwd(plan, seg[i].t0, in, out, n, st);
        if (rc != HARP_OK) return rc;
      } else if (seg[i].k > 1) {
        const int nitems = (int)(d >> seg[i].k);
        const dim3 grid((nitems + kGradThreads - 1) / kGradThreads, nchunks);
#define HARP_GRAD_FWD_RUN(KK)                                                                       \
  do {                                                                                              \
    if (i == 0 && bf)                                                                               \
      hipLaunchKernelGGL((harp_grad_fwd_run_kernel<KK, uint16_t>), grid, dim3(kGradThreads), 0, st, \
                         (const uint16_t *)X, ldx, out, d, n, rows, run_of(seg[i]), nitems, cs.s,   \
                         aligned);                                                                  \
    else if (i == 0)                                                                                \
      hipLaunchKernelGGL((harp_grad_fwd_run_kernel<KK, float>), grid, dim3(kGradThreads), 0, st,    \
                         (const float *)X, ldx, out, d, n, rows, run_of(seg[i]), nitems, cs.s,      \
                         aligned);                                                                  \
    else                                                                                            \
      hipLaunchKernelGGL((harp_grad_fwd_run_kernel<KK, float>), grid, dim3(kGradThreads), 0, st,    \
                         in, d, out, d, n, rows, run_of(seg[i]), nitems, cs.s, aligned);            \
  } while (0)
        if (seg[i].k == 3) HARP_GRAD_FWD_RUN(3);
        else HARP_GRAD_FWD_RUN(2);
#undef HARP_GRAD_FWD_RUN
      } else if (cs.b > 8 && mfma_pass_supported(plan->grad_mfma[0][seg[i].t0], in, d, out, d)) {
        // the stage on the matrix cores (float32 operands), as in a split program
        if (launch_mfma_pass(plan, plan->grad_mfma[0][seg[i].t0], in, d, HARP_F32, out, d, HARP_F32, n,
                             false, st) != HARP_OK)
          return HARP_ERR_DEVICE;
      } else if (cs.b > 8) {
        const int D = (int)(d / cs.b);
#define HARP_GRAD_BIG_FWD(BM)                                                                     \
  hipLaunchKernelGGL((harp_grad_apply_big_kernel<BM, false>),                                     \
                     dim3((D + 63) / 64, nchunks_big, (cs.b + 3) / 4), dim3(kGradThreads), 0, st, \
                     in, out, d, n, rows_big, cs.blocks, D, cs.s, cs.b)
        HARP_GRAD_BIG(cs.b, HARP_GRAD_BIG_FWD);
#undef HARP_GRAD_BIG_FWD
      } else {
        const int D = (int)(d / cs.b);
#define HARP_GRAD_FWD(BB) launch_fwd<BB>(in, out, d, n, rows, nchunks, cs.blocks, D, cs.s, st)
        HARP_GRAD_SWITCH(cs.b, HARP_GRAD_FWD)
#undef HARP_GRAD_FWD
      }
    }
  }
  for (int i = nseg - 1; i >= 0; --i) {
    const ColStage &cs = stages[seg[i].t0];
    const float *in = act + (size_t)i * mat;
    const int nsum = grad_sum_chunks(n, seg[i].k > 1 ? d >> seg[i].k : d / cs.b);
    const int rows_sum = (int)((n + nsum - 1) / nsum);
    const size_t pstride = (size_t)nsum * 4 * (size_t)(d / 2);   // one radix-2 stage's partials
    if (i == 0 && lead > 0) {
      const harp_status_t rc = launch_grad_lead_bwd(plan, lead, X, ldx, bf, g, dX, lddx, n, sums_at, dK, sums, st);
      if (rc != HARP_OK) return rc;
      break;
    }
    if (seg[i].pair) {
      const bool own = last_run && i == nseg - 1;   // reads the caller's G
      const harp_status_t rc = launch_grad_pair_bwd(plan, seg[i].t0, in, own ? G : (const void *)g, own ? ldg : d,
                                                    own && bf, g, n, sums_at, dK, sums, st);
      if (rc != HARP_OK) return rc;
      sums_at += grad_pair_partial_bytes(plan, seg[i].t0, n) / 4;
      continue;
    }
    if (n > 0) {
      if (seg[i].k > 1) {
        const int nitems = (int)(d >> seg[i].k);
        const dim3 grid((nitems + kSumItems - 1) / kSumItems, nsum);
        // what this run reads and writes: the caller's rows at either end, float32 copies between
        const bool xc = (i == 0), gic = (i == nseg - 1), goc = (i == 0) && dx_direct;
#define HARP_GRAD_BWD_RUN(KK, TX_, TGI_, TGO_)                                                       \
  hipLaunchKernelGGL((harp_grad_bwd_run_kernel<KK, TX_, TGI_, TGO_>), grid, dim3(kSumThreads), 0,    \
                     st, xc ? (const TX_ *)X : (const TX_ *)in, xc ? ldx : d,                        \
                     gic ? (const TGI_ *)G : (const TGI_ *)g, gic ? ldg : d,                         \
                     goc ? (TGO_ *)dX : (TGO_ *)g, goc ? lddx : d, d, n, rows_sum, run_of(seg[i]),      \
                     nitems, cs.s, (int)(d / 2), partial, pstride, aligned)
#define HARP_GRAD_BWD_TYPES(KK)                                                          \
  do {                                                                                   \
    if (!bf) HARP_GRAD_BWD_RUN(KK, float, float, float);                                 \
    else if (xc && gic && goc) HARP_GRAD_BWD_RUN(KK, uint16_t, uint16_t, uint16_t);      \
    else if (xc && gic) HARP_GRAD_BWD_RUN(KK, uint16_t, uint16_t, float);                \
    else if (xc && goc) HARP_GRAD_BWD_RUN(KK, uint16_t, float, uint16_t);                \
    else if (xc) HARP_GRAD_BWD_RUN(KK, uint16_t, float, float);                          \
    else if (gic) HARP_GRAD_BWD_RUN(KK, float, uint16_t, float);                         \
    else HARP_GRAD_BWD_RUN(KK, float, float, float);                                     \
  } while (0)
        if (seg[i].k == 3) HARP_GRAD_BWD_TYPES(3);
        else HARP_GRAD_BWD_TYPES(2);
#undef HARP_GRAD_BWD_TYPES
#undef HARP_GRAD_BWD_RUN
      } else if (grad_big_stage(plan, seg[i].t0)) {
        const bool own = g_direct && i == nseg - 1;   // reads the caller's G
        const harp_status_t rc = launch_grad_big(plan, seg[i].t0, in, own ? G : (const void *)g, own ? ldg : d, own && bf, g2,
                                                 n, partial, dK[seg[i].t0], st);
        if (rc != HARP_OK) return rc;
        std::swap(g, g2);
        continue;
      } else if (cs.b > 8) {
        const int D = (int)(d / cs.b);
        const dim3 grid((D + 63) / 64, nchunks_big, (cs.b + 3) / 4);
        // gradient passed back: the transposed blocks on the matrix cores where the stage allows
        const bool own = g_direct && i == nseg - 1;   // reads the caller's G
        const float *gsrc = own ? (const float *)G : g;
        const int64_t gld = own ? ldg : d;
        const bool mf = mfma_pass_supported(plan->grad_mfma[1][seg[i].t0], gsrc, gld, g2, d);
        const bool dkm = dk_mfma_supported(cs.b, cs.s, D, in, d, gsrc, gld, partial, nchunks_big);
        if (dkm) launch_dk_mfma(in, d, gsrc, gld, n, rows_big, nchunks_big, D, cs.s, cs.b, partial, st);
#define HARP_GRAD_BIG_BWD(BM)                                                                      \
  if (!dkm)                                                                                        \
    hipLaunchKernelGGL((harp_grad_dk_big_kernel<BM>), grid, dim3(kGradThreads), 0, st, in, g, d, n, \
                       rows_big, D, cs.s, cs.b, partial);                                          \
  if (!mf)                                                                                         \
    hipLaunchKernelGGL((harp_grad_apply_big_kernel<BM, true>), grid, dim3(kGradThreads), 0, st, g, \
                       g2, d, n, rows_big, cs.blocks, D, cs.s, cs.b)
        HARP_GRAD_BIG(cs.b, HARP_GRAD_BIG_BWD);
#undef HARP_GRAD_BIG_BWD
        if (mf && launch_mfma_pass(plan, plan->grad_mfma[1][seg[i].t0], gsrc, gld, HARP_F32, g2, d, HARP_F32, n,
                                   false, st) != HARP_OK)
          return HARP_ERR_DEVICE;
        std::swap(g, g2);
      } else {
        const int D = (int)(d / cs.b);
#define HARP_GRAD_BWD(BB) launch_bwd<BB>(in, g, d, n, rows_sum, nsum, cs.blocks, D, cs.s, partial, st)
        HARP_GRAD_SWITCH(cs.b, HARP_GRAD_BWD)
#undef HARP_GRAD_BWD
      }
    }
    // the run's sub-stages in one reduction launch
    {
      const int b = stages[seg[i].t0].b;
      const int D = (int)(d / b);
      const int64_t total = (int64_t)D * b * b;
      const unsigned gx = (unsigned)std::min<int64_t>((total + 31) / 32, 8192);
      GradReduceOut ro{};
      for (int j = 0; j < seg[i].k; ++j) {
        ro.dK[j] = dK[seg[i].t0 + j];
        ro.signs[j] = (seg[i].t0 + j == 0) ? plan->dev_signs : nullptr;
      }
      hipLaunchKernelGGL(harp_grad_reduce_kernel, dim3(gx, (unsigned)seg[i].k), dim3(kGradThreads), 0, st,
                         partial, pstride, n > 0 ? (b > 8 ? nchunks_big : nsum) : 0, D, b, ro);
    }
  }
  if (sums.nsides > 0) {
    const harp_status_t rc = launch_grad_sums(sums, st);
    if (rc != HARP_OK) return rc;
  }
  if (dX && n > 0 && !dx_direct) {
    if (bf) launch_convert(g, d, (uint16_t *)dX, lddx, n, d, st);
    else launch_convert(g, d, (float *)dX, lddx, n, d, st);
  }
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

}  // namespace harp
