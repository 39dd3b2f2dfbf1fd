// Gradient path, first stages of a plan as ONE segment of 64 consecutive coordinates: six radix-2
// stages or two radix-8 stages at strides 1 .. 32 (the start of every schedule of the layer widths
// served here).  This file holds the rule and the forward kernel, which stores the segment's output for the
// stages behind it; a wave owns one group of 64 coordinates and a run of rows, and nothing crosses waves: no
// barrier in the row loop.  The way back is harp_grad_lead_bwd_kernel (harp_grad_pair.hip).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "harp_internal.h"

namespace harp {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kSegP = 64;         // coordinates per group
constexpr int kSegWaves = 4;      // waves per workgroup: one group, four runs of rows
constexpr int kSegRows = 8;       // rows per step of a wave
constexpr int kSegRowP = 72;      // LDS pitch of a row (floats): stride-8 reads of four rows hit 32 banks

struct SegBlocks {
  const float *blocks[6];         // dense blocks of the stages, [d / b][b][b]
};

// Four consecutive coordinates as loaded, widened when they are used.  VEC: one access of 16 (float32)
// or 8 (bf16) bytes; otherwise one per element, for a caller's rows that are not on such boundaries.
// The same values go through the same arithmetic either way.
template <typename T, bool VEC> struct SegRaw4;
template <> struct SegRaw4<float, true> {
  float4 v;
  __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const float4 *>(p); }
  __device__ __forceinline__ void widen(float (&x)[4]) const { x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w; }
};
template <> struct SegRaw4<uint16_t, true> {
  uint2 v;
  __device__ __forceinline__ void load(const uint16_t *p) { v = *reinterpret_cast<const uint2 *>(p); }
  __device__ __forceinline__ void widen(float (&x)[4]) const {
    x[0] = __uint_as_float(v.x << 16); x[1] = __uint_as_float(v.x & 0xffff0000u);
    x[2] = __uint_as_float(v.y << 16); x[3] = __uint_as_float(v.y & 0xffff0000u);
  }
};
template <> struct SegRaw4<float, false> {
  float v[4];
  __device__ __forceinline__ void load(const float *p) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = p[i];
  }
  __device__ __forceinline__ void widen(float (&x)[4]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = v[i];
  }
};
template <> struct SegRaw4<uint16_t, false> {
  uint32_t v[4];
  __device__ __forceinline__ void load(const uint16_t *p) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = p[i];
  }
  __device__ __forceinline__ void widen(float (&x)[4]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(v[i] << 16);
  }
};
__device__ __forceinline__ void seg_store8(float *p, const float (&v)[8]) {
  *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
  *reinterpret_cast<float4 *>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}

// Eight coordinates base + e s of a row held by one thread: three radix-2 stages at strides s, 2s,
// 4s (R8 false, 48 values) or one radix-8 stage at stride s.  Lane l of a wave holds row
// 4 (l >> 5) + (l & 3) and item (l >> 2) & 7 of a step (the operand layout of the radix-8 product).
template <bool R8> struct Pass8;
template <> struct Pass8<false> {
  float k[3][4][4];
  __device__ __forceinline__ void load(const float *const *blocks, int base, int s, int) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int si = s << i;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int i0 = base + (((p >> i) << (i + 1)) | (p & ((1 << i) - 1))) * s;
        const float4 f = *reinterpret_cast<const float4 *>(blocks[i] + (size_t)((i0 / (2 * si)) * si + i0 % si) * 4);
        k[i][p][0] = f.x; k[i][p][1] = f.y; k[i][p][2] = f.z; k[i][p][3] = f.w;
      }
    }
  }
  __device__ __forceinline__ void forward(float (&v)[8]) const {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int e0 = ((p >> i) << (i + 1)) | (p & ((1 << i) - 1)), e1 = e0 | (1 << i);
        const float a = v[e0], b = v[e1];
        v[e0] = fmaf(b, k[i][p][2], a * k[i][p][0]);
        v[e1] = fmaf(b, k[i][p][3], a * k[i][p][1]);
      }
  }
};
// The radix-8 blocks multiply on the matrix cores: v_mfma_f32_4x4x1_16b_f32 is sixteen independent
// 4 x 4 products, here 8 blocks x 2 groups of four rows, one k (input coordinate) per instruction
// with float32 operands and the same chain of fused multiply-adds in k as the vector units would
// run.  Operand lanes hold four of a block's outputs each, so a block's 64 values cost 16 registers
// per lane and pass instead of 64, and a pass takes 16 instructions of 8 cycles instead of 64 of 4.
template <> struct Pass8<true> {
  float fw[2][8];   // [half h of the outputs][k]: K[k][4 h + i], i = lane & 3
  __device__ __forceinline__ void load(const float *const *blocks, int base, int s, int lane) {
    const float *p = blocks[0] + (size_t)((base / (8 * s)) * s + base % s) * 64;
    const int i = lane & 3;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int k = 0; k < 8; ++k) fw[h][k] = p[k * 8 + 4 * h + i];
  }
  __device__ __forceinline__ void forward(float (&v)[8]) const {
    f4v y[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) y[h] = __builtin_amdgcn_mfma_f32_4x4x1f32(fw[h][k], v[k], y[h], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = y[0][i];
      v[4 + i] = y[1][i];
    }
  }
};

// Values a wave wrote to its own LDS region are about to be read by other lanes of the same wave:
// LDS operations of a wave complete in order; this only keeps the compiler from reordering them.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Rows of one wave: workgroup blockIdx.y walks `rows` rows, wave w the w-th quarter of them
// (rows is a multiple of 32, so the runs of full workgroups are whole steps).
__device__ __forceinline__ void seg_rows(int64_t n, int rows, int wave, int64_t &r0, int64_t &r1) {
  const int per = rows / kSegWaves;
  r0 = (int64_t)blockIdx.y * rows + (int64_t)wave * per;
  r1 = r0 + per < n ? r0 + per : n;
}

// y = x M for the segment.  Rows move in 16-byte pieces, four coordinates per lane and 256
// contiguous bytes per row (lane (g4 = l >> 4, c = l & 15): rows g4 and 4 + g4, coordinates 4c..);
// the wave's LDS region hands them to the two stage passes and back.  Two steps of rows are
// requested ahead.
template <bool R8, bool VEC, typename TX>
__global__ __launch_bounds__(64 * kSegWaves, 2) void harp_grad_seg_fwd_kernel(
    const TX *__restrict__ X, int64_t ldx, float *__restrict__ Y, int64_t ldy, int64_t n, int rows,
    SegBlocks sb) {
  __shared__ __attribute__((aligned(16))) float lds[kSegWaves][kSegRows * kSegRowP];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l = (int)threadIdx.x & 63;
  const int row = 4 * (l >> 5) + (l & 3), item = (l >> 2) & 7, base = (int)blockIdx.x * kSegP;
  const int g4 = l >> 4, c = l & 15;
  int64_t r0, r1;
  seg_rows(n, rows, wave, r0, r1);
  if (r0 >= r1) return;
  float *w = lds[wave], *t = w + row * kSegRowP;
  SegRaw4<TX, VEC> nx[2][2];
  auto fetch = [&](SegRaw4<TX, VEC> (&q)[2], int64_t r) {   // rows past the end repeat the last one and are not stored
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t rr = r + 4 * h + g4 < r1 ? r + 4 * h + g4 : r1 - 1;
      q[h].load(X + rr * ldx + base + 4 * c);
    }
  };
  fetch(nx[0], r0);
  fetch(nx[1], r0 + kSegRows);
  Pass8<R8> pa, pb;
  pa.load(sb.blocks, base + 8 * item, 1, l);
  pb.load(sb.blocks + (R8 ? 1 : 3), base + item, 8, l);
  auto step = [&](SegRaw4<TX, VEC> (&q)[2], int64_t r) {
    float v[8], x[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      q[h].widen(x);
      *reinterpret_cast<float4 *>(w + (4 * h + g4) * kSegRowP + 4 * c) = make_float4(x[0], x[1], x[2], x[3]);
    }
    fetch(q, r + 2 * kSegRows);
    wave_lds_fence();
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = t[8 * item + e];
    pa.forward(v);
    seg_store8(t + 8 * item, v);
    wave_lds_fence();
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = t[item + 8 * e];
    pb.forward(v);
#pragma unroll
    for (int e = 0; e < 8; ++e) t[item + 8 * e] = v[e];
    wave_lds_fence();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4 o = *reinterpret_cast<const float4 *>(w + (4 * h + g4) * kSegRowP + 4 * c);
      if (r + 4 * h + g4 < r1) *reinterpret_cast<float4 *>(Y + (r + 4 * h + g4) * ldy + base + 4 * c) = o;
    }
    wave_lds_fence();
  };
  for (int64_t r = r0; r < r1; r += 2 * kSegRows) {
    step(nx[0], r);
    step(nx[1], r + kSegRows);   // past the end: nothing is stored
  }
}

SegBlocks seg_blocks(const harp_plan *plan, int nst) {
  SegBlocks sb;
  for (int i = 0; i < 6; ++i) sb.blocks[i] = plan->col[DIR_FWD][std::min(i, nst - 1)].blocks;
  return sb;
}

}  // namespace

// Stages 0 .. k-1 of the plan that form the segment (6 of radix 2, 2 of radix 8), or 0.  Orthogonal
// blocks only: the contractions of dM then leave its rounding errors at the size that sums
// taken block by block have.  n >= 64 is the range over which that has been measured and is tested,
// not where the segment stops paying: whole calls with 1 / 8 / 32 / 63 rows in float32 take 61 / 66 /
// 68 / 69 us stage by stage and 54 / 54 / 54 / 54 us with it at 4096 radix 2, 69 / 112 / 122 / 139 and
// 52 / 59 / 68 / 86 us at 11008 (8, 8, 4, 43).  At 64 rows and up it is 1.15 - 3.3 times as fast from d = 128
// (262144 rows: 2811 -> 1220 us radix 2, 3644 -> 1213 us radix 8) to 28672 (64 rows: 126 -> 105, 166 -> 107 us).
int grad_seg_stages(const harp_plan *plan, int64_t n) {
  if (!plan->orthogonal || n < 64) return 0;
  if (n > (int64_t)65535 * 128) return 0;   // (beyond that the grids and the counts of chunks have not been tried)
  return grad_seg_stages(plan->radices);
}
int grad_seg_stages(const std::vector<int32_t> &radices) {
  const int b = radices[0], k = b == 2 ? 6 : (b == 8 ? 2 : 0);
  if (k == 0 || (int)radices.size() <= k) return 0;   // (the first k alone: 64 coordinates and nothing behind them)
  for (int t = 1; t < k; ++t)
    if (radices[t] != b) return 0;
  return k;
}

// Rows of a workgroup (a multiple of 32): no sums here, so a wave reads its blocks once for as many rows
// as three workgroups per compute unit leave it.
static int grad_seg_fwd_rows(const harp_plan *plan, int64_t n) {
  const int64_t groups = plan->d / kSegP;
  const int64_t chunks = std::max<int64_t>(1, 3 * (int64_t)(plan->num_cu > 0 ? plan->num_cu : 256) / groups);
  const int64_t rows = (n + chunks - 1) / chunks;
  return (int)std::min<int64_t>(std::max<int64_t>((rows + 31) / 32 * 32, 32), 1 << 20);
}
// X is the caller's: one access per element where rows do not lie on boundaries of four.
static bool seg_vec(const void *p, int64_t ld, bool bf) { return ld % 4 == 0 && (uintptr_t)p % (bf ? 8 : 16) == 0; }

harp_status_t launch_grad_seg_fwd(const harp_plan *plan, int nst, const void *X, int64_t ldx, bool bf, float *Y,
                                  int64_t n, hipStream_t st) {
  const int rows = grad_seg_fwd_rows(plan, n);
  const dim3 grid((unsigned)(plan->d / kSegP), (unsigned)((n + rows - 1) / rows)), blk(64 * kSegWaves);
  const SegBlocks sb = seg_blocks(plan, nst);
  const int64_t d = plan->d;
  const bool vec = seg_vec(X, ldx, bf);
#define HARP_SEG_FWD(R8, VEC, T)                                                                       \
  hipLaunchKernelGGL((harp_grad_seg_fwd_kernel<R8, VEC, T>), grid, blk, 0, st, (const T *)X, ldx, Y, d, n, \
                     rows, sb)
#define HARP_SEG_FWD_TYPES(R8)                 \
  do {                                         \
    if (bf && vec) HARP_SEG_FWD(R8, true, uint16_t);   \
    else if (bf) HARP_SEG_FWD(R8, false, uint16_t);    \
    else if (vec) HARP_SEG_FWD(R8, true, float);       \
    else HARP_SEG_FWD(R8, false, float);               \
  } while (0)
  if (nst == 2) HARP_SEG_FWD_TYPES(true);
  else HARP_SEG_FWD_TYPES(false);
#undef HARP_SEG_FWD_TYPES
#undef HARP_SEG_FWD
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

}  // namespace harp
