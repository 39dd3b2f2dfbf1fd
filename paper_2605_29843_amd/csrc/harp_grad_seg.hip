// Gradient path, first stages of a plan as ONE segment of 64 consecutive coordinates: six radix-2
// stages or two radix-8 stages at strides 1 .. 32 (the start of every schedule of the layer widths
// served here).  For a group of 64 coordinates the segment is one linear map M = K_0 K_1 .., and
// the loss depends on the blocks inside it only through
//     dM = sum over rows of x^T g     (64 x 64; x = the segment's input, g = the gradient behind it),
// so the rows are walked once for dM -- a 64 x n x 64 product on the matrix cores
// (v_mfma_f32_16x16x4_f32, float32 operands and sums) -- and once per group, not per row, the block
// gradients are taken out of it: with the 64 rows of dM as a batch whose input rows are the
// identity, dK_t[c] = sum over rows i of A_t[i]^T g_{t+1}[i], A_t = I K_0 .. K_{t-1}.
//
// Stage by stage the same six stages took two (radix 2) kernels each way, every one at the copy
// rate of float32 copies of the batch, plus per-chunk partial sums of every block: 2048 x 4096 bf16
// 85 us of 158.  Here a wave owns one group and a run of rows and nothing crosses waves until the
// end: no barrier in the row loop, x and g read once, dX written once.  The matrix product is
// 64 multiply-adds per coordinate at twice the vector rate (7 us for 2048 x 4096), below the time
// the rows take to stream.  Measured (whole call): 2048 x 4096 bf16 radix 2 158 -> 115 us,
// 1537 x 11008 float32 (8, 8, 4, 43) 653 -> 349 us (the three kernels: 29 + 52 + 10 us for the 412 MB of
// five passes over the batch and the partial sums of 13 chunks, written and read).
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

__device__ __forceinline__ uint32_t seg_bf16(float f) {   // round to nearest even, NaN kept quiet
  const uint32_t u = __float_as_uint(f);
  const uint32_t rounded = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  return ((u & 0x7fffffffu) > 0x7f800000u) ? ((u >> 16) | 0x40u) : rounded;
}

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
template <bool VEC>
__device__ __forceinline__ void seg_store4(float *p, float4 v) {
  if constexpr (VEC) {
    *reinterpret_cast<float4 *>(p) = v;
  } else {
    p[0] = v.x; p[1] = v.y; p[2] = v.z; p[3] = v.w;
  }
}
template <bool VEC>
__device__ __forceinline__ void seg_store4(uint16_t *p, float4 v) {
  if constexpr (VEC) {
    *reinterpret_cast<uint2 *>(p) = make_uint2(seg_bf16(v.x) | (seg_bf16(v.y) << 16), seg_bf16(v.z) | (seg_bf16(v.w) << 16));
  } else {
    p[0] = (uint16_t)seg_bf16(v.x); p[1] = (uint16_t)seg_bf16(v.y);
    p[2] = (uint16_t)seg_bf16(v.z); p[3] = (uint16_t)seg_bf16(v.w);
  }
}

// Eight coordinates base + e s of a row held by one thread: three radix-2 stages at strides s, 2s,
// 4s (R8 false, 48 values) or one radix-8 stage at stride s.  Lane l of a wave holds row
// 4 (l >> 5) + (l & 3) and item (l >> 2) & 7 of a step (the operand layout of the radix-8 product).
template <bool R8> struct Pass8;
template <> struct Pass8<false> {
  float k[3][4][4];
  template <bool FWD>
  __device__ __forceinline__ void load_as(const float *const *blocks, int base, int s, int) {
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
  __device__ __forceinline__ void backward(float (&v)[8]) const {   // v K^T, stages from the last to the first
#pragma unroll
    for (int i = 2; i >= 0; --i)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int e0 = ((p >> i) << (i + 1)) | (p & ((1 << i) - 1)), e1 = e0 | (1 << i);
        const float a = v[e0], b = v[e1];
        v[e0] = fmaf(b, k[i][p][1], a * k[i][p][0]);
        v[e1] = fmaf(b, k[i][p][3], a * k[i][p][2]);
      }
  }
};
// The radix-8 blocks multiply on the matrix cores: v_mfma_f32_4x4x1_16b_f32 is sixteen independent
// 4 x 4 products, here 8 blocks x 2 groups of four rows, one k (input coordinate) per instruction
// with float32 operands and the same chain of fused multiply-adds in k as the vector units would
// run.  Operand lanes hold four of a block's outputs each, so a block's 64 values cost 16 registers
// per lane and pass instead of 64 (the backward kernel: 246 registers, no room to request rows
// ahead), and a pass takes 16 instructions of 8 cycles instead of 64 of 4.
template <> struct Pass8<true> {
  float fw[2][8];   // [half h of the outputs][k]: forward K[k][4 h + i], backward K[4 h + i][k]; i = lane & 3
  template <bool FWD>
  __device__ __forceinline__ void load_as(const float *const *blocks, int base, int s, int lane) {
    const float *p = blocks[0] + (size_t)((base / (8 * s)) * s + base % s) * 64;
    const int i = lane & 3;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (FWD) {
#pragma unroll
        for (int k = 0; k < 8; ++k) fw[h][k] = p[k * 8 + 4 * h + i];
      } else {
        const float4 a = *reinterpret_cast<const float4 *>(p + (4 * h + i) * 8);
        const float4 b = *reinterpret_cast<const float4 *>(p + (4 * h + i) * 8 + 4);
        fw[h][0] = a.x; fw[h][1] = a.y; fw[h][2] = a.z; fw[h][3] = a.w;
        fw[h][4] = b.x; fw[h][5] = b.y; fw[h][6] = b.z; fw[h][7] = b.w;
      }
    }
  }
  __device__ __forceinline__ void multiply(float (&v)[8]) const {
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
  __device__ __forceinline__ void forward(float (&v)[8]) const { multiply(v); }
  __device__ __forceinline__ void backward(float (&v)[8]) const { multiply(v); }
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
  pa.template load_as<true>(sb.blocks, base + 8 * item, 1, l);
  pb.template load_as<true>(sb.blocks + (R8 ? 1 : 3), base + item, 8, l);
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

// dM += x^T g over the wave's rows, and dX = g M^T.  Lane (g4 = l >> 4, c = l & 15) loads coordinates
// 4c .. 4c+3 of rows g4 and 4 + g4: element t of those four is exactly its operand of a 16x16x4
// product whose row (column) index c stands for coordinate 4c + t, so x and g go from memory
// into the matrix cores with no exchange.  g then passes through the wave's LDS region
// into the layout of the two stage passes, and dX back into the layout of the loads.  dX may be X:
// a lane reads its pieces of a row before it writes them and no other lane touches them (X is not
// __restrict__; the last row read again past the end is replaced by zeros).
template <bool R8, bool VEC, typename TX>
__global__ __launch_bounds__(64 * kSegWaves, 2) void harp_grad_seg_bwd_kernel(
    const TX *X, int64_t ldx, const float *__restrict__ G, int64_t ldg, TX *dX, int64_t lddx,
    int64_t n, int rows, SegBlocks sb, float *__restrict__ partial) {
  constexpr int kTile = kSegP * kSegP;
  __shared__ __attribute__((aligned(16))) float lds[kSegWaves * kTile];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l = (int)threadIdx.x & 63;
  const int row = 4 * (l >> 5) + (l & 3), item = (l >> 2) & 7, base = (int)blockIdx.x * kSegP;
  const int g4 = l >> 4, c = l & 15;
  int64_t r0, r1;
  seg_rows(n, rows, wave, r0, r1);
  f4v acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = (f4v){0.f, 0.f, 0.f, 0.f};
  if (r0 < r1) {
    float *w = lds + wave * kTile;
    float *t = w + row * kSegRowP;
    SegRaw4<TX, VEC> nx[2][2];
    SegRaw4<float, true> ng[2][2];
    auto fetch = [&](SegRaw4<TX, VEC> (&qx)[2], SegRaw4<float, true> (&qg)[2], int64_t r) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t rr = r + 4 * h + g4 < r1 ? r + 4 * h + g4 : r1 - 1;
        qx[h].load(X + rr * ldx + base + 4 * c);
        qg[h].load(G + rr * ldg + base + 4 * c);
      }
    };
    fetch(nx[0], ng[0], r0);
    fetch(nx[1], ng[1], r0 + kSegRows);
    Pass8<R8> pa, pb;
    pa.template load_as<false>(sb.blocks, base + 8 * item, 1, l);
    pb.template load_as<false>(sb.blocks + (R8 ? 1 : 3), base + item, 8, l);
    auto step = [&](SegRaw4<TX, VEC> (&qx)[2], SegRaw4<float, true> (&qg)[2], int64_t r) {
      float x[2][4], g[2][4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        qx[h].widen(x[h]);
        qg[h].widen(g[h]);
        const bool ok = r + 4 * h + g4 < r1;   // rows past the end enter as zeros
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[h][i] = ok ? x[h][i] : 0.f;
          g[h][i] = ok ? g[h][i] : 0.f;
        }
        *reinterpret_cast<float4 *>(w + (4 * h + g4) * kSegRowP + 4 * c) =
            make_float4(g[h][0], g[h][1], g[h][2], g[h][3]);
      }
      fetch(qx, qg, r + 2 * kSegRows);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[h][a], g[h][b], acc[a][b], 0, 0, 0);
      if (dX != nullptr) {
        float v[8];
        wave_lds_fence();
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = t[item + 8 * e];
        pb.backward(v);
#pragma unroll
        for (int e = 0; e < 8; ++e) t[item + 8 * e] = v[e];
        wave_lds_fence();
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = t[8 * item + e];
        pa.backward(v);
        seg_store8(t + 8 * item, v);
        wave_lds_fence();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float4 o = *reinterpret_cast<const float4 *>(w + (4 * h + g4) * kSegRowP + 4 * c);
          if (r + 4 * h + g4 < r1) seg_store4<VEC>(dX + (r + 4 * h + g4) * lddx + base + 4 * c, o);
        }
        wave_lds_fence();
      }
    };
    for (int64_t r = r0; r < r1; r += 2 * kSegRows) {
      step(nx[0], ng[0], r);
      step(nx[1], ng[1], r + kSegRows);   // past the end: zeros, nothing is stored
    }
  }
  // the four waves' sums, in the order of the rows, to the chunk's partial sums [64][64]
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<float4 *>(lds + wave * kTile + (16 * g4 + 4 * i + a) * kSegP + 4 * c) =
          make_float4(acc[a][0][i], acc[a][1][i], acc[a][2][i], acc[a][3][i]);
  __syncthreads();
  float *out = partial + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kTile;
  for (int e = 4 * (int)threadIdx.x; e < kTile; e += 4 * 64 * kSegWaves) {
    float4 s = *reinterpret_cast<const float4 *>(lds + e);
#pragma unroll
    for (int q = 1; q < kSegWaves; ++q) {
      const float4 f = *reinterpret_cast<const float4 *>(lds + q * kTile + e);
      s.x += f.x; s.y += f.y; s.z += f.z; s.w += f.w;
    }
    *reinterpret_cast<float4 *>(out + e) = s;
  }
}

// dK of the segment's stages out of dM (chunks of rows added in ascending order within each eight, then
// the sums of eight in ascending order).  One workgroup per group; everything in LDS.  A_t[i][j] is zero unless i and j share the digits from t up, so a
// row of A_t is kept as its S_t entries j = (digits of i from t up, lo), lo < S_t.
struct SegOut {
  float *dK[6];
};
constexpr int kExpThreads = 1024;
template <bool R8>
__global__ __launch_bounds__(kExpThreads) void harp_grad_seg_expand_kernel(
    const float *__restrict__ partial, int nchunks, SegBlocks sb, const int8_t *__restrict__ signs, SegOut out) {
  constexpr int B = R8 ? 8 : 2, M = R8 ? 2 : 6, LB = R8 ? 3 : 1;   // radix, stages, log2(radix)
  constexpr int NB = kSegP / B, NK = kSegP * B;                   // blocks and block values per stage
  constexpr int GP = kSegP + 1;
  constexpr int NA = R8 ? 64 * 9 : 64 * (2 + 4 + 8 + 16 + 32 + 5);   // rows of S_t + 1 floats, t >= 1
  __shared__ float g[kSegP * GP], K[M * NK], A[NA];
  const int tid = (int)threadIdx.x, grp = (int)blockIdx.x;
  for (int e = tid; e < M * NK; e += kExpThreads) K[e] = sb.blocks[e / NK][(size_t)grp * NK + e % NK];
  const float *p = partial + (size_t)grp * (kSegP * kSegP);
  const size_t step = (size_t)gridDim.x * (kSegP * kSegP);
  {   // thread tid sums entries 4 tid .. 4 tid + 3; eight chunks in flight
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int q0 = 0; q0 < nchunks; q0 += 8) {
      float4 f[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        f[q] = *reinterpret_cast<const float4 *>(p + (q0 + q < nchunks ? q0 + q : 0) * step + 4 * tid);
      float4 part = f[0];
#pragma unroll
      for (int q = 1; q < 8; ++q)
        if (q0 + q < nchunks) {
          part.x += f[q].x; part.y += f[q].y; part.z += f[q].z; part.w += f[q].w;
        }
      s.x += part.x; s.y += part.y; s.z += part.z; s.w += part.w;
    }
    float *o = g + (tid >> 4) * GP + 4 * (tid & 15);
    o[0] = s.x; o[1] = s.y; o[2] = s.z; o[3] = s.w;
  }
  __syncthreads();
  // A_{t+1}[i][r2 S + lo] = A_t[i][lo] K_t[block of (hi, lo)][digit t of i][r2]
  int offA[M];
  offA[0] = 0;
#pragma unroll
  for (int t = 1, o = 0; t < M; ++t) {
    offA[t] = o;
    o += 64 * ((1 << (LB * t)) + 1);
  }
#pragma unroll
  for (int t = 0; t + 1 < M; ++t) {
    const int S = 1 << (LB * t);
    for (int e = tid; e < 64 * S * B; e += kExpThreads) {
      const int i = e / (S * B), j = e % (S * B), r2 = j / S, lo = j % S;
      const int r = (i / S) % B, hi = i / (S * B);
      const float a = t == 0 ? 1.0f : A[offA[t] + i * (S + 1) + lo];
      A[offA[t + 1] + i * (S * B + 1) + j] = a * K[t * NK + (hi * S + lo) * (B * B) + r * B + r2];
    }
    __syncthreads();
  }
#pragma unroll
  for (int t = M - 1; t >= 0; --t) {
    const int S = 1 << (LB * t);
    {   // TPO neighbouring threads share the S products of one value
      constexpr int TPO = kExpThreads / NK;
      const int e = tid / TPO, part = tid % TPO;
      const int c = e / (B * B), r = (e / B) % B, r2 = e % B, lo = c % S, hi = c / S;
      float s = 0.f;
      for (int q = part; q < S; q += TPO) {
        const int i = (hi * B + r) * S + q;
        const float a = t == 0 ? 1.0f : A[offA[t] + i * (S + 1) + lo];
        s = fmaf(a, g[i * GP + (hi * B + r2) * S + lo], s);
      }
#pragma unroll
      for (int x = 1; x < TPO; x <<= 1) s += __shfl_xor(s, x);
      // the image holds diag(sigma) K_0: row r of dK_0 takes the sign of coordinate c B + r
      if (t == 0 && signs) s *= (float)signs[(size_t)grp * kSegP + c * B + r];
      if (part == 0) out.dK[t][(size_t)grp * NK + e] = s;
    }
    if (t == 0) break;
    __syncthreads();
    for (int e = tid; e < kSegP * NB; e += kExpThreads) {   // g <- g K_t^T
      const int i = e / NB, c = e % NB, lo = c % S, hi = c / S;
      float *gr = g + i * GP + hi * B * S + lo;
      const float *k = K + t * NK + c * (B * B);
      float v[B];
#pragma unroll
      for (int r = 0; r < B; ++r) v[r] = gr[r * S];
#pragma unroll
      for (int r = 0; r < B; ++r) {
        float s = v[0] * k[r * B];
#pragma unroll
        for (int r2 = 1; r2 < B; ++r2) s = fmaf(v[r2], k[r * B + r2], s);
        gr[r * S] = s;
      }
    }
    __syncthreads();
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
  if (!plan->orthogonal || n < 64 || plan->d <= kSegP || plan->d % kSegP) return 0;
  if (n > (int64_t)65535 * 128) return 0;   // one workgroup per 128 rows at most: blockIdx.y
  const int b = plan->radices[0], k = b == 2 ? 6 : (b == 8 ? 2 : 0);
  if (k == 0 || plan->m <= k) return 0;
  for (int t = 1; t < k; ++t)
    if (plan->radices[t] != b) return 0;
  return k;
}

// Rows of a workgroup (a multiple of 32).  Backward: at most 128, so that no sum runs over more than
// 32 rows before it meets the others (256 left dK of 1537 x 11008 float32 at 2.2e-7 of its norm
// from the float64 result where the sums by 8 rows are at 1.9e-7), at least 32.  Forward: no sums, so
// a wave reads its blocks once for as many rows as three workgroups per compute unit leave it.
static int64_t grad_seg_target(const harp_plan *plan) {   // chunks that give four workgroups per compute unit
  const int64_t groups = plan->d / kSegP;
  return std::max<int64_t>(1, (4 * (int64_t)(plan->num_cu > 0 ? plan->num_cu : 256) + groups - 1) / groups);
}
static int grad_seg_rows(const harp_plan *plan, int64_t n) {
  const int64_t chunks = grad_seg_target(plan);
  const int64_t rows = std::min<int64_t>((n + chunks - 1) / chunks, 128);
  return (int)std::max<int64_t>((rows + 31) / 32 * 32, 32);
}
static int grad_seg_fwd_rows(const harp_plan *plan, int64_t n) {
  const int64_t groups = plan->d / kSegP;
  const int64_t chunks = std::max<int64_t>(1, 3 * (int64_t)(plan->num_cu > 0 ? plan->num_cu : 256) / groups);
  const int64_t rows = (n + chunks - 1) / chunks;
  return (int)std::min<int64_t>(std::max<int64_t>((rows + 31) / 32 * 32, 32), 1 << 20);
}
static int64_t grad_seg_chunks(const harp_plan *plan, int64_t n) {
  const int rows = grad_seg_rows(plan, n);
  return (n + rows - 1) / rows;
}
// Room for at least grad_seg_chunks(n) chunks that never falls as n grows: rows per chunk are rounded up
// to multiples of 32, so the chunks themselves get fewer wherever that rounding takes a step.
size_t grad_seg_partial_bytes(const harp_plan *plan, int64_t n) {
  const int64_t chunks = std::max<int64_t>((n + 127) / 128, std::min<int64_t>((n + 31) / 32, grad_seg_target(plan)));
  return (size_t)chunks * (size_t)plan->d * kSegP * 4;
}

// X and dX are the caller's: one access per element where rows do not lie on boundaries of four.
// Whole call with X shifted by one element, 2048 x 4096 float32 radix 2: 117 us (113 us where it is
// not shifted; 174 us stage by stage).
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

harp_status_t launch_grad_seg_bwd(const harp_plan *plan, int nst, const void *X, int64_t ldx, bool bf,
                                  const float *G, void *dX, int64_t lddx, int64_t n, float *partial,
                                  float *const *dK, hipStream_t st) {
  const int64_t chunks = grad_seg_chunks(plan, n);
  const dim3 grid((unsigned)(plan->d / kSegP), (unsigned)chunks), blk(64 * kSegWaves);
  const SegBlocks sb = seg_blocks(plan, nst);
  const int rows = grad_seg_rows(plan, n);
  const int64_t d = plan->d;
  const bool vec = seg_vec(X, ldx, bf) && (!dX || seg_vec(dX, lddx, bf));
  SegOut out{};
  for (int t = 0; t < nst; ++t) out.dK[t] = dK[t];
#define HARP_SEG_BWD(R8, VEC, T)                                                                         \
  hipLaunchKernelGGL((harp_grad_seg_bwd_kernel<R8, VEC, T>), grid, blk, 0, st, (const T *)X, ldx, G, d, \
                     (T *)dX, lddx, n, rows, sb, partial)
#define HARP_SEG_BWD_TYPES(R8)                                                                           \
  do {                                                                                                   \
    if (bf && vec) HARP_SEG_BWD(R8, true, uint16_t);                                                     \
    else if (bf) HARP_SEG_BWD(R8, false, uint16_t);                                                      \
    else if (vec) HARP_SEG_BWD(R8, true, float);                                                         \
    else HARP_SEG_BWD(R8, false, float);                                                                 \
    hipLaunchKernelGGL((harp_grad_seg_expand_kernel<R8>), dim3(grid.x), dim3(kExpThreads), 0, st, partial, \
                       (int)chunks, sb, plan->dev_signs, out);                                           \
  } while (0)
  if (nst == 2) HARP_SEG_BWD_TYPES(true);
  else HARP_SEG_BWD_TYPES(false);
#undef HARP_SEG_BWD_TYPES
#undef HARP_SEG_BWD
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

}  // namespace harp
