// Column passes of 512 rows: three radix-8 stages of plan_U along the row index of the matrix in one trip
// through device memory, where the passes of up to 128 rows (harp_col.hip) need two (28672 = 8 8 8 | 8 7:
// two trips instead of three).
//
// A tile is 512 rows x 32 columns of float32 in LDS (66 KB, two workgroups per compute unit: one's
// loads and stores run under the other's products).  All columns of a tile share their blocks, sixteen of
// which times four columns are one v_mfma_f32_4x4x1_16b_f32.  The stages at tile strides 1 and 8 run on
// registers, a lane holding the 64 rows of one group at one column (lane: 8 groups, two quads of
// columns); the stage at tile stride 64 on 8 rows at each of eight quads.  The tile makes one round trip
// through LDS in either direction for each of the two, and one between them and device memory.
// Sums run over r in ascending order from zero, as in the kernels whose place it takes.
//
// plan_V's streamed radix-2 stage on the top digit (BV == 2) rides along: the tile is then two segments of
// 16 columns half a row apart, and the stage is applied to the pieces as they arrive.
//
// Bound by bytes: 48 KB of block values per tile come from the L2 beside its 64 KB in and out.
// 28672 x 8192 bf16, radix-8 schedules: one trip of 465 us (1.88 GB, 4.0 TB/s) in the place of 365 (64 rows)
// and 347 us (8 rows); the rotation 1415 -> 1148 us.  Where the passes get fewer they are faster at every
// size (plan_U only, float32, whole call forward / back, us): 512 x 32 12.4 / 13.0 -> 7.1 / 6.9, 512 x 65536
// 119 / 118 -> 59 / 55, 14336 x 4096 319 / 301 -> 246 / 221, 28672 x 32 30 -> 19, 28672 x 2048 323 / 318 ->
// 253 / 239; with plan_V, bf16: 13824 x 5120 893 / 870 -> 454 / 515 (chunks of plan_V included).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "harp_internal.h"
#include "harp_mfma4.h"

namespace harp {

namespace {

constexpr int kWideP = 512;                     // rows per tile
constexpr int kWideCols = 32;                   // columns per tile
constexpr int kWideThreads = 256;
constexpr int kWideGroup = 64 * kWideCols + 8;  // LDS floats per 64 rows: eight groups x 8 columns hit 32 banks twice
constexpr size_t kWideLds = (size_t)8 * kWideGroup * 4;
// block values of a tile: stages at tile strides 1 and 8 as [batch 8][piece 4][group 8][i 4][4], the stage
// at tile stride 64 as [block of 16 rows 4][piece 4][slot 16][i 4][4]
constexpr int kWideTile = 3 * 4096;

// the four columns of quad cq of tile row j; quads are permuted by the row so that four columns x
// sixteen rows, eight quads of a row and eight groups x two quads all spread over the banks
__device__ __forceinline__ int wide_pos(int j, int cq) {
  return (j >> 6) * kWideGroup + (j & 63) * kWideCols + ((cq ^ (j & 7)) << 2);
}

// A 16-byte piece of one row: four columns of float32 or eight of bf16.
template <typename T> struct WidePiece;
template <> struct WidePiece<float> {
  static constexpr int NQ = 1;
  f4v v;
  __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const f4v *>(p); }
  __device__ __forceinline__ void widen(f4v (&q)[1]) const { q[0] = v; }
  __device__ static __forceinline__ void store(float *p, const f4v (&q)[1]) { *reinterpret_cast<f4v *>(p) = q[0]; }
};
template <> struct WidePiece<uint16_t> {
  static constexpr int NQ = 2;
  u4v v;
  __device__ __forceinline__ void load(const uint16_t *p) { v = *reinterpret_cast<const u4v *>(p); }
  __device__ __forceinline__ void widen(f4v (&q)[2]) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      q[e >> 1][2 * (e & 1)] = __uint_as_float(v[e] << 16);
      q[e >> 1][2 * (e & 1) + 1] = __uint_as_float(v[e] & 0xffff0000u);
    }
  }
  __device__ static __forceinline__ void store(uint16_t *p, const f4v (&q)[2]) {
    const u4v o = {pack2(q[0][0], q[0][1]), pack2(q[0][2], q[0][3]), pack2(q[1][0], q[1][1]), pack2(q[1][2], q[1][3])};
    *reinterpret_cast<u4v *>(p) = o;
  }
};

template <typename TI, typename TO, int BV, bool DESC>
__global__ __launch_bounds__(kWideThreads, 2) void harp_colwide_kernel(
    const TI *src, int64_t lds_, TO *dst, int64_t ldd, int S, unsigned nct, unsigned total,
    const float *__restrict__ image, const float *__restrict__ vparams, int Sv) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slot = lane >> 2, col = lane & 3;
  // workgroups of one XCD take neighbouring columns of the same rows: they share lines and block values
  const unsigned id = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (id >= total) return;   // the whole workgroup
  const unsigned T = id / nct;
  const int c0 = (int)(id % nct) * (kWideCols / BV);
  const int64_t row0 = (int64_t)(T / (unsigned)S) * kWideP * S + T % (unsigned)S;
  src += row0 * lds_ + c0;
  dst += row0 * ldd + c0;
  const float *img = image + (size_t)T * kWideTile;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(img), 0, kWideTile * 4, 0x00020000);
  const BlockValues<512> low = {rsrc, ((slot & 7) * 4 + col) * 16};
  const BlockValues<1024> high = {rsrc, lane * 16};
  constexpr int kA = 0, kB = 32, kC = 32;   // first pieces (of 512, 512 and 1024 bytes)
  constexpr int RING = 12;
  f4v ring[RING], hi4[4];

  // rows from device memory, all requested at once; BV == 2: the same columns of both segments
  {
    using P = WidePiece<TI>;
    constexpr int PR = kWideCols / BV / (4 * P::NQ);   // pieces of a row in one segment
    constexpr int RS = kWideThreads / PR, NS = kWideP / RS;
    const int pc = tid % PR, rr = tid / PR;
    P raw[BV][NS];
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int h = 0; h < BV; ++h)
        raw[h][k].load(src + (int64_t)(rr + k * RS) * S * lds_ + (int64_t)h * Sv + pc * 4 * P::NQ);
    if constexpr (!DESC) {
#pragma unroll
      for (int s = 0; s < RING; ++s) ring[s] = low.piece(kA, s);
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) hi4[s] = high.piece(kC, 4 * w + s);
    }
    f4v kv[4][P::NQ];
    if constexpr (BV == 2) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int q = 0; q < P::NQ; ++q)
          kv[v][q] = *reinterpret_cast<const f4v *>(vparams + (size_t)v * Sv + c0 + pc * 4 * P::NQ + 4 * q);
    }
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      f4v x[BV][P::NQ];
#pragma unroll
      for (int h = 0; h < BV; ++h) raw[h][k].widen(x[h]);
      if constexpr (BV == 2) {
#pragma unroll
        for (int q = 0; q < P::NQ; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float a = x[0][q][e], b = x[BV - 1][q][e];
            x[0][q][e] = fmaf(b, kv[2][q][e], a * kv[0][q][e]);
            x[BV - 1][q][e] = fmaf(b, kv[3][q][e], a * kv[1][q][e]);
          }
      }
#pragma unroll
      for (int h = 0; h < BV; ++h)
#pragma unroll
        for (int q = 0; q < P::NQ; ++q)
          *reinterpret_cast<f4v *>(lds + wide_pos(rr + k * RS, h * (8 / BV) + pc * P::NQ + q)) = x[h][q];
    }
  }
  lds_barrier();
  auto low_stages = [&]() {   // tile strides 1 and 8: group g of 64 rows, quad 2 w + (slot >> 3)
    const int g = slot & 7, cq = 2 * w + (slot >> 3);
    float x[1][64];
#pragma unroll
    for (int e = 0; e < 64; ++e) x[0][e] = lds[wide_pos(64 * g + e, cq) + col];
    if constexpr (!DESC) {
      chain_stage<8, 8, 8, 1, 32>(x, ring, low, kA, kB);
#pragma unroll
      for (int s = 0; s < 4; ++s) hi4[s] = high.piece(kC, 4 * w + s);
      chain_stage<8, 8, 1, 8, 0>(x, ring, low, kB, kB);
    } else {
      chain_stage<8, 8, 1, 8, 32>(x, ring, low, kB, kA);
      chain_stage<8, 8, 8, 1, 0>(x, ring, low, kA, kA);
    }
#pragma unroll
    for (int e = 0; e < 64; ++e) lds[wide_pos(64 * g + e, cq) + col] = x[0][e];
  };
  auto high_stage = [&]() {   // tile stride 64: rows lo + 64 r, lo = 16 w + slot, every quad
    const int lo = 16 * w + slot;
#pragma unroll
    for (int c = 0; c < 8; c += 2) {
      float x[2][8];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 8; ++r) x[h][r] = lds[wide_pos(lo + 64 * r, c + h) + col];
      f4v y[2][2];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int o = 0; o < 2; ++o) y[h][o] = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            y[h][o] = __builtin_amdgcn_mfma_f32_4x4x1f32(hi4[(2 * r + o) / 4][(2 * r + o) % 4], x[h][r], y[h][o], 0, 0, 0);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 8; ++r) lds[wide_pos(lo + 64 * r, c + h) + col] = y[h][r / 4][r % 4];
    }
  };
  if constexpr (!DESC) {
    low_stages();
    lds_barrier();
    high_stage();
  } else {
#pragma unroll
    for (int s = 0; s < RING; ++s) ring[s] = low.piece(kB, s);
    high_stage();
    lds_barrier();
    low_stages();
  }
  lds_barrier();
  {
    using P = WidePiece<TO>;
    constexpr int PR = kWideCols / BV / (4 * P::NQ);
    constexpr int RS = kWideThreads / PR, NS = kWideP / RS;
    const int pc = tid % PR, rr = tid / PR;
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int h = 0; h < BV; ++h) {
        f4v q[P::NQ];
#pragma unroll
        for (int e = 0; e < P::NQ; ++e)
          q[e] = *reinterpret_cast<const f4v *>(lds + wide_pos(rr + k * RS, h * (8 / BV) + pc * P::NQ + e));
        P::store(dst + (int64_t)(rr + k * RS) * S * ldd + (int64_t)h * Sv + pc * 4 * P::NQ, q);
      }
  }
}

template <typename TI, typename TO, int BV, bool DESC>
harp_status_t launch_wide_inst(const harp_plan *plan, const ColPass &hp, const void *src, int64_t lds_, void *dst,
                               int64_t ldd, int64_t nrows, int64_t ncols, const float *vparams, int Sv,
                               hipStream_t stream) {
  const int64_t nct = ncols / kWideCols, total = (nrows / kWideP) * nct;
  if (total <= 0) return HARP_OK;
  if (total > 0x7ffffff0 || kWideLds > (size_t)plan->lds_bytes) return HARP_ERR_UNSUPPORTED;
  auto kern = harp_colwide_kernel<TI, TO, BV, DESC>;
  static thread_local int attr_done_dev = -1;   // per instantiation
  if (attr_done_dev != plan->device) {
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            plan->lds_bytes) != hipSuccess) {
      (void)hipGetLastError();
      return HARP_ERR_DEVICE;
    }
    attr_done_dev = plan->device;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)((total + 7) / 8 * 8)), dim3(kWideThreads), kWideLds, stream, (const TI *)src,
                     lds_, (TO *)dst, ldd, (int)hp.S, (unsigned)nct, (unsigned)total, hp.packed, vparams, Sv);
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

template <typename TI, typename TO>
harp_status_t launch_wide_typed(const harp_plan *plan, const ColPass &hp, const void *src, int64_t lds_, void *dst,
                                int64_t ldd, int64_t nrows, int64_t ncols, const PassDesc *vp, hipStream_t stream) {
  const float *vpar = vp ? vp->params : nullptr;
  const int Sv = vp ? (int)vp->S : 0;
#define HARP_WIDE(BV, DESC) \
  launch_wide_inst<TI, TO, BV, DESC>(plan, hp, src, lds_, dst, ldd, nrows, ncols, vpar, Sv, stream)
  if (vp) return hp.desc ? HARP_WIDE(2, true) : HARP_WIDE(2, false);
  return hp.desc ? HARP_WIDE(1, true) : HARP_WIDE(1, false);
#undef HARP_WIDE
}

}  // namespace

// Stages [i0, i0 + 3) of the column image as one pass of 512 rows: three radix-8 stages on adjacent digits, in
// ascending or descending order.
bool col_wide_stages(const std::vector<ColStage> &st, int i0) {
  if (i0 < 0 || i0 + 3 > (int)st.size()) return false;
  for (int e = 0; e < 3; ++e)
    if (st[i0 + e].b != 8) return false;
  const int64_t a = st[i0].s, b = st[i0 + 1].s, c = st[i0 + 2].s;
  return (b == 8 * a && c == 8 * b) || (a == 8 * b && b == 8 * c);
}

// The block values of that pass in the kernel's order (host_image: the plan's dense blocks on the host).
void col_wide_image(const std::vector<ColStage> &st, int i0, int64_t d, const float *host_image, ColPass &cp,
                    std::vector<float> &out) {
  const bool desc = st[i0].s > st[i0 + 1].s;
  cp.P = kWideP;
  cp.S = (int)st[desc ? i0 + 2 : i0].s;
  cp.desc = desc ? 1 : 0;
  const int64_t S = cp.S, tiles = d / kWideP;
  out.assign((size_t)tiles * kWideTile, 0.0f);
  for (int e = 0; e < 3; ++e) {   // by stride
    const ColStage &cs = st[desc ? i0 + 2 - e : i0 + e];
    const float *blocks = host_image + (cs.blocks - st[0].blocks);
    const int64_t s = cs.s;
    for (int64_t T = 0; T < tiles; ++T) {
      float *o = out.data() + (size_t)T * kWideTile + e * 4096;
      const int64_t row0 = (T / S) * kWideP * S + T % S;
      for (int n = 0; n < 64; ++n) {   // block n of the tile: group / slot and batch
        const int sl = e < 2 ? n / 8 : n % 16, bt = e < 2 ? n % 8 : n / 16;
        const int j0 = e == 0 ? 64 * sl + 8 * bt : (e == 1 ? 64 * sl + bt : 16 * bt + sl);
        const int64_t row = row0 + (int64_t)j0 * S;
        const float *K = blocks + ((row / (8 * s)) * s + row % s) * 64;
        const int slots = e < 2 ? 8 : 16;
        for (int r = 0; r < 8; ++r)
          for (int c = 0; c < 8; ++c) {
            const int wv = 2 * r + c / 4;
            o[((size_t)(bt * 4 + wv / 4) * slots * 4 + sl * 4 + c % 4) * 4 + wv % 4] = K[r * 8 + c];
          }
      }
    }
  }
}

// 16-byte pieces on both sides and whole tiles; vp: plan_V's streamed radix-2 stage on the top digit rides along
bool col_wide_supported(const harp_plan *plan, const ColPass &hp, const PassDesc *vp, const void *src, int64_t lds_,
                        harp_dtype_t dt_src, const void *dst, int64_t ldd, harp_dtype_t dt_dst, int64_t nrows,
                        int64_t ncols) {
  if (!hp.packed || hp.P != kWideP || nrows % kWideP != 0 || kWideLds > (size_t)plan->lds_bytes) return false;
  if ((dt_src != HARP_F32 && dt_src != HARP_BF16) || (dt_dst != HARP_F32 && dt_dst != HARP_BF16)) return false;
  if (lds_ % (dt_src == HARP_F32 ? 4 : 8) || ldd % (dt_dst == HARP_F32 ? 4 : 8)) return false;
  if ((uintptr_t)src % 16 || (uintptr_t)dst % 16) return false;
  if ((nrows / kWideP) * (ncols / kWideCols) > 0x7ffffff0) return false;
  if (vp)
    return vp->kind == PASS_POW2_DENSE && vp->k == 1 && vp->P == 2 && vp->V == 4 && !vp->tied &&
           2 * (int64_t)vp->S == ncols && vp->nq == vp->S && vp->nqp == vp->nq && vp->S % (kWideCols / 2) == 0 &&
           (uintptr_t)vp->params % 16 == 0;
  return ncols % kWideCols == 0;
}

harp_status_t launch_col_wide(const harp_plan *plan, const ColPass &hp, const PassDesc *vp, const void *src,
                              int64_t lds_, harp_dtype_t dt_src, void *dst, int64_t ldd, harp_dtype_t dt_dst,
                              int64_t nrows, int64_t ncols, hipStream_t stream) {
  if (!col_wide_supported(plan, hp, vp, src, lds_, dt_src, dst, ldd, dt_dst, nrows, ncols)) return HARP_ERR_UNSUPPORTED;
  if (dt_src == HARP_F32)
    return dt_dst == HARP_F32 ? launch_wide_typed<float, float>(plan, hp, src, lds_, dst, ldd, nrows, ncols, vp, stream)
                              : launch_wide_typed<float, uint16_t>(plan, hp, src, lds_, dst, ldd, nrows, ncols, vp, stream);
  return dt_dst == HARP_F32 ? launch_wide_typed<uint16_t, float>(plan, hp, src, lds_, dst, ldd, nrows, ncols, vp, stream)
                            : launch_wide_typed<uint16_t, uint16_t>(plan, hp, src, lds_, dst, ldd, nrows, ncols, vp, stream);
}

}  // namespace harp
