// Column passes of two small dense stages (radices 8 and 3..8, or 7 and 4: the 64 / 56 / 48 / 32 / 28 rows that
// radix-8 schedules leave to a pass) with the whole tile in registers.
//
// All columns of a tile share their blocks, so a wave is 64 lanes of one operand of v_mfma_f32_4x4x1_16b_f32 with
// the same block in all sixteen slots: a lane holds every row of the tile at two neighbouring columns (rows move as
// 512 contiguous bytes of float32 per wave), and the second stage follows the first by renaming registers.  No
// LDS, no barrier, one wave per workgroup: eight waves of a compute unit load, multiply and store
// independently, where the tile kernel's workgroups pass through five barriers per tile.
// Sums run over r in ascending order from zero, as in that kernel.  A tile's block values are 4 KB.
//
// Bound by bytes.  28672 x 8192, pass of 56 rows, float32 -> bf16: 405 us (3.5 TB/s) on the LDS-tile kernel ->
// 300 us (4.7 TB/s); the rotation 1148 -> 1062 us.  Whole calls, radix-8 schedules, us: 64 x 4096 float32 (plan_U
// only) 10.6 -> 7.0, 4096 x 128 15.0 -> 12.2, 2048 x 2048 bf16 55 -> 31, 4096 x 4096 bf16 118 -> 70,
// 28672 x 3072 bf16 494 -> 446 (chunks of plan_V included).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "harp_internal.h"
#include "harp_mfma4.h"

namespace harp {

namespace {

constexpr int kPairCols = 128;

template <int R1, int R2>
struct PairShape {
  static constexpr int P = R1 * R2;
  static constexpr int N1 = R2 * chain_pieces(R1), N2 = R1 * chain_pieces(R2);   // pieces of 64 bytes
  static constexpr int TILE = (N1 + N2) * 16;                                    // floats
};

__device__ __forceinline__ void pair_load(const float *p, float &a, float &b) {
  const float2 v = *reinterpret_cast<const float2 *>(p);
  a = v.x;
  b = v.y;
}
__device__ __forceinline__ void pair_load(const uint16_t *p, float &a, float &b) {
  const uint32_t v = *reinterpret_cast<const uint32_t *>(p);
  a = __uint_as_float(v << 16);
  b = __uint_as_float(v & 0xffff0000u);
}
__device__ __forceinline__ void pair_store(float *p, float a, float b) { *reinterpret_cast<float2 *>(p) = make_float2(a, b); }
__device__ __forceinline__ void pair_store(uint16_t *p, float a, float b) { *reinterpret_cast<uint32_t *>(p) = pack2(a, b); }

template <typename TI, typename TO, int R1, int R2, bool DESC>
__global__ __launch_bounds__(64, 2) void harp_colpair_kernel(const TI *src, int64_t lds_, TO *dst, int64_t ldd, int S,
                                                             unsigned nct, unsigned total,
                                                             const float *__restrict__ image) {
  using Sh = PairShape<R1, R2>;
  constexpr int P = Sh::P, RING = 8;
  const int lane = (int)threadIdx.x;
  // an XCD takes a run of neighbouring columns of the same rows
  const unsigned id = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (id >= total) return;
  const unsigned T = id / nct;
  const int64_t row0 = (int64_t)(T / (unsigned)S) * P * S + T % (unsigned)S;
  const int64_t c0 = (int64_t)(id % nct) * kPairCols;
  src += row0 * lds_ + c0;
  dst += row0 * ldd + c0;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(image + (size_t)T * Sh::TILE), 0, Sh::TILE * 4,
                                                      0x00020000);
  const BlockValues<64> val = {rsrc, (lane & 3) * 16};
  float x[2][P];
  f4v ring[RING];
#pragma unroll
  for (int j = 0; j < P; ++j) pair_load(src + (int64_t)j * S * lds_ + 2 * lane, x[0][j], x[1][j]);
  constexpr int FIRST = DESC ? Sh::N1 : 0, NF = DESC ? Sh::N2 : Sh::N1;
#pragma unroll
  for (int s = 0; s < RING; ++s)
    if (s < NF) ring[s] = val.piece(FIRST, s);
  if constexpr (!DESC) {
    chain_stage<R1, R2, R1, 1, Sh::N2>(x, ring, val, 0, Sh::N1);
    chain_stage<R2, R1, 1, R1, 0>(x, ring, val, Sh::N1, 0);
  } else {
    chain_stage<R2, R1, 1, R1, Sh::N1>(x, ring, val, Sh::N1, 0);
    chain_stage<R1, R2, R1, 1, 0>(x, ring, val, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < P; ++j) pair_store(dst + (int64_t)j * S * ldd + 2 * lane, x[0][j], x[1][j]);
}

template <typename TI, typename TO, int R1, int R2>
harp_status_t launch_pair_inst(const ColPass &hp, const void *src, int64_t lds_, void *dst, int64_t ldd, int64_t nrows,
                               int64_t ncols, hipStream_t stream) {
  const int64_t nct = ncols / kPairCols, total = (nrows / hp.P) * nct;
  if (total <= 0) return HARP_OK;
  if (total > 0x7ffffff0) return HARP_ERR_UNSUPPORTED;
  const dim3 grid((unsigned)((total + 7) / 8 * 8));
  if (hp.desc)
    hipLaunchKernelGGL((harp_colpair_kernel<TI, TO, R1, R2, true>), grid, dim3(64), 0, stream, (const TI *)src, lds_,
                       (TO *)dst, ldd, (int)hp.S, (unsigned)nct, (unsigned)total, hp.packed);
  else
    hipLaunchKernelGGL((harp_colpair_kernel<TI, TO, R1, R2, false>), grid, dim3(64), 0, stream, (const TI *)src, lds_,
                       (TO *)dst, ldd, (int)hp.S, (unsigned)nct, (unsigned)total, hp.packed);
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

// the pairs (radix at the lower stride, radix at the higher one) the kernel is built for
#define HARP_PAIR_SWITCH(r1, r2, CALL)                      \
  do {                                                      \
    if ((r1) == 7 && (r2) == 4) { CALL(7, 4); }             \
    else if ((r1) == 8) {                                   \
      switch (r2) {                                         \
        case 3: { CALL(8, 3); } break;                      \
        case 4: { CALL(8, 4); } break;                      \
        case 5: { CALL(8, 5); } break;                      \
        case 6: { CALL(8, 6); } break;                      \
        case 7: { CALL(8, 7); } break;                      \
        case 8: { CALL(8, 8); } break;                      \
        default: break;                                     \
      }                                                     \
    }                                                       \
  } while (0)

}  // namespace

// Stages i0, i0 + 1 of the column image as one such pass.
bool col_pair_stages(const std::vector<ColStage> &st, int i0) {
  const ColStage &a = st[i0], &b = st[i0 + 1];
  const ColStage &lo = a.s < b.s ? a : b, &hi = a.s < b.s ? b : a;
  if (hi.s != (int64_t)lo.s * lo.b) return false;
  return (lo.b == 7 && hi.b == 4) || (lo.b == 8 && hi.b >= 3 && hi.b <= 8);
}

void col_pair_image(const std::vector<ColStage> &st, int i0, int64_t d, const float *host_image, ColPass &cp,
                    std::vector<float> &out) {
  const bool desc = st[i0].s > st[i0 + 1].s;
  const ColStage &c1 = st[desc ? i0 + 1 : i0], &c2 = st[desc ? i0 : i0 + 1];
  cp.desc = desc ? 1 : 0;
  cp.r1 = c1.b;
  const int R1 = c1.b, R2 = c2.b, P = R1 * R2;
  const int64_t S = c1.s, tiles = d / P;
  const int n1 = R2 * chain_pieces(R1), n2 = R1 * chain_pieces(R2);
  out.assign((size_t)tiles * (n1 + n2) * 16, 0.0f);
  for (int64_t T = 0; T < tiles; ++T)
    for (int e = 0; e < 2; ++e) {
      const ColStage &cs = e ? c2 : c1;
      const int b = cs.b, nh = b > 4 ? 2 : 1, np = chain_pieces(b);
      const float *blocks = host_image + (cs.blocks - st[0].blocks);
      float *o = out.data() + (size_t)T * (n1 + n2) * 16 + (e ? n1 * 16 : 0);
      for (int v = 0; v < P / b; ++v) {
        const int64_t row = (T / S) * P * S + T % S + (int64_t)(e ? v : v * R1) * S;
        const float *K = blocks + ((row / ((int64_t)b * cs.s)) * cs.s + row % cs.s) * b * b;
        for (int r = 0; r < b; ++r)
          for (int c = 0; c < b; ++c) {
            const int w = r * nh + c / 4;
            o[((v * np + w / 4) * 4 + c % 4) * 4 + w % 4] = K[r * b + c];
          }
      }
    }
}

// whole tiles of 128 columns, pairs of columns aligned (the caller's check for every unguarded column pass)
harp_status_t launch_col_pair(const ColPass &hp, const void *src, int64_t lds_, harp_dtype_t dt_src, void *dst,
                              int64_t ldd, harp_dtype_t dt_dst, int64_t nrows, int64_t ncols, hipStream_t stream) {
  if (!hp.packed || hp.P == 512 || ncols % kPairCols) return HARP_ERR_UNSUPPORTED;
  harp_status_t st = HARP_ERR_UNSUPPORTED;
  const int r2 = hp.P / hp.r1;
#define HARP_PAIR(TI, TO, A, B) st = launch_pair_inst<TI, TO, A, B>(hp, src, lds_, dst, ldd, nrows, ncols, stream)
#define HARP_PAIR_FF(A, B) HARP_PAIR(float, float, A, B)
#define HARP_PAIR_FH(A, B) HARP_PAIR(float, uint16_t, A, B)
#define HARP_PAIR_HF(A, B) HARP_PAIR(uint16_t, float, A, B)
#define HARP_PAIR_HH(A, B) HARP_PAIR(uint16_t, uint16_t, A, B)
  if (dt_src == HARP_F32 && dt_dst == HARP_F32) HARP_PAIR_SWITCH(hp.r1, r2, HARP_PAIR_FF);
  else if (dt_src == HARP_F32) HARP_PAIR_SWITCH(hp.r1, r2, HARP_PAIR_FH);
  else if (dt_dst == HARP_F32) HARP_PAIR_SWITCH(hp.r1, r2, HARP_PAIR_HF);
  else HARP_PAIR_SWITCH(hp.r1, r2, HARP_PAIR_HH);
  return st;
}

}  // namespace harp
