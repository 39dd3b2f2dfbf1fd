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
// Narrow matrices and the last columns beside whole tiles run here too, lanes past the end idle, on guarded LDS
// tiles before (float32, us): 4096 x 32 18.2 -> 11.7, 4096 x 130 30.4 -> 12.4, 4096 x 4100 64 -> 48, 28672 x 1000 159 -> 137.
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

// (four waves per SIMD where the tile leaves room for them; the descending forms would spill)
template <typename TI, typename TO, int R1, int R2, bool DESC>
__global__ __launch_bounds__(64, !DESC && R1 * R2 <= 28 ? 4 : 2) void harp_colpair_kernel(const TI *src, int64_t lds_, TO *dst, int64_t ldd, int S,
                                                             int ncols, unsigned nct, unsigned total,
                                                             const float *__restrict__ image) {
  using Sh = PairShape<R1, R2>;
  constexpr int P = Sh::P, RING = 8;
  const int lane = (int)threadIdx.x;
  // an XCD takes a run of neighbouring columns of the same rows
  const unsigned id = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (id >= total) return;
  const unsigned T = id / nct;
  const int64_t row0 = (int64_t)(T / (unsigned)S) * P * S + T % (unsigned)S;
  const int c0 = (int)(id % nct) * kPairCols;
  src += row0 * lds_ + c0;
  dst += row0 * ldd + c0;
  // the lane's columns behind c0 (ncols is even; lanes past the last columns repeat them and store nothing)
  const unsigned left = (unsigned)(ncols - c0), col = 2 * (unsigned)lane < left ? 2 * (unsigned)lane : left - 2;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(image + (size_t)T * Sh::TILE), 0, Sh::TILE * 4,
                                                      0x00020000);
  const BlockValues<64> val = {rsrc, (lane & 3) * 16};
  float x[2][P];
  f4v ring[RING];
#pragma unroll
  for (int j = 0; j < P; ++j) pair_load(src + (int64_t)j * S * lds_ + col, x[0][j], x[1][j]);
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
  if (2 * (unsigned)lane >= left) return;
#pragma unroll
  for (int j = 0; j < P; ++j) pair_store(dst + (int64_t)j * S * ldd + col, x[0][j], x[1][j]);
}

template <typename TI, typename TO, int R1, int R2>
harp_status_t launch_pair_inst(const ColPass &hp, const void *src, int64_t lds_, void *dst, int64_t ldd, int64_t nrows,
                               int64_t ncols, hipStream_t stream) {
  const int64_t nct = (ncols + kPairCols - 1) / kPairCols, total = (nrows / hp.P) * nct;
  if (total <= 0) return HARP_OK;
  if (total > 0x7ffffff0 || ncols > 0x7fffff00) return HARP_ERR_UNSUPPORTED;
  const dim3 grid((unsigned)((total + 7) / 8 * 8));
  if (hp.desc)
    hipLaunchKernelGGL((harp_colpair_kernel<TI, TO, R1, R2, true>), grid, dim3(64), 0, stream, (const TI *)src, lds_,
                       (TO *)dst, ldd, (int)hp.S, (int)ncols, (unsigned)nct, (unsigned)total, hp.packed);
  else
    hipLaunchKernelGGL((harp_colpair_kernel<TI, TO, R1, R2, false>), grid, dim3(64), 0, stream, (const TI *)src, lds_,
                       (TO *)dst, ldd, (int)hp.S, (int)ncols, (unsigned)nct, (unsigned)total, hp.packed);
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

// The pairs (radix at the lower stride, radix at the higher one) the kernel is built for: what greedy schedules of
// base 8 leave to a pass -- 8 below any last radix 3 .. 8, and 7 below 4 (14336 = 8 8 8 7 4).  Others (7 8, 6 8, 5 4)
// do not come out of those schedules and keep the LDS-tile kernel.
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

// The block values of every tile in the order of harp_colpair_kernel, one float per thread.  A group's stages
// each replace one digit of the coordinate, so entry (i, q) of its block is one product: for every stage
// the entry (its digit of i, its digit of q) of the block at the digits already replaced by q's and not
// yet replaced from i's (float64, rounded once).  On the device, where the stages' blocks are already: on the
// host the products were a sixth of the time that a plan of 4096 radix 2 takes to create.
constexpr int kPackThreads = 256;
__global__ __launch_bounds__(kPackThreads) void harp_colpair_pack_kernel(PairBlocks pb, unsigned total, float *out) {
  const unsigned idx = blockIdx.x * kPackThreads + threadIdx.x;
  if (idx >= total) return;
  const unsigned S = (unsigned)pb.S, P = (unsigned)(pb.grp[0].R * pb.grp[1].R), tile = (unsigned)(pb.words[0] + pb.words[1]);
  const unsigned T = idx / tile;
  int w = (int)(idx % tile);
  const int g = w >= pb.words[0] ? 1 : 0;
  w -= g ? pb.words[0] : 0;
  const PairBlocks::Group &G = pb.grp[g];
  const int b = G.R, per = chain_pieces(b) * 16, v = w / per, x = w % per;
  // word x of a block: piece x / 16, column x / 4 % 4 of a quad; the piece's four words are consecutive (row, half)
  const int nh = b > 4 ? 2 : 1, rh = (x >> 4) * 4 + (x & 3), i = rh / nh, q = rh % nh * 4 + (x >> 2 & 3);
  float value = 0.0f;   // padding of the last piece or of a quad
  if (i < b && q < b) {
    const unsigned row = T / S * P * S + T % S + (unsigned)(g ? v : v * pb.grp[0].R) * S;
    double f = 1.0;
    int e = i;
    for (int t = 0; t < G.n; ++t) {
      const int cb = G.b[t], step = G.step[t], di = e / step % cb, dq = q / step % cb;
      const unsigned cs = (unsigned)G.s[t], at = row + (unsigned)(e - di * step) * (unsigned)G.s0;
      f *= (double)G.blocks[t][(size_t)(at / (cb * cs) * cs + at % cs) * (unsigned)(cb * cb) + (unsigned)(di * cb + dq)];
      e += (dq - di) * step;
    }
    value = (float)f;
  }
  out[idx] = value;
}

}  // namespace

// Stages [i0, e0) of the column image, consecutive digits in ascending or descending order, as one such pass: the
// number of stages of the group at the lower strides, or 0.  A group of several stages acts as one
// dense block of the product of their radices (three radix-2 stages as a block of 8 rows).  Such a
// pass is taken for bf16 matrices only: sums of eight products round more often than three of two, and
// a float32 result of radix-2 schedules would be 1.58e-7 of its norm from the float64 one instead
// of 1.51e-7 (4096 x 2048), which a bf16 result does not show.  bf16 matrix, float32 workspace: 4096 x 11008
// radix 2 inverse 346 -> 308 us (64 rows: 90 -> 73 us in float32, 82 -> 57 us to bf16), 3072 x 11008 261 -> 225.
int col_pair_split(const std::vector<ColStage> &st, int i0, int e0) {
  const int n = e0 - i0;
  if (n < 2) return 0;
  const bool desc = st[i0].s > st[i0 + 1].s;
  auto at = [&](int k) -> const ColStage & { return st[desc ? e0 - 1 - k : i0 + k]; };   // by stride
  for (int k = 0; k + 1 < n; ++k)
    if (at(k + 1).s != at(k).s * at(k).b) return 0;
  int r1 = 1;
  for (int k = 1; k < n; ++k) {
    r1 *= at(k - 1).b;
    if (r1 > 8) return 0;
    int r2 = 1;
    for (int q = k; q < n && r2 <= 8; ++q) r2 *= at(q).b;
    if ((r1 == 7 && r2 == 4) || (r1 == 8 && r2 >= 3 && r2 <= 8)) return k;
  }
  return 0;
}

void col_pair_blocks(const std::vector<ColStage> &st, int i0, int e0, int split, ColPass &cp, PairBlocks &pb) {
  const bool desc = st[i0].s > st[i0 + 1].s;
  pb = PairBlocks();
  for (int t = i0; t < e0; ++t) {   // the two groups, stages in the order they run
    const ColStage &c = st[t];
    PairBlocks::Group &G = pb.grp[(desc ? e0 - 1 - t : t - i0) < split ? 0 : 1];
    G.s0 = G.n ? std::min(G.s0, c.s) : c.s;
    G.R = G.n ? G.R * c.b : c.b;
    G.blocks[G.n] = c.blocks;
    G.b[G.n] = c.b;
    G.s[G.n++] = c.s;
  }
  for (PairBlocks::Group &G : pb.grp)
    for (int t = 0; t < G.n; ++t) G.step[t] = G.s[t] / G.s0;
  pb.S = pb.grp[0].s0;
  for (int g = 0; g < 2; ++g) pb.words[g] = pb.grp[1 - g].R * chain_pieces(pb.grp[g].R) * 16;
  cp.desc = desc ? 1 : 0;
  cp.composite = pb.grp[0].n > 1 || pb.grp[1].n > 1 ? 1 : 0;
  cp.r1 = pb.grp[0].R;
}

size_t col_pair_floats(const PairBlocks &pb, int64_t d) {
  return (size_t)(d / (pb.grp[0].R * pb.grp[1].R)) * (size_t)(pb.words[0] + pb.words[1]);
}

harp_status_t launch_pair_pack(const PairBlocks &pb, int64_t d, float *out, hipStream_t stream) {
  const size_t total = col_pair_floats(pb, d);
  if (total > 0x7ffffff0) return HARP_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(harp_colpair_pack_kernel, dim3((unsigned)((total + kPackThreads - 1) / kPackThreads)),
                     dim3(kPackThreads), 0, stream, pb, (unsigned)total, out);
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

// an even number of columns, pairs of columns aligned (the caller's check)
harp_status_t launch_col_pair(const ColPass &hp, const void *src, int64_t lds_, harp_dtype_t dt_src, void *dst,
                              int64_t ldd, harp_dtype_t dt_dst, int64_t nrows, int64_t ncols, hipStream_t stream) {
  if (!hp.packed || hp.P == 512 || ncols % 2) return HARP_ERR_UNSUPPORTED;
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
