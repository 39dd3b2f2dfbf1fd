// Gradient path, two passes of up to eight coordinates in one launch.  A pass is one stage of radix 2 .. 8, or
// a run of up to three radix-2 stages taken as one block of 2, 4 or 8 coordinates whose values are the products
// of the stages' own (one path leads from a coordinate to another, so a product has no sums).  Pass a, eight
// coordinates, is followed by pass b; P = 8 B coordinates base + e S belong together.  Per row
//     y = x K_a,   dM_b += y^T g,   g' = g K_b^T,   dM_a += x^T g',   g <- g' K_a^T,
// and only the 8 x 8 sums dM leave the chip per chunk of rows (the reduction takes a run's block gradients
// out of them).  Everything is on v_mfma_f32_4x4x1_16b_f32: sixteen 4 x 4 outer products, float32 operands and
// sums.  With a block's values as one operand and four rows as the other it is a product y = x K (the result's
// lane holds the row); with four coordinates of x and four of g of one row it is an update of dM.  So an operand of
// a block costs 16 registers and its sums 16, where a thread of its own needs 64 + 64, and the two
// passes fit one launch: before, each run of three stages was a launch forward (which stored its output) and one
// backward, all on float32 copies of the batch in device memory.  Lanes: l >> 2 is the block (one of 16), l & 3 the row
// ("row layout") or the coordinate ("coordinate layout").  A change of pass goes through LDS, in
// either layout; a change of layout inside a pass is a 4 x 4 transposition in the quad.
// Bound by the rows' way through device memory and, in a short launch, by the arrival of the first ones: 2048 x 4096 bf16
// radix 2, pair 84 MB of rows + 17 MB of sums in 29 us, first 64 coordinates 67 + 4 MB in 20 us, all four reductions 7 us (run
// by run 18 + 19 + 12 (forward) + 8, a 64 x 64 product per group and its expansion 27 + 9); whole calls, us:
// 2048 x 4096 bf16 radix 2 102 -> 66; 4096 x 4096 radix 8 212 -> 121; 2048 x 8192 float32 radix 8 294 -> 223;
// 1170 x 14336 bf16 (8, 8, 8, 7, 4) 300 -> 220; 64 rows of 2048 .. 28672 1.06 - 1.66 times as fast.  The results are as far from
// the float64 ones as before or closer (333 rows, float32: dK 1.2 - 1.9e-7, dX 0.93 - 1.5e-7 of the norm).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "harp_internal.h"
#include "harp_mfma4.h"

namespace harp {
namespace {

__device__ __forceinline__ float pair_widen(float v) { return v; }
__device__ __forceinline__ float pair_widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ uint32_t pair_bf16(float f) {   // round to nearest even, NaN kept quiet
  const uint32_t u = __float_as_uint(f);
  const uint32_t rounded = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  return ((u & 0x7fffffffu) > 0x7f800000u) ? ((u >> 16) | 0x40u) : rounded;
}

template <int CTRL>
__device__ __forceinline__ float quad_move(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
// v[i] of lane j of a quad <-> v[j] of lane i
__device__ __forceinline__ void quad_transpose(float (&v)[4], bool odd, bool high) {
#pragma unroll
  for (int a = 0; a < 4; a += 2) {
    const float up = quad_move<0xB1>(v[a + 1]), down = quad_move<0xB1>(v[a]);
    v[a] = odd ? up : v[a];
    v[a + 1] = odd ? v[a + 1] : down;
  }
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const float up = quad_move<0x4E>(v[a + 2]), down = quad_move<0x4E>(v[a]);
    v[a] = high ? up : v[a];
    v[a + 2] = high ? v[a + 2] : down;
  }
}

// Operands of a pass's products, lane's output 4 h + i (i = lane & 3), input k: K[k][4 h + i] of y = v K and K[4 h + i][k]
// of y = v K^T.  `load` requests the block at (hi, lo) of a pass with stride s, `forward` and `backward` make the operands
// of it; what the two requests of a kernel bring is in flight together.  (With one load per product
// of a run, 48 to an operand, under a branch each, a launch took 25 us longer.)  Outputs past
// the block repeat its last one and are not used.
template <int B>
struct PassOperand {
  static constexpr int NH = (B + 3) / 4;
  static constexpr bool CAN_RUN = B == 2 || B == 4 || B == 8;
  static constexpr int NST = B == 8 ? 3 : (B == 4 ? 2 : 1), H = B / 2;
  float4 q[CAN_RUN ? NST : 1][CAN_RUN ? H : 1];   // a run: block of pair p of stage i, (00, 01, 10, 11)
  float v[NH][B];                                 // one stage: rows 4 h + i
  __device__ __forceinline__ void load(const PassBlocks &pb, int hi, int lo, int s, int i) {
    if (CAN_RUN && pb.nst > 0) {
      // pair p of any stage of the run (its bit taken out of the coordinate) is block c0 + p s of the stage
      const size_t c0 = (size_t)hi * H * s + lo;
#pragma unroll
      for (int t = 0; t < NST; ++t)
#pragma unroll
        for (int p = 0; p < H; ++p)
          q[t][p] = *reinterpret_cast<const float4 *>(pb.blocks[t] + (c0 + (size_t)p * s) * 4);
    } else {
      const float *b = pb.blocks[0] + ((size_t)hi * s + lo) * (B * B);
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const int o = 4 * h + i < B ? 4 * h + i : B - 1;
        if constexpr (B % 4 == 0) {
#pragma unroll
          for (int k = 0; k < B; k += 4) {
            const float4 f = *reinterpret_cast<const float4 *>(b + o * B + k);
            v[h][k] = f.x; v[h][k + 1] = f.y; v[h][k + 2] = f.z; v[h][k + 3] = f.w;
          }
        } else {
#pragma unroll
          for (int k = 0; k < B; ++k) v[h][k] = b[o * B + k];
        }
      }
    }
  }
  __device__ __forceinline__ float at(int t, int p, int k, int m) const {
    const float4 f = q[t][p];
    return k ? (m ? f.w : f.z) : (m ? f.y : f.x);
  }
  // x y z with the first product's rounding error carried along: rounded once (twice left dX of radix 2 plans 15 %
  // further from the exact one)
  static __device__ __forceinline__ float product(float x, float y, float z) {
    const float p = x * y;
    return fmaf(p, z, fmaf(x, y, -p) * z);
  }
  static __device__ __forceinline__ float pick(bool c, float a, float b) { return c ? a : b; }   // (both are there)
  // bits of a coordinate, lowest first; stage t's pair is made of the other bits, of the output below t and of the input above
  __device__ __forceinline__ void forward(const PassBlocks &pb, bool odd, bool high, float (&f)[NH][B]) const {
    if (CAN_RUN && pb.nst > 0) {
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int k = 0; k < B; ++k) {
          const int k0 = k & 1, k1 = (k >> 1) & 1, k2 = k >> 2;
          const int p0 = B == 2 ? 0 : k1 + 2 * k2;
          const float x = pick(odd, at(0, p0, k0, 1), at(0, p0, k0, 0));
          if constexpr (B == 2) {
            f[h][k] = x;
          } else {
            const float y = pick(high, pick(odd, at(1, 1 + 2 * k2, k1, 1), at(1, 2 * k2, k1, 1)),
                                 pick(odd, at(1, 1 + 2 * k2, k1, 0), at(1, 2 * k2, k1, 0)));
            if constexpr (B == 4) f[h][k] = x * y;
            else
              f[h][k] = product(x, y, pick(high, pick(odd, at(2, 3, k2, h), at(2, 2, k2, h)),
                                           pick(odd, at(2, 1, k2, h), at(2, 0, k2, h))));
          }
        }
    } else if constexpr (B % 4 == 0) {   // the rows, transposed four by four
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int g = 0; g < NH; ++g) {
          float u[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) u[k] = v[g][4 * h + k];
          quad_transpose(u, odd, high);
#pragma unroll
          for (int k = 0; k < 4; ++k) f[h][4 * g + k] = u[k];
        }
    } else {
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int g = 0; g < NH; ++g) {
          float u[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) u[k] = v[g][4 * h + k < B ? 4 * h + k : B - 1];
          quad_transpose(u, odd, high);
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (4 * g + k < B) f[h][4 * g + k] = u[k];
        }
    }
  }
  __device__ __forceinline__ void backward(const PassBlocks &pb, bool odd, bool high, float (&f)[NH][B]) const {
    if (CAN_RUN && pb.nst > 0) {
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int m = 0; m < B; ++m) {
          const int m0 = m & 1, m1 = (m >> 1) & 1, m2 = m >> 2;
          if constexpr (B == 2) {
            f[h][m] = pick(odd, at(0, 0, 1, m0), at(0, 0, 0, m0));
          } else {
            const float x = pick(high, pick(odd, at(0, 1 + 2 * h, 1, m0), at(0, 1 + 2 * h, 0, m0)),
                                 pick(odd, at(0, 2 * h, 1, m0), at(0, 2 * h, 0, m0)));
            const float y = pick(high, at(1, m0 + 2 * h, 1, m1), at(1, m0 + 2 * h, 0, m1));
            if constexpr (B == 4) f[h][m] = x * y;
            else f[h][m] = product(x, y, at(2, m0 + 2 * m1, h, m2));
          }
        }
    } else {
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int k = 0; k < B; ++k) f[h][k] = v[h][k];
    }
  }
};
// y = v K (or v K^T).  Inputs above the fourth have sums of their own, added at the end: sums of four and one of two,
// instead of one of eight, are closer to the exact ones, and twice as many products are independent.
template <int B>
__device__ __forceinline__ void pass_multiply(const float (&f)[(B + 3) / 4][B], const float *v, f4v (&y)[(B + 3) / 4]) {
  constexpr int NH = (B + 3) / 4;
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    f4v u[NH];
#pragma unroll
    for (int p = 0; p < NH; ++p) u[p] = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int p = 0; p < NH; ++p) {
        const int in = 4 * p + k < B ? 4 * p + k : 0;
        if (4 * p + k < B) u[p] = __builtin_amdgcn_mfma_f32_4x4x1f32(f[h][in], v[in], u[p], 0, 0, 0);
      }
    y[h] = u[0];
    if constexpr (NH > 1) y[h] += u[1];
  }
}
// dM[4 a + i][4 b + j] += x[row][4 a + i] g[row][4 b + j], four rows; both in coordinate layout
template <int NH>
__device__ __forceinline__ void pass_sums(const float (&x)[NH][4], const float (&g)[NH][4], f4v (&acc)[NH][NH]) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int a = 0; a < NH; ++a)
#pragma unroll
      for (int b = 0; b < NH; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[a][r], g[b][r], acc[a][b], 0, 0, 0);
}
// Sums of a few rows are made from zero and then added to those of the chunk: one sum over all of the chunk's rows (up to
// 64) left dK of 333 rows 5 - 28 % further from the exact one than sums of eight do.  Eight rows are two sets of
// four; four are summed in pass a where a step has one set for each wave (second passes of two, and of eight with float32
// gradient rows) and in pass b of the latter.
template <int NH>
__device__ __forceinline__ void sums_clear(f4v (&acc)[NH][NH]) {
#pragma unroll
  for (int a = 0; a < NH; ++a)
#pragma unroll
    for (int b = 0; b < NH; ++b) acc[a][b] = (f4v){0.f, 0.f, 0.f, 0.f};
}
template <int NH>
__device__ __forceinline__ void sums_add(f4v (&to)[NH][NH], const f4v (&from)[NH][NH]) {
#pragma unroll
  for (int a = 0; a < NH; ++a)
#pragma unroll
    for (int b = 0; b < NH; ++b) to[a][b] += from[a][b];
}

// Byte offset from a scalar row address: 32 bits for rows of fewer than 2^25 elements, a few rows at a time.
template <typename T, typename I>
__device__ __forceinline__ T pair_at(const T *p, I i) {
  return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + i * (I)sizeof(T));
}

constexpr int kPairWaves = 8;
// Sets of four rows that give each of eight waves one of pass a's B pieces of work per set, and how many times that
// a step takes (two: the barriers and the way through LDS are waited for half as often).
constexpr int pair_sets(int B) { return B == 2 ? 4 : (B <= 4 ? 2 : 1); }
// (Eight and eight coordinates of float32 gradient rows: 259 registers of 256 with two.)
constexpr int pair_times(int B, int bytes) { return B == 2 || (B == 8 && bytes == 4) ? 1 : 2; }
constexpr int pair_room(int B, int sets) { return 32 * ((B + 3) / 4) * 64 * sets; }   // floats of one exchange

// The passes at strides S (a multiple of 16) and 8 S.  A workgroup owns 16 neighbouring groups of P
// coordinates (runs of 64 bytes of a float32 row) and a chunk of rows; block l >> 2 of a wave is the group.  In pass a wave
// w works on the eight coordinates from 8 (w mod B) S on, of sets w / B, w / B + 8 / B ..; in pass b on coordinates
// w S + 8 S i, i < B, of every set.  What a wave hands over lies in LDS as [coordinate][set][group][row], the row's place
// exchanged by the coordinate's low bits so that both layouts read without conflicts.  Gout may be Gin: all
// of a step's rows have arrived, in every wave, before its second barrier, and are written behind it.
// I: of the offsets of gradient rows.
template <int B, typename TG, typename I = uint32_t>
__global__ __launch_bounds__(64 * kPairWaves, 2) void harp_grad_pair_bwd_kernel(
    const float *__restrict__ X, const TG *Gin, int64_t ldg, float *Gout, int64_t d, int64_t n, int rows,
    PassBlocks pa, PassBlocks pb, int S, int tiles, int share, float *__restrict__ partial_a,
    float *__restrict__ partial_b) {
  constexpr int N1 = pair_sets(B), NA = pair_times(B, sizeof(TG)), NS = N1 * NA, NH = (B + 3) / 4, PITCH = 64 * NS;
  constexpr int ROOM = pair_room(B, NS);
  __shared__ float lds[2 * ROOM];
  float *lx = lds, *lg = lds + ROOM;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) & 7, l = (int)threadIdx.x & 63;
  const int grp = l >> 2, q = l & 3;
  const bool odd = q & 1, high = q & 2;
  unsigned wg = blockIdx.x;
  if (share > 1) {   // tiles that share lines go to one XCD
    const unsigned xcd = wg & 7u, k = wg >> 3;
    wg = ((k / share) * 8u + xcd) * share + k % share;
  }
  const int tile = (int)(wg % (unsigned)tiles), chunk = (int)(wg / (unsigned)tiles);
  const int q0 = tile * 16, hi = q0 / S, lo = q0 % S + grp;
  const int item = w % B, set = w / B;
  const bool work_a = 8 % B == 0 || set < N1;
  const int64_t r0 = (int64_t)chunk * rows, r1 = r0 + rows < n ? r0 + rows : n;
  const int at = hi * 8 * B * S + lo, at_a = at + 8 * item * S, at_b = at + w * S;

  float nx[NA][8];
  TG ng[NS][B];
  auto fetch = [&](int64_t first) {   // rows past the end repeat the last one
    const int64_t r = first < r1 ? first : r1 - 1;
    const int last = (int)(r1 - 1 - r);
    const float *xr = X + r * d;
    const TG *gr = Gin + r * ldg;
    if (work_a) {
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        const int row = 4 * (set + N1 * j) + q < last ? 4 * (set + N1 * j) + q : last;
        const uint32_t o = (uint32_t)row * (uint32_t)d + (uint32_t)at_a;
#pragma unroll
        for (int e = 0; e < 8; ++e) nx[j][e] = pair_at(xr + e * S, o);
      }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int row = 4 * s + q < last ? 4 * s + q : last;
      const I o = (I)row * (I)ldg + (I)at_b;
#pragma unroll
      for (int i = 0; i < B; ++i) ng[s][i] = pair_at(gr + 8 * i * S, o);
    }
  };
  PassOperand<8> oa;
  PassOperand<B> ob;
  oa.load(pa, hi * B + item, lo, S, q);
  ob.load(pb, hi, lo + w * S, 8 * S, q);
  fetch(r0);
  float fa[2][8], fat[2][8], fbt[NH][B];
  oa.forward(pa, odd, high, fa);
  __builtin_amdgcn_sched_barrier(0);
  oa.backward(pa, odd, high, fat);
  __builtin_amdgcn_sched_barrier(0);
  ob.backward(pb, odd, high, fbt);
  f4v acc_a[2][2], acc_b[NH][NH];
  sums_clear<2>(acc_a);
  sums_clear<NH>(acc_b);
  int place[4];   // of row r (or coordinate 4 h + r) beside the lane's own
#pragma unroll
  for (int r = 0; r < 4; ++r) place[r] = 4 * grp + (r ^ q);
  const int own_a = 4 * grp + (q ^ (item & 3)), own_b = 4 * grp + (q ^ (w & 3));
  const float *px = lx + (w + 8 * q) * PITCH, *pg = lg + (8 * item + q) * PITCH + 64 * set;

  for (int64_t r = r0; r < r1; r += 4 * NS) {
    float x[NA][8], g[NS][B];
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) x[j][e] = work_a ? nx[j][e] : 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int i = 0; i < B; ++i) g[s][i] = pair_widen(ng[s][i]);
    fetch(r + 4 * NS);
    if (r + 4 * NS > r1) {   // rows past the end enter as zeros
#pragma unroll
      for (int j = 0; j < NA; ++j)
        if (r + 4 * (set + N1 * j) + q >= r1) {
#pragma unroll
          for (int e = 0; e < 8; ++e) x[j][e] = 0.f;
        }
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (r + 4 * s + q >= r1) {
#pragma unroll
          for (int i = 0; i < B; ++i) g[s][i] = 0.f;
        }
    }
    if (work_a) {
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        f4v y[2];
        pass_multiply<8>(fa, x[j], y);
#pragma unroll
        for (int m = 0; m < 8; ++m) lx[(8 * item + m) * PITCH + 64 * (set + N1 * j) + own_a] = y[m / 4][m % 4];
      }
    }
    lds_barrier();
    f4v few_b[NH][NH];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float xt[NH][4], gt[NH][4];
      if (s % 2 == 0) sums_clear<NH>(few_b);
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          xt[h][c] = px[32 * h * PITCH + 64 * s + place[c]];   // (coordinates past the block: whatever lies there)
          gt[h][c] = 4 * h + c < B ? g[s][4 * h + c < B ? 4 * h + c : 0] : 0.f;
        }
      f4v z[NH];
      pass_multiply<B>(fbt, g[s], z);
#pragma unroll
      for (int h = 0; h < NH; ++h) quad_transpose(gt[h], odd, high);
      pass_sums<NH>(xt, gt, few_b);
      if (s % 2 == 1 || s == NS - 1) sums_add<NH>(acc_b, few_b);
#pragma unroll
      for (int i = 0; i < B; ++i) lg[(w + 8 * i) * PITCH + 64 * s + own_b] = z[i / 4][i % 4];
      __builtin_amdgcn_sched_barrier(0);   // (sets side by side need more registers than there are)
    }
    lds_barrier();
    if (work_a) {
      f4v few_a[2][2];
      sums_clear<2>(few_a);
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        const int s64 = 64 * N1 * j;
        float xt[2][4], gt[2][4], ga[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          ga[e] = lg[(8 * item + e) * PITCH + 64 * set + s64 + place[e & 3]];
          gt[e / 4][e % 4] = pg[(e / 4) * 4 * PITCH + s64 + place[e & 3]];
          xt[e / 4][e % 4] = x[j][e];
        }
        quad_transpose(xt[0], odd, high);
        quad_transpose(xt[1], odd, high);
        f4v z[2];
        pass_multiply<8>(fat, ga, z);
        pass_sums<2>(xt, gt, few_a);
        const int64_t row = r + 4 * (set + N1 * j) + q;
        if (row < r1) {
          float *o = Gout + row * d + at_a;
#pragma unroll
          for (int e = 0; e < 8; ++e) o[(size_t)e * S] = z[e / 4][e % 4];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      sums_add<2>(acc_a, few_a);
    }
  }
  // the sums of a chunk: [sixteen blocks][value][block]
  const int lo16 = (q0 % S) / 16, S16 = S / 16;
  float *sums_a = partial_a + ((size_t)chunk * (d / 128) + (hi * B + item) * S16 + lo16) * (64 * 16);
  float *sums_b = partial_b + ((size_t)chunk * (d / (16 * B)) + (hi * 8 + w) * S16 + lo16) * (B * B * 16);
#pragma unroll
  for (int a = 0; a < NH; ++a)
#pragma unroll
    for (int b = 0; b < NH; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * a + i < B && 4 * b + q < B)
          sums_b[((4 * a + i) * B + 4 * b + q) * 16 + grp] = acc_b[a][b][i];
  if constexpr (N1 > 1) {   // pass a: the sums of the waves with the same coordinates, in the order of their first sets
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 16; ++v) lds[(w * 16 + v) * 64 + l] = acc_a[v / 8][(v / 4) & 1][v & 3];
    __syncthreads();
#pragma unroll
    for (int s = 1; s < N1; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc_a[v / 8][(v / 4) & 1][v & 3] += lds[((item + s * B) * 16 + v) * 64 + l];
  }
  if (set == 0) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          sums_a[((4 * a + i) * 8 + 4 * b + q) * 16 + grp] = acc_a[a][b][i];
  }
}

// y = x K_a K_b: the forward half, for plans with stages behind pass b.
template <int B>
__global__ __launch_bounds__(64 * kPairWaves, 2) void harp_grad_pair_fwd_kernel(
    const float *__restrict__ X, float *__restrict__ Y, int64_t d, int64_t n, int rows, PassBlocks pa, PassBlocks pb,
    int S, int tiles, int share) {
  constexpr int NS = pair_sets(B), NH = (B + 3) / 4, PITCH = 64 * NS, ROOM = pair_room(B, NS);
  __shared__ float lds[2 * ROOM];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) & 7, l = (int)threadIdx.x & 63;
  const int grp = l >> 2, q = l & 3;
  unsigned wg = blockIdx.x;
  if (share > 1) {
    const unsigned xcd = wg & 7u, k = wg >> 3;
    wg = ((k / share) * 8u + xcd) * share + k % share;
  }
  const int tile = (int)(wg % (unsigned)tiles), chunk = (int)(wg / (unsigned)tiles);
  const int q0 = tile * 16, hi = q0 / S, lo = q0 % S + grp;
  const int item = w % B, set = w / B;
  const bool work_a = 8 % B == 0 || set < NS;
  const int64_t r0 = (int64_t)chunk * rows, r1 = r0 + rows < n ? r0 + rows : n;
  const int at = hi * 8 * B * S + lo, at_a = at + 8 * item * S, at_b = at + w * S;
  float nx[2][8];
  auto fetch = [&](int64_t r, float (&v)[8]) {   // rows past the end repeat the last one and are not stored
    if (!work_a) return;
    const int64_t row = r + 4 * set + q < r1 ? r + 4 * set + q : r1 - 1;
    const float *xr = X + r0 * d;
    const uint32_t o = (uint32_t)(row - r0) * (uint32_t)d + (uint32_t)at_a;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = pair_at(xr + e * S, o);
  };
  fetch(r0, nx[0]);
  fetch(r0 + 4 * NS, nx[1]);
  PassOperand<8> oa;
  PassOperand<B> ob;
  oa.load(pa, hi * B + item, lo, S, q);
  ob.load(pb, hi, lo + w * S, 8 * S, q);
  float fa[2][8], fb[NH][B];
  oa.forward(pa, q & 1, q & 2, fa);
  ob.forward(pb, q & 1, q & 2, fb);
  const int own = 4 * grp + q;
  auto step = [&](int64_t r, float (&v)[8], float *lx) {
    f4v y[2];
    if (work_a) {
      pass_multiply<8>(fa, v, y);
#pragma unroll
      for (int m = 0; m < 8; ++m) lx[(8 * item + m) * PITCH + 64 * set + own] = y[m / 4][m % 4];
    }
    fetch(r + 8 * NS, v);
    lds_barrier();   // (the other half of the room is written next: one barrier a step)
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      float u[B];
      f4v z[NH];
#pragma unroll
      for (int i = 0; i < B; ++i) u[i] = lx[(w + 8 * i) * PITCH + 64 * s + own];
      pass_multiply<B>(fb, u, z);
      const int64_t row = r + 4 * s + q;
      if (row < r1) {
        float *o = Y + row * d + at_b;
#pragma unroll
        for (int i = 0; i < B; ++i) o[(size_t)(8 * i) * S] = z[i / 4][i % 4];
      }
    }
  };
  for (int64_t r = r0; r < r1; r += 8 * NS) {
    step(r, nx[0], lds);
    step(r + 4 * NS, nx[1], lds + ROOM);   // past the end: nothing is stored
  }
}

// The passes at strides 1 and 8, the first 64 coordinates of a plan: x are the caller's rows and so is what is
// passed back (diag(signs) is in the blocks).  A wave owns two neighbouring groups of 64 coordinates and a run of rows: block
// l >> 2 is (group, coordinates 8 item ..), so nothing crosses waves before the sums at the end and there is no
// barrier in the loop.  VEC: 16-byte accesses, else one per element, for rows that are not on such boundaries;
// the same values go through the same arithmetic.  dX may be X: a lane reads its pieces of a row before it
// writes them and no other lane touches them (the last row read again past the end is replaced by zeros).
template <typename T, bool VEC> struct LeadRaw;   // eight consecutive coordinates as loaded
template <> struct LeadRaw<float, true> {
  float4 a, b;
  __device__ __forceinline__ void load(const float *p) {
    a = *reinterpret_cast<const float4 *>(p);
    b = *reinterpret_cast<const float4 *>(p + 4);
  }
  __device__ __forceinline__ void widen(float (&x)[8]) const {
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  }
};
template <> struct LeadRaw<uint16_t, true> {
  uint4 v;
  __device__ __forceinline__ void load(const uint16_t *p) { v = *reinterpret_cast<const uint4 *>(p); }
  __device__ __forceinline__ void widen(float (&x)[8]) const {
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(u[i] << 16);
      x[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
    }
  }
};
template <typename T> struct LeadRaw<T, false> {
  T v[8];
  __device__ __forceinline__ void load(const T *p) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = p[i];
  }
  __device__ __forceinline__ void widen(float (&x)[8]) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = pair_widen(v[i]);
  }
};
template <bool VEC>
__device__ __forceinline__ void lead_store(float *p, const f4v (&v)[2]) {
  if constexpr (VEC) {
    *reinterpret_cast<f4v *>(p) = v[0];
    *reinterpret_cast<f4v *>(p + 4) = v[1];
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = v[i / 4][i % 4];
  }
}
template <bool VEC>
__device__ __forceinline__ void lead_store(uint16_t *p, const f4v (&v)[2]) {
  if constexpr (VEC) {
    *reinterpret_cast<uint4 *>(p) =
        make_uint4(pair_bf16(v[0][0]) | (pair_bf16(v[0][1]) << 16), pair_bf16(v[0][2]) | (pair_bf16(v[0][3]) << 16),
                   pair_bf16(v[1][0]) | (pair_bf16(v[1][1]) << 16), pair_bf16(v[1][2]) | (pair_bf16(v[1][3]) << 16));
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = (uint16_t)pair_bf16(v[i / 4][i % 4]);
  }
}

constexpr int kLeadWaves = 4;
constexpr int kLeadPitch = 72;   // of a row of 64 in LDS: rows, coordinates 8 apart and their quads spread over the banks

template <bool VEC, typename TX>
__global__ __launch_bounds__(64 * kLeadWaves, 2) void harp_grad_lead_bwd_kernel(
    const TX *X, int64_t ldx, const float *__restrict__ G, TX *dX, int64_t lddx, int64_t d, int64_t n, int rows,
    int tiles, PassBlocks pa, PassBlocks pb, float *__restrict__ partial_a, float *__restrict__ partial_b) {
  constexpr int ROOM = 8 * kLeadPitch + 4;
  __shared__ __attribute__((aligned(16))) float lds[kLeadWaves * 32 * 64];
  static_assert(2 * ROOM <= 32 * 64, "a wave's two exchanges fit in the space of its sums");
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l = (int)threadIdx.x & 63;
  const int half = l >> 5, item = (l >> 2) & 7, q = l & 3;
  const bool odd = q & 1, high = q & 2;
  const int groups = (int)(d / 64), tile = (int)(blockIdx.x % (unsigned)tiles), chunk = (int)(blockIdx.x / (unsigned)tiles);
  const bool ok = 2 * tile + half < groups;   // (an odd number of groups: the last one twice, stored once)
  const int grp = ok ? 2 * tile + half : groups - 1;
  const int per = rows / kLeadWaves;
  const int64_t r0 = (int64_t)chunk * rows + (int64_t)w * per, r1 = r0 + per < n ? r0 + per : n;
  float *lx = lds + w * 2 * ROOM, *lg = lx + ROOM;
  const int at = 64 * grp + 8 * item;
  f4v acc_a[2][2], acc_b[2][2];
  sums_clear<2>(acc_a);
  sums_clear<2>(acc_b);
  if (r0 < r1) {
    LeadRaw<TX, VEC> nx[2];
    LeadRaw<float, true> ng[2];
    auto fetch = [&](int64_t r, LeadRaw<TX, VEC> &nx, LeadRaw<float, true> &ng) {
      const int64_t rr = r + q < r1 ? r + q : r1 - 1;
      nx.load(X + rr * ldx + at);
      ng.load(G + rr * d + at);
    };
    fetch(r0, nx[0], ng[0]);
    PassOperand<8> oa, ob;
    oa.load(pa, grp * 8 + item, 0, 1, q);
    ob.load(pb, grp, item, 8, q);
    fetch(r0 + 4, nx[1], ng[1]);
    float fa[2][8], fat[2][8], fbt[2][8];
    oa.forward(pa, odd, high, fa);
    oa.backward(pa, odd, high, fat);
    ob.backward(pb, odd, high, fbt);
    const int slot0 = half * (4 * kLeadPitch + 4);   // the rows of a group; the second group's four banks on
    const int mine = slot0 + q * kLeadPitch + 8 * item;
    f4v few_a[2][2], few_b[2][2];
    auto step = [&](int64_t r, LeadRaw<TX, VEC> &nx, LeadRaw<float, true> &ng) {
      float x[8], g[8];
      nx.widen(x);
      ng.widen(g);
      fetch(r + 8, nx, ng);
      if (r + q >= r1) {   // rows past the end enter as zeros
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = g[e] = 0.f;
      }
      f4v y[2];
      *reinterpret_cast<float4 *>(lg + mine) = make_float4(g[0], g[1], g[2], g[3]);
      *reinterpret_cast<float4 *>(lg + mine + 4) = make_float4(g[4], g[5], g[6], g[7]);
      pass_multiply<8>(fa, x, y);
      *reinterpret_cast<f4v *>(lx + mine) = y[0];
      *reinterpret_cast<f4v *>(lx + mine + 4) = y[1];
      wave_fence();
      float xt[2][4], gt[2][4], v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xt[e / 4][e % 4] = lx[slot0 + (e % 4) * kLeadPitch + item + 8 * q + 32 * (e / 4)];
        gt[e / 4][e % 4] = lg[slot0 + (e % 4) * kLeadPitch + item + 8 * q + 32 * (e / 4)];
        v[e] = lg[slot0 + q * kLeadPitch + item + 8 * e];
      }
      wave_fence();
      f4v z[2];
      pass_multiply<8>(fbt, v, z);
      pass_sums<2>(xt, gt, few_b);
#pragma unroll
      for (int e = 0; e < 8; ++e) lg[slot0 + q * kLeadPitch + item + 8 * e] = z[e / 4][e % 4];
      wave_fence();
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        gt[e / 4][e % 4] = lg[slot0 + (e % 4) * kLeadPitch + 8 * item + q + 4 * (e / 4)];
        xt[e / 4][e % 4] = x[e];
      }
      const f4v ga0 = *reinterpret_cast<const f4v *>(lg + mine), ga1 = *reinterpret_cast<const f4v *>(lg + mine + 4);
      wave_fence();
      quad_transpose(xt[0], odd, high);
      quad_transpose(xt[1], odd, high);
      pass_sums<2>(xt, gt, few_a);
      if (dX != nullptr) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = ga0[e];
          v[4 + e] = ga1[e];
        }
        pass_multiply<8>(fat, v, z);
        if (r + q < r1 && ok) lead_store<VEC>(dX + (r + q) * lddx + at, z);
      }
    };
    for (int64_t r = r0; r < r1; r += 8) {
      sums_clear<2>(few_a);
      sums_clear<2>(few_b);
      step(r, nx[0], ng[0]);
      step(r + 4, nx[1], ng[1]);   // past the end: zeros, nothing is stored
      sums_add<2>(acc_a, few_a);
      sums_add<2>(acc_b, few_b);
    }
  }
  // the waves' sums in the order of the rows
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 32; ++v)
    lds[(w * 32 + v) * 64 + l] = v < 16 ? acc_a[(v / 8) & 1][(v / 4) & 1][v & 3] : acc_b[(v / 8) & 1][(v / 4) & 1][v & 3];
  __syncthreads();
  const size_t at16 = (size_t)blockIdx.x * (64 * 16);
#pragma unroll
  for (int k = 0; k < 32 / kLeadWaves; ++k) {
    const int v = w * (32 / kLeadWaves) + k;
    float s = lds[v * 64 + l];
#pragma unroll
    for (int u = 1; u < kLeadWaves; ++u) s += lds[(u * 32 + v) * 64 + l];
    const int row = 4 * ((v / 8) & 1) + (v & 3), col = 4 * ((v / 4) & 1) + q;
    (v < 16 ? partial_a : partial_b)[at16 + (row * 8 + col) * 16 + (l >> 2)] = s;   // (blocks past the last are not read)
  }
}

// dK of the stages of both passes: the chunks' sums in a fixed order (four runs of chunks, ascending in each, then the
// four in ascending order), then, for a run of radix-2 stages, each stage's blocks out of the run's sums:
//     dK_i = (K_0 .. K_{i-1})^T dM (K_{i+1} ..)^T  at stage i's pairs.
// The image holds diag(signs) K_0, so row r of dK_0 takes the sign of its coordinate.
constexpr int kRedBlocks = 16, kRedThreads = 1024, kRedPitch = 16, kRedSlices = 4;
__global__ __launch_bounds__(kRedThreads) void harp_grad_pair_reduce_kernel(GradSums pr) {
  __shared__ __attribute__((aligned(16))) float part[kRedSlices][64 * kRedPitch];
  __shared__ float K[3][4][4][kRedBlocks];
  const GradSums::Side &sd = pr.side[blockIdx.y];
  const int c0 = (int)blockIdx.x * kRedBlocks, D = sd.blocks, B = sd.B, BB = B * B;
  if (c0 >= D) return;
  const int nc = D - c0 < kRedBlocks ? D - c0 : kRedBlocks;   
  const int tid = (int)threadIdx.x, nst = sd.pb.nst, H = B / 2;
  {
    const int slice = tid / (4 * 64), e = 4 * (tid % (4 * 64));   // four values of each chunk of a slice
    const int per = (sd.nchunks + kRedSlices - 1) / kRedSlices, k0 = slice * per, k1 = k0 + per < sd.nchunks ? k0 + per : sd.nchunks;
    const size_t step = (size_t)((D + kRedBlocks - 1) / kRedBlocks) * (BB * kRedBlocks);
    const float *p = sd.partial + (size_t)blockIdx.x * (BB * kRedBlocks) + (e < BB * kRedBlocks ? e : 0);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = k0; k < k1; k += 16) {
      float4 f[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) f[u] = *reinterpret_cast<const float4 *>(p + (size_t)(k + u < k1 ? k + u : k) * step);
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (k + u < k1) {
          s.x += f[u].x; s.y += f[u].y; s.z += f[u].z; s.w += f[u].w;
        }
    }
    *reinterpret_cast<float4 *>(&part[slice][e]) = s;
  }
  // blocks of a run: a pair's four values each
  if (tid < nst * H * kRedBlocks) {
    const int cl = tid % kRedBlocks, p = tid / kRedBlocks % H, i = tid / (kRedBlocks * H), c = c0 + (cl < nc ? cl : 0);
    const float4 f = *reinterpret_cast<const float4 *>(sd.pb.blocks[i] + (size_t)((c / sd.s) * H * sd.s + c % sd.s + p * sd.s) * 4);
    K[i][p][0][cl] = f.x; K[i][p][1][cl] = f.y; K[i][p][2][cl] = f.z; K[i][p][3][cl] = f.w;
  }
  __syncthreads();
  if (tid < 64 * kRedBlocks) {
    const int at = (tid / kRedBlocks) * kRedPitch + tid % kRedBlocks;
    float s = part[0][at];
#pragma unroll
    for (int i = 1; i < kRedSlices; ++i) s += part[i][at];
    part[0][at] = s;
  }
  __syncthreads();
  auto M = [&](int k, int m, int cl) { return part[0][(k * B + m) * kRedPitch + cl]; };
  if (nst == 0) {
    for (int e = tid; e < nc * BB; e += kRedThreads) {
      const int cl = e / BB, v = e % BB, c = c0 + cl;
      float s = part[0][v * kRedPitch + cl];
      if (sd.signs) s *= (float)sd.signs[(size_t)c * B + v / B];
      sd.dK[0][(size_t)c * BB + v] = s;
    }
    return;
  }
  for (int e = tid; e < nst * H * 4 * nc; e += kRedThreads) {
    // pairs of a run at stride 1 lie one after the other, those of one at a larger stride a row of runs apart
    const int v = e & 3, r = v >> 1, r2 = v & 1, rest = e >> 2;
    const int i = rest / (H * nc), u = rest % (H * nc);
    const int p = sd.s == 1 ? u % H : u / nc, cl = sd.s == 1 ? u / H : u % nc;
    const int b0 = p & 1, b1 = p >> 1;   // the pair's two other bits, lower first
    float s = 0.f;
    if (nst == 1) {
      s = M(r, r2, cl);
    } else if (nst == 2) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
        s += i == 0 ? M(r + 2 * b0, r2 + 2 * t, cl) * K[1][r2][2 * b0 + t][cl]
                    : M(t + 2 * r, b0 + 2 * r2, cl) * K[0][r][2 * t + b0][cl];
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (i == 0)        // bits (r, b0, b1): g back through stages 2 and 1
            s += M(r + 2 * b0 + 4 * b1, r2 + 2 * t + 4 * q, cl) * (K[2][r2 + 2 * t][2 * b1 + q][cl] * K[1][r2 + 2 * b1][2 * b0 + t][cl]);
          else if (i == 1)   // bits (b0, r, b1): x through stage 0, g back through stage 2
            s += M(t + 2 * r + 4 * b1, b0 + 2 * r2 + 4 * q, cl) * (K[0][r + 2 * b1][2 * t + b0][cl] * K[2][b0 + 2 * r2][2 * b1 + q][cl]);
          else               // bits (b0, b1, r): x through stages 0 and 1
            s += M(t + 2 * q + 4 * r, b0 + 2 * b1 + 4 * r2, cl) * (K[0][q + 2 * r][2 * t + b0][cl] * K[1][b0 + 2 * r][2 * q + b1][cl]);
        }
    }
    const int c = c0 + cl, blk = (c / sd.s) * H * sd.s + c % sd.s + p * sd.s;
    if (i == 0 && sd.signs) s *= (float)sd.signs[(size_t)blk * 2 + r];
    sd.dK[i][(size_t)blk * 4 + v] = s;
  }
}

// Stages of one pass at stage t: one of radix up to 8, or as many radix-2 stages as follow, up to three.
int pass_stages(const std::vector<int32_t> &radices, int t) {
  const int m = (int)radices.size();
  if (t >= m || radices[t] > 8) return 0;
  if (radices[t] != 2) return 1;
  int k = 1;
  while (k < 3 && t + k < m && radices[t + k] == 2) ++k;
  return k;
}
int pass_size(const std::vector<int32_t> &radices, int t, int k) {
  int B = 1;
  for (int i = 0; i < k; ++i) B *= radices[t + i];
  return B;
}
int pass_stages(const harp_plan *plan, int t) { return pass_stages(plan->radices, t); }
int pass_size(const harp_plan *plan, int t, int k) { return pass_size(plan->radices, t, k); }
PassBlocks pass_blocks(const harp_plan *plan, int t, int k) {
  PassBlocks pb;
  for (int i = 0; i < 3; ++i) pb.blocks[i] = plan->col[DIR_FWD][t + std::min(i, k - 1)].blocks;
  pb.nst = plan->radices[t] == 2 ? k : 0;
  return pb;
}
int num_cu(const harp_plan *plan) { return plan->num_cu > 0 ? plan->num_cu : 256; }

// Rows of a workgroup: a multiple of `step` from `least_rows` (what the workspace is sized for) up to `most`, so that no sum runs over more rows than that before it
// meets the others.  The launch takes as many rounds as its workgroups (`tiles` across) fill the chip's `slots`, and a round
// costs its rows and about kChunkCost more (block values, first rows, sums).
constexpr int kChunkCost = 24;
int chunk_rows(int64_t n, int64_t tiles, int64_t slots, int step, int least_rows, int most) {
  int best = 0;
  int64_t least = 0;
  for (int rows = (least_rows + step - 1) / step * step; rows <= most; rows += step) {
    const int64_t rounds = (tiles * ((n + rows - 1) / rows) + slots - 1) / slots, cost = rounds * (rows + kChunkCost);
    if (best == 0 || cost <= least) {
      best = rows;
      least = cost;
    }
  }
  return best;
}
constexpr int kPairLeast = 16, kPairRows = 64, kLeadLeast = 32, kLeadRows = 128;
int64_t pair_slots(const harp_plan *plan) { return num_cu(plan); }
int64_t lead_slots(const harp_plan *plan) { return 2 * (int64_t)num_cu(plan); }

// the sums of a launch, passes of ka and kb stages from stage t on, for the reduction at the end of the call
// (callers have seen to it that there is room for two more: sums_room)
void add_sums(const harp_plan *plan, int t, int ka, int kb, const float *partial_a, const float *partial_b, int64_t chunks,
              float *const *dK, GradSums &sums) {
  for (int i = 0; i < 2; ++i) {
    const int t0 = i ? t + ka : t, k = i ? kb : ka;
    GradSums::Side &sd = sums.side[sums.nsides++];
    sd.partial = i ? partial_b : partial_a;
    sd.pb = pass_blocks(plan, t0, k);
    for (int j = 0; j < 3; ++j) sd.dK[j] = dK[t0 + std::min(j, k - 1)];
    sd.signs = t0 == 0 ? plan->dev_signs : nullptr;
    sd.B = pass_size(plan, t0, k);
    sd.s = plan->col[DIR_FWD][t0].s;
    sd.blocks = (int)(plan->d / sd.B);
    sd.nchunks = (int)chunks;
  }
}

bool sums_room(const GradSums &sums) { return sums.nsides + 2 <= kGradMostSides; }

}  // namespace

// Stages of the pair of passes that starts at stage t, or 0: eight coordinates first, then 2 .. 8, at a
// stride of 16 neighbouring groups.
int grad_pair_stages(const std::vector<int32_t> &radices, int t) {
  const int ka = pass_stages(radices, t);
  if (ka == 0 || pass_size(radices, t, ka) != 8 || pass_size(radices, 0, t) % 16 != 0) return 0;
  const int kb = pass_stages(radices, t + ka);
  return kb == 0 ? 0 : ka + kb;
}

// (at least as many chunks as chunk_rows makes, and never fewer for more rows)
size_t grad_pair_partial_bytes(const harp_plan *plan, int t, int64_t n) {
  const int ka = pass_stages(plan, t), B = pass_size(plan, t + ka, pass_stages(plan, t + ka));
  return (size_t)((n + kPairLeast - 1) / kPairLeast) * (size_t)plan->d * (8 + B) * 4;
}
size_t grad_lead_partial_bytes(const harp_plan *plan, int64_t n) {
  return (size_t)((n + kLeadLeast - 1) / kLeadLeast) * (size_t)((plan->d + 127) / 128) * 2 * 1024 * 4;
}

#define HARP_PAIR_SIZE(B, CALL) \
  switch (B) {                  \
    case 2: CALL(2); break;     \
    case 3: CALL(3); break;     \
    case 4: CALL(4); break;     \
    case 5: CALL(5); break;     \
    case 6: CALL(6); break;     \
    case 7: CALL(7); break;     \
    default: CALL(8); break;    \
  }

// Tiles side by side that share a line of 128 bytes of the rows with the smaller elements.
static int pair_share(int64_t tiles, int64_t total, bool bf) {
  const int s = bf ? 4 : 2;
  return tiles % s == 0 && total % (8 * s) == 0 ? s : 1;
}

harp_status_t launch_grad_pair_fwd(const harp_plan *plan, int t, const float *X, float *Y, int64_t n, hipStream_t st) {
  const int ka = pass_stages(plan, t), kb = pass_stages(plan, t + ka), B = pass_size(plan, t + ka, kb);
  const int64_t d = plan->d, tiles = d / (128 * B);
  const int rows = chunk_rows(n, tiles, pair_slots(plan), 4 * pair_sets(B), kPairLeast, kPairRows);
  const int64_t total = tiles * ((n + rows - 1) / rows);
  const PassBlocks pa = pass_blocks(plan, t, ka), pb = pass_blocks(plan, t + ka, kb);
  const int S = (int)plan->strides[t], share = pair_share(tiles, total, false);
#define HARP_PAIR_FWD(BB)                                                                                        \
  hipLaunchKernelGGL((harp_grad_pair_fwd_kernel<BB>), dim3((unsigned)total), dim3(64 * kPairWaves), 0, st, X, Y, d, \
                     n, rows, pa, pb, S, (int)tiles, share)
  HARP_PAIR_SIZE(B, HARP_PAIR_FWD)
#undef HARP_PAIR_FWD
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

// Gradient rows further apart than 32-bit offsets reach are copied to float32 first, but for bf16 rows of eight and eight
// coordinates, whose sums float32 rows would not give (fewer rows a step): their kernel exists with 64-bit offsets, too.
constexpr int64_t kPairPitch = (int64_t)1 << 25;
bool grad_pair_reads(const harp_plan *plan, int t, int64_t ldg, bool bf) {
  const int ka = pass_stages(plan, t), kb = pass_stages(plan, t + ka);
  return ldg < kPairPitch || (bf && pass_size(plan, t + ka, kb) == 8);
}

harp_status_t launch_grad_pair_bwd(const harp_plan *plan, int t, const float *X, const void *G, int64_t ldg, bool bf,
                                   float *Gout, int64_t n, float *partial, float *const *dK, GradSums &sums,
                                   hipStream_t st) {
  if (!sums_room(sums)) return HARP_ERR_UNSUPPORTED;
  const int ka = pass_stages(plan, t), kb = pass_stages(plan, t + ka), B = pass_size(plan, t + ka, kb);
  const int64_t d = plan->d, tiles = d / (128 * B);
  const int rows = chunk_rows(n, tiles, pair_slots(plan), 4 * pair_sets(B) * pair_times(B, bf ? 2 : 4), kPairLeast, kPairRows);
  const int64_t chunks = (n + rows - 1) / rows, total = tiles * chunks;
  const PassBlocks pa = pass_blocks(plan, t, ka), pb = pass_blocks(plan, t + ka, kb);
  const int S = (int)plan->strides[t], share = pair_share(tiles, total, bf);
  const int64_t tiles16 = d / 128;
  float *partial_b = partial + (size_t)chunks * (size_t)tiles16 * 1024;
#define HARP_PAIR_BWD_T(BB, T, I)                                                                                \
  hipLaunchKernelGGL((harp_grad_pair_bwd_kernel<BB, T, I>), dim3((unsigned)total), dim3(64 * kPairWaves), 0, st, X, \
                     (const T *)G, ldg, Gout, d, n, rows, pa, pb, S, (int)tiles, share, partial, partial_b)
#define HARP_PAIR_BWD(BB)                          \
  if (bf) HARP_PAIR_BWD_T(BB, uint16_t, uint32_t); \
  else HARP_PAIR_BWD_T(BB, float, uint32_t)
  if (ldg >= kPairPitch) HARP_PAIR_BWD_T(8, uint16_t, uint64_t);
  else HARP_PAIR_SIZE(B, HARP_PAIR_BWD)
#undef HARP_PAIR_BWD
#undef HARP_PAIR_BWD_T
  add_sums(plan, t, ka, kb, partial, partial_b, chunks, dK, sums);
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

// X and dX are the caller's: one access per element where rows do not lie on boundaries of 16 bytes.
static bool lead_vec(const void *p, int64_t ld, bool bf) { return ld % (bf ? 8 : 4) == 0 && (uintptr_t)p % 16 == 0; }

harp_status_t launch_grad_lead_bwd(const harp_plan *plan, int nst, const void *X, int64_t ldx, bool bf, const float *G,
                                   void *dX, int64_t lddx, int64_t n, float *partial, float *const *dK, GradSums &sums,
                                   hipStream_t st) {
  if (!sums_room(sums)) return HARP_ERR_UNSUPPORTED;
  const int64_t d = plan->d, tiles = (d + 127) / 128;
  const int rows = chunk_rows(n, tiles, lead_slots(plan), 4 * kLeadWaves, kLeadLeast, kLeadRows);
  const int64_t chunks = (n + rows - 1) / rows;
  const dim3 grid((unsigned)(tiles * chunks));
  const PassBlocks pa = pass_blocks(plan, 0, nst / 2), pb = pass_blocks(plan, nst / 2, nst / 2);
  const bool vec = lead_vec(X, ldx, bf) && (!dX || lead_vec(dX, lddx, bf));
  const int64_t tiles16 = tiles;
  float *partial_b = partial + (size_t)chunks * (size_t)tiles16 * 1024;
#define HARP_LEAD_BWD(VEC, T)                                                                                       \
  hipLaunchKernelGGL((harp_grad_lead_bwd_kernel<VEC, T>), grid, dim3(64 * kLeadWaves), 0, st, (const T *)X, ldx, G, \
                     (T *)dX, lddx, d, n, rows, (int)tiles, pa, pb, partial, partial_b)
  if (bf && vec) HARP_LEAD_BWD(true, uint16_t);
  else if (bf) HARP_LEAD_BWD(false, uint16_t);
  else if (vec) HARP_LEAD_BWD(true, float);
  else HARP_LEAD_BWD(false, float);
#undef HARP_LEAD_BWD
  add_sums(plan, 0, nst / 2, nst / 2, partial, partial_b, chunks, dK, sums);
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

harp_status_t launch_grad_sums(const GradSums &sums, hipStream_t st) {
  int most = 0;
  for (int i = 0; i < sums.nsides; ++i) most = std::max(most, sums.side[i].blocks);
  hipLaunchKernelGGL(harp_grad_pair_reduce_kernel, dim3((unsigned)((most + kRedBlocks - 1) / kRedBlocks), (unsigned)sums.nsides),
                     dim3(kRedThreads), 0, st, sums);
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

}  // namespace harp
