// Chains of four small dense stages 8, 8, 8, R4 (R4 = 3 .. 8) on chunks of 512 R4 coordinates: the radix-8
// schedules, on the float32 matrix instruction v_mfma_f32_4x4x1_16b_f32.
//
// That instruction is sixteen independent 4 x 4 outer-product updates.  Sixteen blocks of a stage
// times four rows are one operand: lane 4 b + row holds the coordinates of block slot b and that row
// in registers, lane 4 b + i the block's values K[k][4 h + i]; after one instruction per input k and
// half h of the outputs the lane (b, row) holds the outputs -- the layout the inputs had.  A block
// of 64 values costs 16 registers per lane and is used for four rows at once, and a product runs at
// twice the rate of the vector units, with the same float32 chain of fused multiply-adds.
//
// A workgroup takes eight rows of one chunk (HV == 2), or four where there are few (HV == 1, see the
// launch).  A wave owns sixteen groups of 64 coordinates (8 R4 in the high stages) of the rows, and a
// lane holds all coordinates of its group and of HV rows (row, row + 4): two stages whose digits both
// lie inside the group follow each other by renaming registers.  A tile so makes one exchange through
// LDS, between the two low stages (groups of 64 consecutive coordinates) and the high ones (groups of
// 8 R4 coordinates 64 apart); one block per thread needed three.  The exchange takes four rows at a
// time, so that a workgroup needs half the LDS of its rows and two of them (four small ones) share a
// compute unit: one's loads, exchanges and stores run under the other's products.  Rows enter and
// leave in 16-byte pieces through the same LDS rows; bf16 rows r and r + 4 travel as the two halves
// of one word.
//
// What bounds it: the block values (0.5 MB for a chunk of 4096) come through the compute unit's load path
// of 64 bytes per clock once per tile, as long as its matrix instructions take (2300 clocks a stage).
// 2048 x 4096 bf16 (8,8,8,8), one tile per compute unit: 18.3 us on one block per thread -> 14.5 us, of
// which 1.6 us are the launch, 3 us the rows' arrival, 6 us stages, 2 us the exchange, 2 us the
// stores; 777 x 14336 transposed (8,8,8,7 | 4), both launches: 60 -> 36 us; six rows of 14336:
// 18.3 -> 12.5 us (9.9 in tiles of four rows); 28672 x 8192 bf16 -> float32: 472 -> 325 us (1.41 GB).
// One row of 4096 (float32 / bf16, replayed): 7.0 / 6.9 us on one block per thread, 9.9 / 9.8 in a tile
// of eight, 7.0 / 6.9 in one of four (rows that are not there are neither loaded nor stored, and all
// waves share a row's stores).  Touching every line of the values at the start of a launch, so that
// the first reads find them in the L2, was slower (six rows: 13.6 -> 15.5 us).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "harp_internal.h"
#include "harp_mfma4.h"

namespace harp {

namespace {

constexpr int R3 = 8;   // radix of the third stage

// Sizes of one instance; also the layout of the block values: per chunk the stages at strides 1, 8,
// 64, 64 R3 one after the other, a stage as [unit or block of 16 lo][batch][piece][lane][4].
template <int R4, int HV = 2>
struct ChainShape {
  static constexpr int H = R3 * R4;                   // groups of 64 in a chunk, coordinates of a high group
  static constexpr int CHUNK = 64 * H;
  static constexpr int UNITS = (H + 15) / 16;         // sixteen groups each; the last one may be half full
  static constexpr int NW = H > 32 ? 4 : 2;           // waves
  static constexpr int LB = 4 / NW;                   // blocks of 16 lo per wave in the high stages
  static constexpr int PITCH = CHUNK + 8;             // LDS row (floats): four rows x 8 lo hit 32 banks
  // 16-byte pieces of block values a lane holds: those in use and the next two batches.  Outputs come in
  // aligned quads while the inputs they replace are spread over other quads, so a stage of two rows per lane
  // needs up to 64 registers more than its coordinates: with a ring of 16 most shapes spilled (2048 x 4096 bf16
  // 15.3 us against 14.6, six rows of 14336 13.6 against 12.5).  Radix 4 has smaller batches: eight pieces are as
  // many ahead; its waves hold two blocks of 16 lo, and five of its seven instances still spill 7 to 35 registers, with the stage above on the way
  // in all six of them 33 to 39 (and radix 7 under a stage of radix 4 with float32 rows, 4); those are ahead of two launches all the same
  // (8, 8, 8, 4, 4 transposed, bf16, us: 300 rows 17.6 -> 14.5, 3000 rows 70 -> 63, 8000 rows 189 -> 149; float32 18.9 -> 14.2, 84 -> 83, 262 -> 199).
  // One row per lane has room: one row of 4096 bf16 7.1 us with a ring of 12, 6.9 with 16, 7.0 with 24, 7.3 with 48.
  static constexpr int RING = HV == 1 ? 16 : R4 == 4 ? 8 : 12;
  static constexpr int NA = 32;                       // pieces per unit, stages at strides 1 and 8
  static constexpr int NC = R4 * chain_pieces(R3);    // pieces per block of 16 lo
  static constexpr int ND = R3 * chain_pieces(R4);
  static constexpr int64_t OFF_B = (int64_t)UNITS * NA * 256;   // floats
  static constexpr int64_t OFF_C = 2 * OFF_B;
  static constexpr int64_t OFF_D = OFF_C + (int64_t)4 * NC * 256;
  static constexpr int64_t TOTAL = OFF_D + (int64_t)4 * ND * 256;
};

// TOP: radix of the stage above the chunk, which a transposed program runs first; 0: none, or not here.
template <typename TI, typename TO, int R4, bool TRN, int HV, int TOP = 0>
__global__ __launch_bounds__((64 * ChainShape<R4>::NW), 2) void harp_chain_kernel(
    const TI *X, int64_t ldx, TO *Y, int64_t ldy, int64_t n, int R, unsigned ntile, unsigned total,
    const float *__restrict__ image, const float *__restrict__ tparams) {
  using S = ChainShape<R4, HV>;
  constexpr int H = S::H, NW = S::NW, LB = S::LB;
  constexpr bool BI = sizeof(TI) == 2, BO = sizeof(TO) == 2;
  constexpr int NR8 = S::CHUNK / 512, NR4 = S::CHUNK / 256;   // 16-byte pieces of a row per lane: bf16, float32
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slot = lane >> 2, row = lane & 3;   // block slot and row of the operand layout
  // Workgroups go to the eight XCDs in turn; an XCD takes a run of tiles of the same chunk, so that its
  // L2 holds the block values of few chunks.
  const unsigned id = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (id >= total) return;   // the whole workgroup
  // (TOP: of the same rows, all chunks one after the other, so that the row is read from memory once; few rows are
  // less than the block values)
  constexpr bool ROWS_FIRST = TOP > 0 && HV == 2;
  const unsigned nch = ROWS_FIRST ? total / ntile : 1;
  const int kch = (int)(ROWS_FIRST ? id % nch : id / ntile);
  const int64_t r0 = (int64_t)(ROWS_FIRST ? id / nch : id % ntile) * R;
  const int nr = (int)((n - r0 < R) ? (n - r0) : R);
  const BlockValues<1024> val = {__builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(image + (int64_t)kch * S::TOTAL), 0,
                                                              (int)(S::TOTAL * 4), 0x00020000),
                           lane * 16};
  const TI *Xt = X + r0 * ldx + (TOP > 0 ? 0 : (int64_t)kch * S::CHUNK);
  TO *Yt = Y + r0 * ldy + (int64_t)kch * S::CHUNK;

  // low side: unit u, its groups and coordinates (40 and 48 groups: the fourth wave repeats the last
  // unit's work and keeps nothing of it)
  const int u = S::UNITS < NW && w >= S::UNITS ? S::UNITS - 1 : w;
  const bool low = S::UNITS == NW || w < S::UNITS;
  const int ngr = (H % 16 != 0 && u == S::UNITS - 1) ? H % 16 : 16;   // groups in the unit (8 or 16)
  const int gl = slot < ngr ? slot : ngr - 1;
  // first pieces of the wave's block values in each stage
  const int iA = u * S::NA, iB = (int)(S::OFF_B / 256) + u * S::NA;
  const int iC = (int)(S::OFF_C / 256) + w * LB * S::NC, iD = (int)(S::OFF_D / 256) + w * LB * S::ND;

  // LDS position of coordinate (group j, lo) of row r & 3: bit 2 of lo flipped in odd groups (16-byte
  // accesses of four rows x two groups then fall into different banks)
  auto pos = [](int r, int j, int lo) { return r * S::PITCH + j * 64 + (lo ^ ((j & 1) << 2)); };
  // a row's consecutive coordinates 4 c .. 4 c + 3
  auto pos4 = [](int r, int c) { return r * S::PITCH + ((c ^ ((c >> 4) & 1)) << 2); };
  // 16 bytes of a row; rows past the end are zero (a tile of four rows) or repeat the last one, and are not stored
  auto row_piece = [&](int r, int at) {
    if (HV == 1 && r >= nr) return (u4v){0u, 0u, 0u, 0u};
    return *reinterpret_cast<const u4v *>(Xt + (int64_t)(r < nr ? r : nr - 1) * ldx + at);
  };

  f4v ring[S::RING];
  auto first_pieces = [&](int p, int cnt) {
#pragma unroll
    for (int s = 0; s < S::RING; ++s)
      if (s < cnt) ring[s] = val.piece(p, s);
  };
  // a lane's 16-byte pieces 2 l and 2 l + 1 of eight words: which one goes first alternates every four
  // lanes, so that eight lanes hit all banks
  const int sw = (lane >> 2) & 1;

  // Stores.  A tile of eight: a wave writes whole rows (forward) and reads LDS for all its rows at once, stored or
  // not; a tile of four: a row's pieces go over the waves, as a lone row is not one wave's work, and rows that are
  // not there cost nothing.  Tiles of eight stored the second way: rotation of 28672 x 8192 1077 -> 1085 us.
  constexpr bool SHARE = HV == 1;

  if constexpr (!TRN) {
    float x[HV][64];
    // rows of the unit through the wave's own part of the LDS rows (bf16: rows r and r + 4 one after
    // the other), coordinates of a group side by side
    if constexpr (BI) {
      u4v raw[4 * HV][2];
#pragma unroll
      for (int r = 0; r < 4 * HV; ++r)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (i * 512 < ngr * 64)
            raw[r][i] = row_piece(r, u * 1024 + (i * 64 + lane) * 8);
      first_pieces(iA, S::NA);
      __builtin_amdgcn_sched_barrier(0);
      char *base = reinterpret_cast<char *>(lds) + u * 4096;
      auto at = [&](int r, int g, int s) {
        return reinterpret_cast<u4v *>(base + (r & 3) * S::PITCH * 4 + (r >> 2) * (ngr * 128) + g * 128 +
                                       ((s ^ (((g & 1) << 2) + (r & 3))) << 4));
      };
#pragma unroll
      for (int r = 0; r < 4 * HV; ++r)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (low && i * 512 < ngr * 64) *at(r, i * 8 + (lane >> 3), lane & 7) = raw[r][i];
      wave_fence();
#pragma unroll
      for (int h = 0; h < HV; ++h)
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const u4v q = *at(row + 4 * h, gl, s);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x[h][8 * s + 2 * e] = __uint_as_float(q[e] << 16);
            x[h][8 * s + 2 * e + 1] = __uint_as_float(q[e] & 0xffff0000u);
          }
        }
    } else {
      u4v raw[4 * HV][4];
#pragma unroll
      for (int r = 0; r < 4 * HV; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i * 256 < ngr * 64)
            raw[r][i] = row_piece(r, u * 1024 + (i * 64 + lane) * 4);
      first_pieces(iA, S::NA);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int h = 0; h < HV; ++h) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (low && i * 256 < ngr * 64)
              *reinterpret_cast<u4v *>(lds + pos4(r, u * 256 + i * 64 + lane)) = raw[4 * h + r][i];
        wave_fence();
#pragma unroll
        for (int s = 0; s < 16; ++s) {
          const f4v q = *reinterpret_cast<const f4v *>(lds + pos(row, u * 16 + gl, 4 * s));
#pragma unroll
          for (int e = 0; e < 4; ++e) x[h][4 * s + e] = q[e];
        }
        wave_fence();
      }
    }
    wave_fence();
    chain_stage<8, 8, 8, 1, S::NA>(x, ring, val, iA, iB);
    chain_stage<8, 8, 1, 8, S::NC>(x, ring, val, iB, iC);
    float y[LB][HV][H];
#pragma unroll
    for (int h = 0; h < HV; ++h) {
      if (low && slot < ngr) {
#pragma unroll
        for (int s = 0; s < 16; ++s)
          *reinterpret_cast<f4v *>(lds + pos(row, u * 16 + slot, 4 * s)) =
              (f4v){x[h][4 * s], x[h][4 * s + 1], x[h][4 * s + 2], x[h][4 * s + 3]};
      }
      lds_barrier();
#pragma unroll
      for (int b = 0; b < LB; ++b)
#pragma unroll
        for (int j = 0; j < H; ++j) y[b][h][j] = lds[pos(row, j, (w * LB + b) * 16 + slot)];
      lds_barrier();
    }
#pragma unroll
    for (int b = 0; b < LB; ++b) {
      chain_stage<R3, R4, R3, 1, S::ND>(y[b], ring, val, iC + b * S::NC, iD + b * S::ND);
      chain_stage<R4, R3, 1, R3, (S::LB > 1 ? S::NC : 0)>(y[b], ring, val, iD + b * S::ND,
                                                          iC + (b + 1 < LB ? b + 1 : b) * S::NC);
    }
    if constexpr (BO) {
#pragma unroll
      for (int b = 0; b < LB; ++b)
#pragma unroll
        for (int j = 0; j < H; ++j)
          lds[pos(row, j, (w * LB + b) * 16 + slot)] = __uint_as_float(pack2(y[b][0][j], y[b][HV - 1][j]));
      lds_barrier();
#pragma unroll
      for (int r = SHARE ? 0 : w; r < 4; r += SHARE ? 1 : NW) {
        if (SHARE && r >= nr) break;
#pragma unroll
        for (int i0 = 0; i0 < NR8; i0 += SHARE ? NW : 1) {
          const int i = i0 + (SHARE ? w : 0);
          if (i >= NR8) break;
          const int c = 2 * (i * 64 + lane);
          const u4v a = *reinterpret_cast<const u4v *>(lds + pos4(r, c + sw));
          const u4v b = *reinterpret_cast<const u4v *>(lds + pos4(r, c + 1 - sw));
          const u4v lo = sw ? b : a, hi = sw ? a : b;
          const u4v p0 = {__builtin_amdgcn_perm(lo[1], lo[0], 0x05040100u), __builtin_amdgcn_perm(lo[3], lo[2], 0x05040100u),
                          __builtin_amdgcn_perm(hi[1], hi[0], 0x05040100u), __builtin_amdgcn_perm(hi[3], hi[2], 0x05040100u)};
          const u4v p1 = {__builtin_amdgcn_perm(lo[1], lo[0], 0x07060302u), __builtin_amdgcn_perm(lo[3], lo[2], 0x07060302u),
                          __builtin_amdgcn_perm(hi[1], hi[0], 0x07060302u), __builtin_amdgcn_perm(hi[3], hi[2], 0x07060302u)};
          if (SHARE || r < nr) *reinterpret_cast<u4v *>(Yt + (int64_t)r * ldy + (i * 64 + lane) * 8) = p0;
          if (HV == 2 && r + 4 < nr) *reinterpret_cast<u4v *>(Yt + (int64_t)(r + 4) * ldy + (i * 64 + lane) * 8) = p1;
        }
      }
    } else {
#pragma unroll
      for (int h = 0; h < HV; ++h) {
        if (h) lds_barrier();
#pragma unroll
        for (int b = 0; b < LB; ++b)
#pragma unroll
          for (int j = 0; j < H; ++j) lds[pos(row, j, (w * LB + b) * 16 + slot)] = y[b][h][j];
        lds_barrier();
#pragma unroll
        for (int r = SHARE ? 0 : w; r < 4; r += SHARE ? 1 : NW)
          if (4 * h + r < nr) {
#pragma unroll
            for (int i = SHARE ? w : 0; i < NR4; i += SHARE ? NW : 1)
              *reinterpret_cast<u4v *>(Yt + (int64_t)(4 * h + r) * ldy + (i * 64 + lane) * 4) =
                  *reinterpret_cast<const u4v *>(lds + pos4(r, i * 64 + lane));
          }
      }
    }
  } else {
    float y[LB][HV][H];
    if constexpr (TOP > 0) {
      // The stage above the chunk on the way in: coordinate c of the chunk is the sum over the row's TOP chunks of
      // x[j][c] K_c[j][kch], in the order in which the stage's own kernel adds.  A wave takes the same coordinates of all
      // rows, so their TOP values of K are read once per tile.  (The row is read once per chunk, the last TOP - 1 times from
      // the caches.)
      constexpr int PW = (NR4 + NW - 1) / NW;
      f4v z[PW][4 * HV];
      first_pieces(iD, S::ND);
#pragma unroll
      for (int k = 0; k < PW; ++k) {
        const int c = ((w + k * NW < NR4 ? w + k * NW : NR4 - 1) * 64 + lane) * 4;   // (past the end the last ones once more)
        f4v f[TOP];
#pragma unroll
        for (int j = 0; j < TOP; ++j)
          f[j] = *reinterpret_cast<const f4v *>(tparams + (size_t)(j * TOP + kch) * S::CHUNK + c);
#pragma unroll
        for (int r = 0; r < 4 * HV; ++r) {
          const TI *p = Xt + (int64_t)(r < nr ? r : nr - 1) * ldx + c;
#pragma unroll
          for (int j = 0; j < TOP; ++j) {
            float x[4];
            if constexpr (BI) {
              const uint2 q = *reinterpret_cast<const uint2 *>(p + (int64_t)j * S::CHUNK);
              x[0] = __uint_as_float(q.x << 16);
              x[1] = __uint_as_float(q.x & 0xffff0000u);
              x[2] = __uint_as_float(q.y << 16);
              x[3] = __uint_as_float(q.y & 0xffff0000u);
            } else {
              const f4v q = *reinterpret_cast<const f4v *>(p + (int64_t)j * S::CHUNK);
#pragma unroll
              for (int e = 0; e < 4; ++e) x[e] = q[e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) z[k][r][e] = j == 0 ? x[e] * f[0][e] : fmaf(x[e], f[j][e], z[k][r][e]);
          }
        }
      }
#pragma unroll
      for (int h = 0; h < HV; ++h) {
        if (h) lds_barrier();
#pragma unroll
        for (int k = 0; k < PW; ++k)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            *reinterpret_cast<f4v *>(lds + pos4(r, (w + k * NW < NR4 ? w + k * NW : NR4 - 1) * 64 + lane)) = z[k][4 * h + r];
        lds_barrier();
#pragma unroll
        for (int b = 0; b < LB; ++b)
#pragma unroll
          for (int j = 0; j < H; ++j) y[b][h][j] = lds[pos(row, j, (w * LB + b) * 16 + slot)];
      }
    } else if constexpr (BI) {
      u4v raw[LB][HV][NR8];   // wave w: rows w (w, w + 2) and the one four further on
#pragma unroll
      for (int k = 0; k < LB; ++k)
#pragma unroll
        for (int h = 0; h < HV; ++h)
#pragma unroll
          for (int i = 0; i < NR8; ++i)
            raw[k][h][i] = row_piece(w + k * NW + 4 * h, (i * 64 + lane) * 8);
      first_pieces(iD, S::ND);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < LB; ++k)
#pragma unroll
        for (int i = 0; i < NR8; ++i) {
          const u4v p = raw[k][0][i], q = raw[k][HV - 1][i];
          u4v a, b;
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            a[2 * e] = __builtin_amdgcn_perm(q[e], p[e], 0x05040100u);
            a[2 * e + 1] = __builtin_amdgcn_perm(q[e], p[e], 0x07060302u);
            b[2 * e] = __builtin_amdgcn_perm(q[2 + e], p[2 + e], 0x05040100u);
            b[2 * e + 1] = __builtin_amdgcn_perm(q[2 + e], p[2 + e], 0x07060302u);
          }
          const int c = 2 * (i * 64 + lane);
          *reinterpret_cast<u4v *>(lds + pos4(w + k * NW, c + sw)) = sw ? b : a;
          *reinterpret_cast<u4v *>(lds + pos4(w + k * NW, c + 1 - sw)) = sw ? a : b;
        }
      lds_barrier();
#pragma unroll
      for (int b = 0; b < LB; ++b)
#pragma unroll
        for (int j = 0; j < H; ++j) {
          const uint32_t q = __float_as_uint(lds[pos(row, j, (w * LB + b) * 16 + slot)]);
          y[b][0][j] = __uint_as_float(q << 16);
          if constexpr (HV == 2) y[b][1][j] = __uint_as_float(q & 0xffff0000u);
        }
    } else {
      u4v raw[HV][LB][NR4];
#pragma unroll
      for (int h = 0; h < HV; ++h)
#pragma unroll
        for (int k = 0; k < LB; ++k)
#pragma unroll
          for (int i = 0; i < NR4; ++i)
            raw[h][k][i] = row_piece(4 * h + w + k * NW, (i * 64 + lane) * 4);
      first_pieces(iD, S::ND);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int h = 0; h < HV; ++h) {
        if (h) lds_barrier();
#pragma unroll
        for (int k = 0; k < LB; ++k)
#pragma unroll
          for (int i = 0; i < NR4; ++i)
            *reinterpret_cast<u4v *>(lds + pos4(w + k * NW, i * 64 + lane)) = raw[h][k][i];
        lds_barrier();
#pragma unroll
        for (int b = 0; b < LB; ++b)
#pragma unroll
          for (int j = 0; j < H; ++j) y[b][h][j] = lds[pos(row, j, (w * LB + b) * 16 + slot)];
      }
    }
#pragma unroll
    for (int b = 0; b < LB; ++b) {
      chain_stage<R4, R3, 1, R3, S::NC>(y[b], ring, val, iD + b * S::ND, iC + b * S::NC);
      if (b + 1 < LB)
        chain_stage<R3, R4, R3, 1, S::ND>(y[b], ring, val, iC + b * S::NC, iD + (b + 1 < LB ? b + 1 : b) * S::ND);
      else
        chain_stage<R3, R4, R3, 1, S::NA>(y[b], ring, val, iC + b * S::NC, iB);
    }
    float x[HV][64];
#pragma unroll
    for (int h = 0; h < HV; ++h) {
      lds_barrier();   // everyone has read the rows that are overwritten here
#pragma unroll
      for (int b = 0; b < LB; ++b)
#pragma unroll
        for (int j = 0; j < H; ++j) lds[pos(row, j, (w * LB + b) * 16 + slot)] = y[b][h][j];
      lds_barrier();
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const f4v q = *reinterpret_cast<const f4v *>(lds + pos(row, u * 16 + gl, 4 * s));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[h][4 * s + e] = q[e];
      }
    }
    wave_fence();
    chain_stage<8, 8, 1, 8, S::NA>(x, ring, val, iB, iA);
    chain_stage<8, 8, 8, 1, 0>(x, ring, val, iA, iA);
    // back through the wave's own part of the LDS rows: 16-byte stores of whole lines
    if constexpr (BO) {
      char *base = reinterpret_cast<char *>(lds) + u * 4096;
      auto at = [&](int r, int g, int s) {
        return reinterpret_cast<u4v *>(base + (r & 3) * S::PITCH * 4 + (r >> 2) * (ngr * 128) + g * 128 +
                                       ((s ^ (((g & 1) << 2) + (r & 3))) << 4));
      };
      if (low && slot < ngr) {
#pragma unroll
        for (int h = 0; h < HV; ++h)
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            u4v q;
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = pack2(x[h][8 * s + 2 * e], x[h][8 * s + 2 * e + 1]);
            *at(row + 4 * h, slot, s) = q;
          }
      }
      wave_fence();
#pragma unroll
      for (int r = 0; r < 4 * HV; ++r)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (low && i * 512 < ngr * 64 && (!SHARE || r < nr)) {
            const u4v q = *at(r, i * 8 + (lane >> 3), lane & 7);
            if (r < nr) *reinterpret_cast<u4v *>(Yt + (int64_t)r * ldy + u * 1024 + (i * 64 + lane) * 8) = q;
          }
    } else {
#pragma unroll
      for (int h = 0; h < HV; ++h) {
        if (low && slot < ngr) {
#pragma unroll
          for (int s = 0; s < 16; ++s)
            *reinterpret_cast<f4v *>(lds + pos(row, u * 16 + slot, 4 * s)) =
                (f4v){x[h][4 * s], x[h][4 * s + 1], x[h][4 * s + 2], x[h][4 * s + 3]};
        }
        wave_fence();
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (low && i * 256 < ngr * 64 && (!SHARE || r < nr)) {
              const u4v q = *reinterpret_cast<const u4v *>(lds + pos4(r, u * 256 + i * 64 + lane));
              if (4 * h + r < nr)
                *reinterpret_cast<u4v *>(Yt + (int64_t)(4 * h + r) * ldy + u * 1024 + (i * 64 + lane) * 4) = q;
            }
        wave_fence();
      }
    }
  }
}

template <typename TI, typename TO, int R4, bool TRN, int HV, int TOP = 0>
harp_status_t launch_chain_rows(const harp_plan *plan, const ChainImage &ci, const void *X, int64_t ldx, void *Y,
                                int64_t ldy, int64_t n, hipStream_t stream, const float *tparams = nullptr) {
  using S = ChainShape<R4, HV>;
  constexpr size_t lds = (size_t)4 * S::PITCH * 4;
  if (lds > (size_t)plan->lds_bytes) return HARP_ERR_UNSUPPORTED;
  int R = 4 * HV;
  if (plan->rows_override > 0 && plan->rows_override < R) R = plan->rows_override;
  const int nchunk = (int)(plan->d / S::CHUNK);
  const int64_t ntile = (n + R - 1) / R;
  const int64_t total = ntile * nchunk;
  if (total > 0x7ffffff0) return HARP_ERR_UNSUPPORTED;
  auto kern = harp_chain_kernel<TI, TO, R4, TRN, HV, TOP>;
  static thread_local int attr_done_dev = -1;   // per instantiation
  if (attr_done_dev != plan->device) {
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            plan->lds_bytes) != hipSuccess) {
      (void)hipGetLastError();
      return HARP_ERR_DEVICE;
    }
    attr_done_dev = plan->device;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)((total + 7) / 8 * 8)), dim3(64 * S::NW), lds, stream, (const TI *)X, ldx,
                     (TO *)Y, ldy, n, R, (unsigned)ntile, (unsigned)total, ci.img, tparams);
  return hipGetLastError() == hipSuccess ? HARP_OK : HARP_ERR_DEVICE;
}

bool chain_rows_of_four(const harp_plan *plan, int64_t n, int chunk) {
  const int64_t cus = plan->num_cu > 0 ? plan->num_cu : 256;
  return plan->rows_override > 0 ? plan->rows_override <= 4 : (n + 3) / 4 * (plan->d / chunk) <= cus;
}

template <typename TI, typename TO, int R4, bool TRN>
harp_status_t launch_chain_inst(const harp_plan *plan, const ChainImage &ci, const void *X, int64_t ldx, void *Y,
                                int64_t ldy, int64_t n, hipStream_t stream) {
  // Tiles of four rows while they are no more than compute units: each is done sooner (a stage's products are
  // half), and the units with a tile of eight would otherwise stand beside idle ones.  Beyond that a tile of eight
  // uses the block values twice as often.  Eight / four rows, bf16, us: 4096 at 1 row 9.8 / 6.9, 512 rows 10.6 / 8.2,
  // 1024 rows (256 tiles) 12.0 / 9.6, 1030 rows 12.1 / 13.8; 14336 (two launches) at 6 rows 12.5 / 9.9, 256 rows (256 tiles)
  // 17.9 / 15.7, 512 rows 23.0 / 24.0; 2048 at 1024 rows 8.9 / 5.8.
  return chain_rows_of_four(plan, n, ChainShape<R4>::CHUNK) ? launch_chain_rows<TI, TO, R4, TRN, 1>(plan, ci, X, ldx, Y, ldy, n, stream)
              : launch_chain_rows<TI, TO, R4, TRN, 2>(plan, ci, X, ldx, Y, ldy, n, stream);
}

template <int R4>
harp_status_t launch_chain_shape(const harp_plan *plan, const ChainImage &ci, const void *X, int64_t ldx,
                                 harp_dtype_t dt_in, void *Y, int64_t ldy, harp_dtype_t dt_out, int64_t n,
                                 hipStream_t stream) {
#define HARP_CHAIN_IO(TI, TO)                                                                  \
  (ci.trn ? launch_chain_inst<TI, TO, R4, true>(plan, ci, X, ldx, Y, ldy, n, stream)      \
          : launch_chain_inst<TI, TO, R4, false>(plan, ci, X, ldx, Y, ldy, n, stream))
  if (dt_in == HARP_BF16)
    return dt_out == HARP_BF16 ? HARP_CHAIN_IO(uint16_t, uint16_t) : HARP_CHAIN_IO(uint16_t, float);
  if (dt_out == HARP_F32) return HARP_CHAIN_IO(float, float);
  // float32 in, bf16 out: only behind the streamed stages of a transposed split program
  if (!ci.trn) return HARP_ERR_UNSUPPORTED;
  return launch_chain_inst<float, uint16_t, R4, true>(plan, ci, X, ldx, Y, ldy, n, stream);
#undef HARP_CHAIN_IO
}

template <int R4>
void pack_chain(const Program &pg, int p0, bool trn, const std::vector<size_t> &offsets, int64_t nchunk,
                std::vector<float> &image, size_t off) {
  using S = ChainShape<R4>;
  for (int e = 0; e < 4; ++e) {   // the stages by stride
    const int p = trn ? p0 + 3 - e : p0 + e, b = pg.pass[p].b, nh = b > 4 ? 2 : 1, np = chain_pieces(b);
    const int64_t nq = pg.pass[p].nq, s = pg.pass[p].S, nqc = S::CHUNK / b;
    const int units = e < 2 ? S::UNITS : 4, batches = e < 2 ? 8 : (e == 2 ? R4 : R3);
    const int64_t base = e == 0 ? 0 : (e == 1 ? S::OFF_B : (e == 2 ? S::OFF_C : S::OFF_D));
    for (int64_t k = 0; k < nchunk; ++k)
      for (int u = 0; u < units; ++u) {
        // (past the chunk's groups: zeros)
        const int slots = e < 2 && S::H - 16 * u < 16 ? S::H - 16 * u : 16;
        for (int v = 0; v < batches; ++v)
          for (int r = 0; r < b; ++r)
            for (int c = 0; c < b; ++c) {
              const int w = r * nh + c / 4;
              const float *from = image.data() + offsets[p] + (size_t)(r * b + c) * nq + k * nqc;
              float *to = image.data() + off + (size_t)(k * S::TOTAL + base) +
                          ((((size_t)u * batches + v) * np + w / 4) * 64 + c % 4) * 4 + w % 4;
              for (int slot = 0; slot < slots; ++slot) {
                // coordinate of the block's input 0 inside the chunk, then the block
                const int64_t c0 = e == 0   ? (u * 16 + slot) * 64 + 8 * v
                                   : e == 1 ? (u * 16 + slot) * 64 + v
                                   : e == 2 ? (int64_t)v * 64 * R3 + u * 16 + slot
                                            : (int64_t)v * 64 + u * 16 + slot;
                to[slot * 16] = from[(c0 / (b * s)) * s + c0 % s];
              }
            }
      }
  }
}

#define HARP_CHAIN_R4(r4, STMT)                              \
  switch (r4) {                                               \
    case 3: { constexpr int R4 = 3; STMT; } break;            \
    case 4: { constexpr int R4 = 4; STMT; } break;            \
    case 5: { constexpr int R4 = 5; STMT; } break;            \
    case 6: { constexpr int R4 = 6; STMT; } break;            \
    case 7: { constexpr int R4 = 7; STMT; } break;            \
    default: { constexpr int R4 = 8; STMT; } break;           \
  }

}  // namespace

// The chunk passes [p0, p0 + np) as a chain of radices 8, 8, 8, R4: appends the block values in the
// kernel's order to the program's host image.
void build_chain_image(HostProgram &hp, int p0, int np, int64_t d, const std::vector<size_t> &offsets,
                       std::vector<float> &image) {
  hp.chain = ChainImage();
  if (np != 4) return;
  const Program &pg = hp.prog;
  const bool trn = pg.pass[p0].S != 1;
  int64_t s = 1;
  for (int e = 0; e < 4; ++e) {
    const PassDesc &pd = pg.pass[trn ? p0 + 3 - e : p0 + e];
    if (pd.kind != PASS_SMALL || pd.tied || pd.S != s || (e < 3 ? pd.b != 8 : pd.b < 3)) return;
    s *= pd.b;
  }
  if (s != hp.chunk || d % s) return;
  const int r4 = pg.pass[trn ? p0 : p0 + 3].b;
  const size_t off = (image.size() + 63) / 64 * 64;
  const int64_t nchunk = d / s;
  HARP_CHAIN_R4(r4, (image.resize(off + (size_t)(nchunk * ChainShape<R4>::TOTAL), 0.0f),
                     pack_chain<R4>(pg, p0, trn, offsets, nchunk, image, off)));
  hp.chain.host_off = (int64_t)off;
  hp.chain.r4 = r4;
  hp.chain.trn = trn;
}

harp_status_t launch_chain_kernel(const harp_plan *plan, const ChainImage &ci, const void *X, int64_t ldx,
                                  harp_dtype_t dt_in, void *Y, int64_t ldy, harp_dtype_t dt_out, int64_t n,
                                  hipStream_t stream) {
  harp_status_t st = HARP_ERR_UNSUPPORTED;
  HARP_CHAIN_R4(ci.r4, (st = launch_chain_shape<R4>(plan, ci, X, ldx, dt_in, Y, ldy, dt_out, n, stream)));
  return st;
}

// Transposed split program whose one stage above the chain has radix 2 .. 4: one launch, no intermediate (bf16: 12 bytes per
// coordinate become 4).  Not in place: a workgroup may store its chunk of a row before another one has read it.  Larger radices are
// neither built nor measured: a row would be read that many times.  Two launches / one, us, bf16: 8192 (8, 8, 8, 8 | 2) at 1 row 9.6 / 8.0, 514 rows
// 19.3 / 15.0, 2048 rows 51 / 25; 14336 (8, 8, 8, 7 | 4) at 8 rows 10.2 / 9.2, 300 rows 19.6 / 17.7, 777 rows 35 / 27, 2048 rows
// 82 / 57; float32: 5120 (8, 8, 8, 5 | 2) at 3000 rows 58 / 36, 14336 at 777 rows 45 / 33.  Tiles of eight go row by row over an XCD; with a
// run of tiles of one chunk, as without the stage, the row came from memory TOP times (14336: 777 rows 30, 2048 rows 68).
// Tiles of four keep that order: few rows are less than the block values (20 rows of 14336 11.3 -> 10.6).
bool chain_top_supported(const harp_plan *plan, const HostProgram &hp, const void *X, int64_t ldx, harp_dtype_t dt_in,
                         const void *Y, int64_t ldy, harp_dtype_t dt_out) {
  const PassDesc &pd = hp.prog.pass[0];
  if (!hp.chain.img || !hp.chain.trn || hp.chunk_first || hp.prog.npass != hp.n_chunk + 1 || X == Y) return false;
  if (dt_in != dt_out || !radix_supported(plan, hp, 1, hp.n_chunk, hp.chunk, X, ldx, Y, ldy) ||
      radix_rebuilds_in_kernel(plan, hp.prog, 1, hp.n_chunk, hp.chunk))
    return false;
  const bool dense = (pd.kind == PASS_SMALL && (pd.b == 3 || pd.b == 4)) ||
                     (pd.kind == PASS_POW2_DENSE && pd.k == 1 && pd.P == 2 && pd.V == 4);
  return dense && !pd.tied && pd.nq == hp.chunk && pd.nqp == hp.chunk && pd.S == hp.chunk && (uintptr_t)pd.params % 16 == 0;
}

harp_status_t launch_chain_top(const harp_plan *plan, const HostProgram &hp, const void *X, int64_t ldx, void *Y, int64_t ldy,
                               harp_dtype_t dt, int64_t n, hipStream_t stream) {
  const PassDesc &pd = hp.prog.pass[0];
  harp_status_t st = HARP_ERR_UNSUPPORTED;
  const bool four = chain_rows_of_four(plan, n, hp.chunk);
#define HARP_CHAIN_TOP_T(T, TX, HV) \
  (launch_chain_rows<TX, TX, R4, true, HV, T>(plan, hp.chain, X, ldx, Y, ldy, n, stream, pd.params))
#define HARP_CHAIN_TOP(T)                                                                                             \
  HARP_CHAIN_R4(hp.chain.r4, st = dt == HARP_BF16 ? (four ? HARP_CHAIN_TOP_T(T, uint16_t, 1) : HARP_CHAIN_TOP_T(T, uint16_t, 2)) \
                                                  : (four ? HARP_CHAIN_TOP_T(T, float, 1) : HARP_CHAIN_TOP_T(T, float, 2)))
  if (pd.P == 2) HARP_CHAIN_TOP(2)
  else if (pd.P == 3) HARP_CHAIN_TOP(3)
  else if (pd.P == 4) HARP_CHAIN_TOP(4)
#undef HARP_CHAIN_TOP
#undef HARP_CHAIN_TOP_T
  return st;
}

}  // namespace harp
