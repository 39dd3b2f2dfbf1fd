// Building blocks of the kernels that multiply small dense blocks on v_mfma_f32_4x4x1_16b_f32 (sixteen
// independent 4 x 4 outer-product updates): harp_chain.hip (rows), harp_colwide.hip and harp_colpair.hip
// (columns).  The barrier is harp_grad.hip's as well.
#ifndef HARP_MFMA4_H_
#define HARP_MFMA4_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace harp {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

// registers (16-byte pieces) of one lane for one stage batch: B inputs times one or two halves of the outputs
constexpr int chain_pieces(int B) { return (B * (B > 4 ? 2 : 1) + 3) / 4; }

#if defined(__HIPCC__)
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  bf2 v;
  v.x = (__bf16)lo;
  v.y = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

// Block values in device memory, pieces of PB bytes: a buffer descriptor, so that a piece is addressed by one register (16
// times the lane's place in it), a scalar offset and an immediate.  With 64-bit addresses the compiler kept one per
// piece, spilled them, and every reload waited for all loads in flight (a stage took twice as long).
template <int PB>
struct BlockValues {
  __amdgpu_buffer_rsrc_t rsrc;
  int voff;
  __device__ __forceinline__ f4v piece(int stage_piece, int s) const {   // piece s of the stage that starts at piece stage_piece
    return __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, (stage_piece + s) * PB, 0));
  }
};

// One stage on the registers of a lane, G independent sets of coordinates: NB blocks of radix B, input r of
// block v at x[v * SV + r * SR].
// Piece s of the stage lies in ring slot s % RING.  A slot that has been used takes the stage's piece
// RING further on, or, when there is none, the next stage's piece of that slot.
template <int B, int NB, int SV, int SR, int NNEXT, int G, int NX, int RING, int PB>
__device__ __forceinline__ void chain_stage(float (&x)[G][NX], f4v (&ring)[RING], const BlockValues<PB> &val, int own,
                                            int next) {
  constexpr int NH = B > 4 ? 2 : 1, NP = chain_pieces(B), CNT = NB * NP;
#pragma unroll
  for (int s = CNT; s < RING; ++s)   // slots the stage does not use
    if (s < NNEXT) ring[s] = val.piece(next, s);
#pragma unroll
  for (int v = 0; v < NB; ++v) {
    f4v acc[G][NH];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int h = 0; h < NH; ++h) acc[g][h] = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < B; ++r)
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int g = 0; g < G; ++g)
          acc[g][h] = __builtin_amdgcn_mfma_f32_4x4x1f32(ring[(v * NP + (r * NH + h) / 4) % RING][(r * NH + h) % 4],
                                                         x[g][v * SV + r * SR], acc[g][h], 0, 0, 0);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int c = 0; c < B; ++c) x[g][v * SV + c * SR] = acc[g][c / 4][c % 4];
#pragma unroll
    for (int s = v * NP; s < (v + 1) * NP; ++s) {
      if (s + RING < CNT)
        ring[s % RING] = val.piece(own, s + RING);
      else if (s % RING < NNEXT)
        ring[s % RING] = val.piece(next, s % RING);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

__device__ __forceinline__ void lds_barrier() {   // LDS only: loads in flight stay in flight
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ void wave_fence() {   // other lanes of this wave read what it wrote to LDS
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
#endif

}  // namespace harp
#endif
